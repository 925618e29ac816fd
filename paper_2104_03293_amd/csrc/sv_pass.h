// The tile pass and its launch variants (see sv_kernels.hip for how a pass works).
// The instantiations are spread over sv_pass_*.hip: each is a large straight-line
// kernel, and one file with all of them takes minutes to compile.
#pragma once
#include <hip/hip_runtime.h>

#include "sv_device.h"
#include "sv_internal.h"

namespace svk {

// Value of the lane whose id differs in one bit, per 32-bit word: lane bit 3
// by a DPP row_ror:8 move (within a 16-lane row), lane bit 4 by a ds_swizzle
// in bit mode (and 0x1f, xor 0x10 within 32 lanes; no LDS storage).
constexpr int kLaneX8 = 0x128;
constexpr int kLaneX16 = 0x10000 | (0x10 << 10) | 0x1f;
template <int CTRL>
__device__ __forceinline__ int lane_xor_word(int w) {
    if constexpr (CTRL & 0x10000)
        return __builtin_amdgcn_ds_swizzle(w, CTRL & 0xffff);
    else
        return __builtin_amdgcn_update_dpp(0, w, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_xor(float x) {
    return __int_as_float(lane_xor_word<CTRL>(__float_as_int(x)));
}
template <int CTRL>
__device__ __forceinline__ double lane_xor(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = lane_xor_word<CTRL>((int)(b & 0xffffffffll));
    const int hi = lane_xor_word<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Butterfly of one qubit held by a lane bit: both lanes of a pair apply
// x <- x - i t x_partner (the same form for the upper and the lower member).
// With gradient accumulation each lane adds Im(conj(lam_self) psi_partner), so
// that the pair sum of the register form is split over the two lanes.
template <int CTRL, typename Real, int R, int NV, bool QF = false>
__device__ __forceinline__ void lane_round(Real (&vr)[NV][1 << R], Real (&vi)[NV][1 << R], int flags, Real t,
                                           double cosb, double (&pend)[NV], double& gsum) {
    constexpr int NR = 1 << R;
    if constexpr (NV == 2) {
        if (flags & MIX_GBETA) {
            double gb = 0.0;
#pragma unroll
            for (int r = 0; r < NR; r++) {
                const Real pr = lane_xor<CTRL>(vr[0][r]), pi = lane_xor<CTRL>(vi[0][r]);
                gb += (double)(vr[1][r] * pi - vi[1][r] * pr);
            }
            gsum += gb * pend[0] * pend[1];
        }
    }
#pragma unroll
    for (int v = 0; v < NV; v++) {
        const bool mine = NV == 1 || (flags & (1 << v)) != 0;
        const Real tv = mine ? t : (Real)0;
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const Real pr = lane_xor<CTRL>(vr[v][r]), pi = lane_xor<CTRL>(vi[v][r]);
            vr[v][r] = fma(tv, pi, vr[v][r]);
            vi[v][r] = fma(-tv, pr, vi[v][r]);
        }
        pend[v] *= mine ? cosb : 1.0;
    }
    if constexpr (NV == 1 && QF) {
        if (flags & MIX_GBETA) {
            // one-vector quadratic form, taken after the butterfly (which leaves it unchanged)
            // in a loop of its own: each lane adds Re(conj(self) partner), so the two lanes
            // of a pair give 2 Re(conj(a) b)
            double gq[2] = {0.0, 0.0};
#pragma unroll
            for (int r = 0; r < NR; r++) {
                const Real pr = lane_xor<CTRL>(vr[0][r]), pi = lane_xor<CTRL>(vi[0][r]);
                gq[r & 1] = fma((double)vr[0][r], (double)pr, gq[r & 1]);
                gq[r & 1] = fma((double)vi[0][r], (double)pi, gq[r & 1]);
                // keep the scheduler from hoisting every cross-lane move ahead of the sums
                // (their results would all be live at once)
                if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            gsum += (gq[0] + gq[1]) * pend[0] * pend[0];
        }
    }
}

// Butterflies of every active register slot of the current layout; each slot
// multiplies the pending scale of the touched vectors by cos(beta).  With
// gradient accumulation the pair terms Im(conj(lam_a) psi_b) + Im(conj(lam_b) psi_a)
// are taken before each slot's butterfly, weighted by both pending scales.
template <typename Real, int R, int NV, bool QF = false>
__device__ __forceinline__ void mix_round(Real (&vr)[NV][1 << R], Real (&vi)[NV][1 << R], int act, int flags,
                                          Real t, double cosb, double (&pend)[NV], double& gsum) {
    constexpr int NR = 1 << R;
#pragma unroll
    for (int k = 0; k < R; k++) {
        // inactive slots run as identity butterflies (t = 0, no scale): branch-free
        // code keeps the amplitude registers in place
        const bool on = (act >> k) & 1;
        const Real tk = on ? t : (Real)0;
        if constexpr (NV == 2) {
            if ((flags & MIX_GBETA) && on) {
                double gb = 0.0;
                if constexpr (sizeof(Real) == 8) {
                    // complex128: the four products of each pair fused into two
                    // alternating FP64 accumulators
                    double g2 = 0.0;
#pragma unroll
                    for (int r = 0; r < NR; r++) {
                        if (r & (1 << k)) continue;
                        const int r2 = r | (1 << k);
                        double& acc = ((r >> (k == 0 ? 1 : 0)) & 1) ? g2 : gb;
                        acc = fma(vr[1][r], vi[0][r2], acc);
                        acc = fma(-vi[1][r], vr[0][r2], acc);
                        acc = fma(vr[1][r2], vi[0][r], acc);
                        acc = fma(-vi[1][r2], vr[0][r], acc);
                    }
                    gb += g2;
                } else {
#pragma unroll
                    for (int r = 0; r < NR; r++) {
                        if (r & (1 << k)) continue;
                        const int r2 = r | (1 << k);
                        // pair term in the storage precision, summed in FP64 (FP64 products
                        // change the complex64 gradient by ~1e-10 of the coefficient scale, far
                        // below the f32 rounding of the stored vectors, and spill the
                        // four-waves-per-SIMD kernels)
                        const Real q = vr[1][r] * vi[0][r2] - vi[1][r] * vr[0][r2] + vr[1][r2] * vi[0][r] -
                                       vi[1][r2] * vr[0][r];
                        gb += (double)q;
                    }
                }
                gsum += gb * pend[0] * pend[1];
            }
        }
#pragma unroll
        for (int v = 0; v < NV; v++) {
            // A vector the op does not touch runs identity butterflies (t = 0)
            // instead of a branch, which would force register copies at the
            // join.  One-vector passes always mix psi.
            const bool mine = NV == 1 || (flags & (1 << v)) != 0;
            const Real tv = mine ? tk : (Real)0;
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (r & (1 << k)) continue;
                const int r2 = r | (1 << k);
                butterfly<Real>(vr[v][r], vi[v][r], vr[v][r2], vi[v][r2], tv);
            }
            pend[v] *= (on && mine) ? cosb : 1.0;
        }
    }
    if constexpr (NV == 1 && QF) {
        if (flags & MIX_GBETA) {
            // quadratic forms 2 Re(conj(a) b) of the pairs of every active slot.  A butterfly
            // on any qubit leaves the form of every other qubit unchanged, so all of them are
            // taken once, after the round, from the final values and pending scale.
            double g4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < R; k++) {
                if (!((act >> k) & 1)) continue;
                int j = 0;
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    if (r & (1 << k)) continue;
                    const int r2 = r | (1 << k);
                    double& acc = g4[j++ & 3];
                    acc = fma((double)vr[0][r], (double)vr[0][r2], acc);
                    acc = fma((double)vi[0][r], (double)vi[0][r2], acc);
                }
            }
            gsum += 2.0 * ((g4[0] + g4[1]) + (g4[2] + g4[3])) * pend[0] * pend[0];
        }
    }
}

// General single-qubit layer, register slots: slot k holds tile bit
// (rbpack >> 4k) & 15 and applies that bit's matrix M[l] to every register
// pair (bit k = 0, bit k = 1).  Inactive slots read the identity entry of tile
// bit 15 (never a qubit of a 13- or 14-bit tile), which keeps the code
// branch-free.  REALM: every matrix is real (two FMAs per amplitude instead
// of eight).  unit: every matrix has a unit diagonal (one FMA per amplitude
// for real matrices, four for complex ones).  The matrices are read through
// the constant address space (the host writes them before the launch): scalar
// loads of every slot's entries, issued together ahead of the butterflies.
template <typename Real, int R, bool REALM, bool UNIT>
__device__ __forceinline__ void gen_round(Real (&vr)[1][1 << R], Real (&vi)[1][1 << R], int act, uint32_t rbpack,
                                          const SV_CONST double* __restrict__ M) {
    constexpr int NR = 1 << R;
    if constexpr (UNIT) {
        // off-diagonal entries only: (u, v) <- (u + m01 v, m10 u + v)
        Real mo[R][4];  // slot k: m01 re, m10 re, m01 im, m10 im
#pragma unroll
        for (int k = 0; k < R; k++) {
            const bool on = (act >> k) & 1;
            const SV_CONST double* m = M + 8 * (on ? ((rbpack >> (4 * k)) & 15u) : 15u);
            mo[k][0] = (Real)m[2];
            mo[k][1] = (Real)m[4];
            if constexpr (!REALM) {
                mo[k][2] = (Real)m[3];
                mo[k][3] = (Real)m[5];
            }
        }
#pragma unroll
        for (int k = 0; k < R; k++) {
            const Real b0 = mo[k][0], c0 = mo[k][1];
            Real b1 = 0, c1 = 0;
            if constexpr (!REALM) {
                b1 = mo[k][2];
                c1 = mo[k][3];
            }
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (r & (1 << k)) continue;
                const int r2 = r | (1 << k);
                const Real ur = vr[0][r], ui = vi[0][r], wr = vr[0][r2], wi = vi[0][r2];
                if constexpr (REALM) {
                    vr[0][r] = fma(b0, wr, ur);
                    vi[0][r] = fma(b0, wi, ui);
                    vr[0][r2] = fma(c0, ur, wr);
                    vi[0][r2] = fma(c0, ui, wi);
                } else {
                    vr[0][r] = fma(b0, wr, fma(-b1, wi, ur));
                    vi[0][r] = fma(b0, wi, fma(b1, wr, ui));
                    vr[0][r2] = fma(c0, ur, fma(-c1, ui, wr));
                    vi[0][r2] = fma(c0, ui, fma(c1, ur, wi));
                }
            }
        }
    } else {
    Real me[R][8];  // slot k: a0 b0 c0 d0 (real parts), then a1 b1 c1 d1 (imaginary parts)
#pragma unroll
    for (int k = 0; k < R; k++) {
        const bool on = (act >> k) & 1;
        const SV_CONST double* m = M + 8 * (on ? ((rbpack >> (4 * k)) & 15u) : 15u);
#pragma unroll
        for (int j = 0; j < 4; j++) me[k][j] = (Real)m[2 * j];
        if constexpr (!REALM) {
#pragma unroll
            for (int j = 0; j < 4; j++) me[k][4 + j] = (Real)m[2 * j + 1];
        }
    }
#pragma unroll
    for (int k = 0; k < R; k++) {
        const Real a0 = me[k][0], b0 = me[k][1], c0 = me[k][2], d0 = me[k][3];
        Real a1 = 0, b1 = 0, c1 = 0, d1 = 0;
        if constexpr (!REALM) {
            a1 = me[k][4];
            b1 = me[k][5];
            c1 = me[k][6];
            d1 = me[k][7];
        }
#pragma unroll
        for (int r = 0; r < NR; r++) {
            if (r & (1 << k)) continue;
            const int r2 = r | (1 << k);
            const Real ur = vr[0][r], ui = vi[0][r], wr = vr[0][r2], wi = vi[0][r2];
            if constexpr (REALM) {
                vr[0][r] = fma(a0, ur, b0 * wr);
                vi[0][r] = fma(a0, ui, b0 * wi);
                vr[0][r2] = fma(c0, ur, d0 * wr);
                vi[0][r2] = fma(c0, ui, d0 * wi);
            } else {
                vr[0][r] = fma(a0, ur, fma(-a1, ui, fma(b0, wr, -b1 * wi)));
                vi[0][r] = fma(a0, ui, fma(a1, ur, fma(b0, wi, b1 * wr)));
                vr[0][r2] = fma(c0, ur, fma(-c1, ui, fma(d0, wr, -d1 * wi)));
                vi[0][r2] = fma(c0, ui, fma(c1, ur, fma(d0, wi, d1 * wr)));
            }
        }
    }
    }
}

// General single-qubit layer, lane bit POS (the partner lane is lane ^ 2^POS):
// the lane whose bit is 0 holds u and forms m00 u + m01 v, its partner forms
// m10 u + m11 v.  l is the tile bit of that lane position.  Both rows are read
// as scalars; each lane selects its own.  unit: unit diagonal, each lane adds
// its off-diagonal entry times the partner's value to its own.
template <int CTRL, int POS, typename Real, int R, bool REALM, bool UNIT>
__device__ __forceinline__ void gen_lane(Real (&vr)[1][1 << R], Real (&vi)[1][1 << R], int l,
                                         const SV_CONST double* __restrict__ M) {
    constexpr int NR = 1 << R;
    const SV_CONST double* m = M + 8 * l;
    const bool hi = ((threadIdx.x >> POS) & 1u) != 0;
    if constexpr (UNIT) {
        const double m2 = m[2], m4 = m[4];
        const Real orr = (Real)(hi ? m4 : m2);
        Real oi = (Real)0;
        if constexpr (!REALM) {
            const double m3 = m[3], m5 = m[5];
            oi = (Real)(hi ? m5 : m3);
        }
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const Real pr = lane_xor<CTRL>(vr[0][r]), pi = lane_xor<CTRL>(vi[0][r]);
            const Real xr = vr[0][r], xi = vi[0][r];
            if constexpr (REALM) {
                vr[0][r] = fma(orr, pr, xr);
                vi[0][r] = fma(orr, pi, xi);
            } else {
                vr[0][r] = fma(orr, pr, fma(-oi, pi, xr));
                vi[0][r] = fma(orr, pi, fma(oi, pr, xi));
            }
        }
        return;
    }
    const double m0 = m[0], m2 = m[2], m4 = m[4], m6 = m[6];
    const Real sr = (Real)(hi ? m6 : m0), orr = (Real)(hi ? m4 : m2);
    Real si = (Real)0, oi = (Real)0;
    if constexpr (!REALM) {
        const double m1 = m[1], m3 = m[3], m5 = m[5], m7 = m[7];
        si = (Real)(hi ? m7 : m1);
        oi = (Real)(hi ? m5 : m3);
    }
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const Real pr = lane_xor<CTRL>(vr[0][r]), pi = lane_xor<CTRL>(vi[0][r]);
        const Real xr = vr[0][r], xi = vi[0][r];
        if constexpr (REALM) {
            vr[0][r] = fma(sr, xr, orr * pr);
            vi[0][r] = fma(sr, xi, orr * pi);
        } else {
            vr[0][r] = fma(sr, xr, fma(-si, xi, fma(orr, pr, -oi * pi)));
            vi[0][r] = fma(sr, xi, fma(si, xr, fma(orr, pi, oi * pr)));
        }
    }
}

// Tile bit held by thread-index bit j of a layout (the j-th set bit of tmask).
__device__ __forceinline__ int tmask_bit(uint32_t tmask, int j) {
    for (int i = 0; i < j; i++) tmask &= tmask - 1u;
    return __builtin_ctz(tmask);
}

// KC > 0: the pass geometry has exactly KC layouts (compile time, straight-line
// layout walks); KC == 0: generic kernel with a runtime layout count (used for
// states smaller than one tile and for phase angles that need the library's sincos).
template <typename Real, int T, int R, int NV, int NS, int MINB, bool PH, bool INTE, int KC, int NTM = 0,
          bool PERSIST = false, bool SPZ = PH, int GEN = 0, int QFM = 0>
__global__ void __launch_bounds__(1 << (T - R), MINB) k_pass(const PassArgs a) {
    using V2 = typename V2T<Real>::type;
    constexpr int NT = 1 << (T - R);
    constexpr int NR = 1 << R;
    constexpr int NH = NR / 2;  // registers per pivot half
    constexpr int NW = NT / 64;

    // one-vector kernels exchange half a tile at a time (pivot layouts, two
    // workgroups per CU); two-vector kernels run one workgroup per CU (register
    // bound) and exchange whole tiles.
    constexpr bool FULLX = NV == 2;
    __shared__ V2 xbuf[FULLX ? (1 << T) : (1 << (T - 1))];
    __shared__ double s_g[kTF];  // tile fields g_l and E_fixed (entry kTF - 1)
    __shared__ double s_red[NW][NS];
    __shared__ double s_spin[NW][kTF];  // per-wave spin sums (PT_SPINZ)

    const uint32_t t = threadIdx.x;
    CGeoBuf* __restrict__ geo = (CGeoBuf*)a.geo;
    const TileGeom tg{a.c, a.lo, a.g};
    V2* __restrict__ psi = reinterpret_cast<V2*>(a.psi);
    V2* __restrict__ lam = reinterpret_cast<V2*>(a.lam);

    // Persistent launches (fewer workgroups than tiles) walk the tiles with a
    // grid stride; the second half of such a grid may start late, so that the
    // workgroups sharing a CU alternate between streaming and arithmetic
    // instead of loading and computing in lockstep.
    if (PERSIST && a.stagger > 0 && blockIdx.x >= gridDim.x / 2) {
        for (int i = 0; i < a.stagger; i++) __builtin_amdgcn_s_sleep(127);
    }
    uint64_t tile = blockIdx.x;
    if (!PERSIST && a.xcd > 0) {
        // K = 8 * 2^(xcd - 1) interleaved streams: workgroup b walks stream b mod K
        const int kb = 2 + a.xcd;
        if ((a.ntiles & ((1ull << kb) - 1ull)) == 0 && gridDim.x == a.ntiles)
            tile = (uint64_t)(blockIdx.x & ((1u << kb) - 1u)) * (a.ntiles >> kb) + (blockIdx.x >> kb);
    }
    do {
        const uint64_t base = tg.base(tile);

        // ---- load in layout 0 (issued before the per-tile field computation so
        // that the field loop overlaps the memory latency)
        int cur = 0;
        CGeoLayout* L = &geo->L[0];
        uint32_t thr_u = thread_index_bits<T - R>(t, L->tmask);
        uint64_t thr_goff = tg.gmap(thr_u);

        Real vr[NV][NR], vi[NV][NR];
        // Phantom bits exist only for states smaller than one tile (PH); full tiles
        // load without per-register tests.
        if (a.load & 4) {
#pragma unroll
            for (int r = 0; r < NR; r++) {
                bool valid = true;
                if constexpr (PH) valid = ((thr_u | L->reg_u[r]) & a.phantom) == 0u;
                vr[0][r] = valid ? (Real)a.amp0 : (Real)0;
                vi[0][r] = 0;
            }
        } else if (a.load & 1) {
            const V2* __restrict__ src = (a.src ? reinterpret_cast<const V2*>(a.src) : psi) + (base | thr_goff);
            if (NTM & 1) {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    const V2 v = ld_nt(src + L->reg_goff[r]);
                    vr[0][r] = v.x;
                    vi[0][r] = v.y;
                }
            } else {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    V2 v;
                    if constexpr (PH) {
                        v.x = 0;
                        v.y = 0;
                        if (((thr_u | L->reg_u[r]) & a.phantom) == 0u) v = src[L->reg_goff[r]];
                    } else {
                        v = src[L->reg_goff[r]];
                    }
                    vr[0][r] = v.x;
                    vi[0][r] = v.y;
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < NR; r++) {
                vr[0][r] = 0;
                vi[0][r] = 0;
            }
        }
        if constexpr (NV == 2) {
            const V2* __restrict__ src = lam + (base | thr_goff);
#pragma unroll
            for (int r = 0; r < NR; r++) {
                V2 v;
                v.x = 0;
                v.y = 0;
                bool ok = (a.load & 2) != 0;
                if constexpr (PH) ok = ok && ((thr_u | L->reg_u[r]) & a.phantom) == 0u;
                if (ok) v = src[L->reg_goff[r]];
                vr[1][r] = v.x;
                vi[1][r] = v.y;
            }
        }

        if ((t & 63) == 0) {
#pragma unroll
            for (int q = 0; q < NS; q++) s_red[t >> 6][q] = 0.0;
#pragma unroll
            for (int q = 0; q < kTF; q++) s_spin[t >> 6][q] = 0.0;
        }
        double pend[NV];  // uniform scale every register of vector v still has to be multiplied by
#pragma unroll
        for (int v = 0; v < NV; v++) pend[v] = 1.0;

        // ---- fields seen by the tile bits (only passes that evaluate E need them)
        if (a.need_e && t < kTF) s_g[t] = a.tf[tile * kTF + t];
        __syncthreads();  // s_g ready

        // The pass program has a fixed shape: two mixer slots, one point slot, two
        // mixer slots (absent slots have kind 0).  A compile-time shape keeps the
        // amplitude registers in place across ops.
        constexpr int SLOT_KIND[kMaxOps] = {OP_MIX, OP_MIX, OP_POINT, OP_MIX, OP_MIX};
#pragma unroll
        for (int oi = 0; oi < kMaxOps; oi++) {
            const Op op = a.ops[oi];
            if (op.kind == 0) continue;
            if (SLOT_KIND[oi] == OP_MIX) {
                const int K = KC > 0 ? KC : a.nlayouts;
                const bool fwd = (cur == 0);
                double gsum = 0.0;
                auto round = [&](int step) {
                    const int j = fwd ? step : (K - 1 - step);
                    if (step > 0) {
                        // LDS exchange cur -> j: in two halves split by the pivot (register
                        // slot R-1) for one vector, as whole tiles for two vectors
                        CGeoLayout* Lt = &geo->L[j];
                        const uint32_t new_u = thread_index_bits<T - R>(t, Lt->tmask);
                        // byte offsets: one XOR with the table entry per access
                        const uint32_t src = lds_swizzle(thr_u, a.swz) * (uint32_t)sizeof(V2);
                        const uint32_t dst = lds_swizzle(new_u, a.swz) * (uint32_t)sizeof(V2);
                        char* xb = reinterpret_cast<char*>(xbuf);
#pragma unroll
                        for (int v = 0; v < NV; v++) {
                            constexpr int NHALF = FULLX ? 1 : 2;
                            constexpr int NQ = FULLX ? NR : NH;
#pragma unroll
                            for (int h = 0; h < NHALF; h++) {
                                __syncthreads();
#pragma unroll
                                for (int q = 0; q < NQ; q++) {
                                    const int r = h * NQ + q;
                                    V2 x;
                                    x.x = vr[v][r];
                                    x.y = vi[v][r];
                                    *reinterpret_cast<V2*>(xb + (src ^ L->reg_lds[r])) = x;
                                }
                                __syncthreads();
#pragma unroll
                                for (int q = 0; q < NQ; q++) {
                                    const int r = h * NQ + q;
                                    const V2 x = *reinterpret_cast<const V2*>(xb + (dst ^ Lt->reg_lds[r]));
                                    vr[v][r] = x.x;
                                    vi[v][r] = x.y;
                                }
                            }
                        }
                        cur = j;
                        L = Lt;
                        thr_u = new_u;
                        thr_goff = tg.gmap(thr_u);
                    }
                    const int act = fwd ? L->act_fwd : L->act_bwd;
                    if constexpr (GEN != 0) {
                        // general single-qubit layers (one vector, no pending scale)
                        static_assert(NV == 1, "general layers are one-vector passes");
                        const SV_CONST double* __restrict__ M =
                            (const SV_CONST double*)(a.gmat + op.qidx * kGenBlock);
                        // GEN: 1 complex, 2 real, 3 complex unit-diagonal, 4 real unit-diagonal
                        constexpr bool RM = GEN == 2 || GEN == 4;
                        constexpr bool UN = GEN >= 3;
                        gen_round<Real, R, RM, UN>(vr, vi, act, L->rbpack, M);
                        const int dl = L->dpp;
                        if (dl & 8) gen_lane<kLaneX8, 3, Real, R, RM, UN>(vr, vi, tmask_bit(L->tmask, 3), M);
                        if constexpr (sizeof(Real) == 4 && T == 14) {
                            if (dl & 16) gen_lane<kLaneX16, 4, Real, R, RM, UN>(vr, vi, tmask_bit(L->tmask, 4), M);
                        }
                        return;
                    }
                    mix_round<Real, R, NV, (QFM > 0)>(vr, vi, act, op.flags, (Real)op.a, op.b, pend, gsum);
                    // lane-bit butterflies (one-vector kernels): position 3 (DPP);
                    // position 4 (swizzle) for 14-bit complex64 tiles (a second branch
                    // in the complex128 kernel would exhaust its registers)
                    const int dl = L->dpp;
                    if constexpr (NV == 2) {
                        (void)dl;  // two-vector plans butterfly every qubit in registers
                    } else if constexpr (sizeof(Real) == 8) {
                        if (dl != 0)
                            lane_round<kLaneX8, Real, R, NV, (QFM > 0)>(vr, vi, op.flags, (Real)op.a, op.b, pend, gsum);
                    } else if constexpr (T == 14 && MINB <= 2) {
                        if (dl & 8)
                            lane_round<kLaneX8, Real, R, NV, (QFM > 0)>(vr, vi, op.flags, (Real)op.a, op.b, pend, gsum);
                        else if (dl & 16)
                            lane_round<kLaneX16, Real, R, NV, (QFM > 0)>(vr, vi, op.flags, (Real)op.a, op.b, pend, gsum);
                    } else {
                        // 13-bit complex64 tiles, and 14-bit tiles in the four-waves-per-SIMD
                        // kernel (the second branch would not fit its 128 registers), plan lane
                        // position 3 only
                        if (dl != 0)
                            lane_round<kLaneX8, Real, R, NV, (QFM > 0)>(vr, vi, op.flags, (Real)op.a, op.b, pend, gsum);
                    }
                };
                if constexpr (KC > 0) {
#pragma unroll
                    for (int step = 0; step < KC; step++) round(step);
                } else {
                    for (int step = 0; step < K; step++) round(step);
                }
                if (op.flags & MIX_GBETA) wave_add<NS>(s_red, op.slot, gsum);
                if constexpr (GEN >= 3) pend[0] *= op.b;  // unit-diagonal layers: product of the diagonal moduli
            } else {  // OP_POINT
                // Walk the registers in Gray-code order: consecutive registers differ in
                // one bit k, so E changes by +-2 f[k] and the phase by exp(-+2i gamma f[k]).
                double f[R];
                const double e0 = thread_energy<R, T - R>(L, geo, t, s_g, f);
                const int fl = op.flags;
                // E of register r = e0 + (Gray-walk sum of +-2 f[k]) + Q[r]
                if constexpr (QFM >= 2) {
                    // passes of the adjoint sweeps: zeta = psi (1 + i t E) in the first pass, the
                    // form sum E |zeta|^2 at the phase of each layer (nothing else is reduced)
                    // one loop per flag, so that no per-register select keeps the old and the
                    // new amplitudes alive together.  PT_REDUCE (norm, <H_C>, P_gs of the state
                    // the sweep starts from) comes before zeta is formed.
                    if (QFM == 3 && (fl & PT_REDUCE)) {
                        double r_n = 0.0, r_e = 0.0, r_p = 0.0, e_run = e0;
#pragma unroll
                        for (int i = 0; i < NR; i++) {
                            const int r = i ^ (i >> 1);
                            if (i > 0) {
                                const int k = __builtin_ctz(i);
                                e_run += ((r >> k) & 1) ? 2.0 * f[k] : -2.0 * f[k];
                            }
                            const double e = e_run + L->Q[r];
                            const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                            const double p2 = fma(pr, pr, pi * pi);
                            r_n += p2;
                            r_e = fma(e, p2, r_e);
                            if (fabs(e - a.emin) <= a.etol) r_p += p2;
                        }
                        const double s2 = pend[0] * pend[0];
                        wave_add<NS>(s_red, op.slot, r_n * s2);
                        wave_add<NS>(s_red, op.slot + 1, r_e * s2);
                        wave_add<NS>(s_red, op.slot + 2, r_p * s2);
                    }
                    if (fl & PT_ZETA) {
                        const double zt = op.b;
                        double e_run = e0;
#pragma unroll
                        for (int i = 0; i < NR; i++) {
                            const int r = i ^ (i >> 1);
                            if (i > 0) {
                                const int k = __builtin_ctz(i);
                                e_run += ((r >> k) & 1) ? 2.0 * f[k] : -2.0 * f[k];
                            }
                            const double te = zt * (e_run + L->Q[r]);
                            const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                            vr[0][r] = (Real)fma(-te, pi, pr);
                            vi[0][r] = (Real)fma(te, pr, pi);
                        }
                    }
                    if (fl & PT_EFORM) {
                        double r_f = 0.0, e_run = e0;
#pragma unroll
                        for (int i = 0; i < NR; i++) {
                            const int r = i ^ (i >> 1);
                            if (i > 0) {
                                const int k = __builtin_ctz(i);
                                e_run += ((r >> k) & 1) ? 2.0 * f[k] : -2.0 * f[k];
                            }
                            const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                            r_f = fma(e_run + L->Q[r], fma(pr, pr, pi * pi), r_f);
                        }
                        wave_add<NS>(s_red, op.slot2, r_f * pend[0] * pend[0]);
                    }
                }
                constexpr int kRedFlags = QFM > 0 ? 0 : (PT_REDUCE | PT_LAM_INIT | PT_GGAMMA | PT_SPINZ | PT_E2);
                if (fl & kRedFlags) {
                    // one sweep over the registers feeds every reduction of the op
                    // (|psi|^2 is formed once; the spin sums of one-vector passes
                    // take it for each register bit k: +-|psi|^2 by bit k of r)
                    double r_n = 0.0, r_e = 0.0, r_p = 0.0, r_g = 0.0, r_e2 = 0.0;
                    double Sk[R];
#pragma unroll
                    for (int k = 0; k < R; k++) Sk[k] = 0.0;
                    // spin sums exist in the generic kernels and in dedicated fast variants
                    const bool spins = SPZ && NV == 1 && (fl & PT_SPINZ) != 0;
                    double e_run = e0;
#pragma unroll
                    for (int i = 0; i < NR; i++) {
                        const int r = i ^ (i >> 1);
                        if (i > 0) {
                            const int k = __builtin_ctz(i);
                            e_run += ((r >> k) & 1) ? 2.0 * f[k] : -2.0 * f[k];
                        }
                        const double e = e_run + L->Q[r];
                        const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                        if (fl & (PT_REDUCE | PT_SPINZ | PT_E2)) {
                            const double p2 = pr * pr + pi * pi;
                            r_n += p2;
                            r_e += e * p2;
                            if (fl & PT_E2) r_e2 += e * e * p2;
                            if (fabs(e - a.emin) <= a.etol) r_p += p2;
                            if (spins) {
#pragma unroll
                                for (int k = 0; k < R; k++) Sk[k] += ((r >> k) & 1) ? p2 : -p2;
                            }
                        }
                        if constexpr (NV == 2) {
                            if (fl & PT_LAM_INIT) {
                                vr[1][r] = (Real)(e * pr);
                                vi[1][r] = (Real)(e * pi);
                            }
                            if (fl & PT_GGAMMA) {
                                const Real q = vr[1][r] * vi[0][r] - vi[1][r] * vr[0][r];
                                r_g += e * (double)q;
                            }
                        }
                    }
                    const double s2 = pend[0] * pend[0];
                    if (fl & PT_REDUCE) {
                        wave_add<NS>(s_red, op.slot, r_n * s2);
                        wave_add<NS>(s_red, op.slot + 1, r_e * s2);
                        wave_add<NS>(s_red, op.slot + 2, r_p * s2);
                    }
                    if (fl & PT_E2) wave_add<NS>(s_red, op.slot3, r_e2 * s2);
                    if constexpr (NV == 1 && SPZ) {
                        if (spins) {
                            // tile bit l: register bit k -> Sk[k]; lane bit j -> +-norm per lane; wave
                            // bit -> +-the wave's norm
                            const uint32_t rbp = L->rbpack;
#pragma unroll
                            for (int k = 0; k < R; k++) wave_add<kTF>(s_spin, (rbp >> (4 * k)) & 15u, Sk[k] * s2);
                            const double nrm = r_n * s2, wn = wave_sum(nrm);
                            uint32_t m = L->tmask;
#pragma unroll
                            for (int j = 0; j < T - R; j++) {
                                const int l = __builtin_ctz(m);
                                m &= m - 1u;
                                if (j < 6) {
                                    wave_add<kTF>(s_spin, l, ((t >> j) & 1u) ? nrm : -nrm);
                                } else if ((t & 63) == 0) {
                                    s_spin[t >> 6][l] += ((t >> j) & 1u) ? wn : -wn;
                                }
                            }
                            if ((t & 63) == 0) s_spin[t >> 6][kTF - 1] += wn;
                        }
                    }
                    if constexpr (NV == 2) {
                        if (fl & PT_LAM_INIT) pend[1] = pend[0];
                        if (fl & PT_GGAMMA) wave_add<NS>(s_red, op.slot2, r_g * pend[0] * pend[1]);
                    }
                }
                if (fl & (PT_PHASE_PSI | PT_PHASE_LAM)) {
                    const double gam = op.a;
                    const SV_CONST double* __restrict__ qph = (const SV_CONST double*)(a.ptab + a.qph_off[op.qidx]);
                    double2 gk[R];
                    double2 run;
                    // PT_DIAG: the phase also applies a diagonal of single-qubit factors,
                    // exp(-i sum_q th_q s_q) (two local-field sums more, in one pass of a program)
                    double th0 = 0.0, thk[R];
#pragma unroll
                    for (int k = 0; k < R; k++) thk[k] = 0.0;
                    if constexpr (GEN == 3) {
                        if (fl & PT_DIAG) {
                            const double* __restrict__ D = a.gmat + (size_t)op.b * kGenBlock;
                            const int q = (int)(t & 63u);
                            double x = 0.0;
                            if (q < a.n) x = ((base >> q) & 1ull) ? D[16 + q] : -D[16 + q];
                            th0 = wave_sum(x) + D[kGenBlock - 1];
                            uint32_t m = L->tmask;
#pragma unroll
                            for (int j = 0; j < T - R; j++) {
                                const double th = D[__builtin_ctz(m)];
                                m &= m - 1u;
                                th0 += ((t >> j) & 1u) ? th : -th;
                            }
#pragma unroll
                            for (int k = 0; k < R; k++) {
                                thk[k] = D[(L->rbpack >> (4 * k)) & 15u];
                                th0 -= thk[k];
                                thk[k] *= 2.0;
                            }
                        }
                    }
                    // (real general layers: the host sends other energies to the complex kernels; with the
                    // code for them the pass of four Hadamard layers, n = 23 complex64, took 103 us, without 98)
                    if (INTE && (GEN == 2 || GEN == 4 || a.lut_half >= 0)) {
                        // energies on the grid Z / q: factors from the table exp(-i gamma m / q)
                        const SV_CONST double* __restrict__ lut =
                            (const SV_CONST double*)(a.ptab + a.lut_off[op.qidx] + a.lut_half);
                        const int Lh = a.lut_half;
#pragma unroll
                        for (int k = 0; k < R; k++) {
                            const int m = min(max((int)(2.0 * f[k] * a.lut_q), -Lh), Lh);
                            gk[k] = ctab(lut, m);
                        }
                        run = ctab(lut, min(max((int)(e0 * a.lut_q), -Lh), Lh));
                    } else {
                        // One evaluation at a time: the fma(0, previous sine, x) link (exact
                        // for finite values) keeps the scheduler from interleaving the R + 1 of
                        // them, which would exhaust the register file.  INTE kernels take other
                        // energies too, up to kTileMaxAngle (270 instructions per thread and phase,
                        // within the registers of two workgroups per CU: n = 23 complex128, p = 8 920 ->
                        // 600 us, the rate of integer couplings); the others call the library.
                        double link = 0.0;
#pragma unroll
                        for (int k = 0; k < R; k++) {
                            const double x = GEN == 3 ? fma(0.0, link, fma(2.0 * gam, f[k], thk[k]))
                                                      : fma(0.0, link, 2.0 * gam * f[k]);
                            if constexpr (INTE) {
                                gk[k] = cis_neg(x);
                                link = gk[k].y;
                            } else {
                                double sn, cs;
                                sincos(x, &sn, &cs);
                                gk[k] = make_double2(cs, -sn);
                                link = sn;
                            }
                        }
                        const double x = GEN == 3 ? fma(0.0, link, fma(gam, e0, th0)) : fma(0.0, link, gam * e0);
                        if constexpr (INTE) {
                            run = cis_neg(x);
                        } else {
                            double sn, cs;
                            sincos(x, &sn, &cs);
                            run = make_double2(cs, -sn);
                        }
                    }
                    // the phase has modulus one: the pending scales stay pending (they are
                    // applied at the store)
#pragma unroll
                    for (int i = 0; i < NR; i++) {
                        const int r = i ^ (i >> 1);
                        if (i > 0) {
                            const int k = __builtin_ctz(i);
                            const double2 g = ((r >> k) & 1) ? gk[k] : make_double2(gk[k].x, -gk[k].y);
                            run = cmul(run, g);
                        }
                        const double2 ph = cmul(run, ctab(qph, r));
#pragma unroll
                        for (int v = 0; v < NV; v++) {
                            if constexpr (sizeof(Real) == 8) {
                                const double xr = vr[v][r], xi = vi[v][r];
                                vr[v][r] = xr * ph.x - xi * ph.y;
                                vi[v][r] = xr * ph.y + xi * ph.x;
                            } else {
                                const float cr = (float)ph.x, ci = (float)ph.y;
                                const float xr = vr[v][r], xi = vi[v][r];
                                vr[v][r] = xr * cr - xi * ci;
                                vi[v][r] = xr * ci + xi * cr;
                            }
                        }
                    }
                }
            }
        }

        // ---- store in the current layout (applying what is left of the pending scales)
#pragma unroll
        for (int v = 0; v < NV; v++) {
            if (!(a.store & (1 << v))) continue;
            V2* __restrict__ dst = (v == 0 ? psi : lam) + (base | thr_goff);
            const Real sc = (Real)pend[v];
            const bool unit = pend[v] == 1.0;
            if (NTM & 2) {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    V2 x;
                    x.x = unit ? vr[v][r] : vr[v][r] * sc;
                    x.y = unit ? vi[v][r] : vi[v][r] * sc;
                    st_nt(dst + L->reg_goff[r], x);
                }
            } else {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    if constexpr (PH) {
                        if (((thr_u | L->reg_u[r]) & a.phantom) != 0u) continue;
                    }
                    V2 x;
                    x.x = unit ? vr[v][r] : vr[v][r] * sc;
                    x.y = unit ? vi[v][r] : vi[v][r] * sc;
                    dst[L->reg_goff[r]] = x;
                }
            }
        }

        // ---- per-tile partial sums, fixed order
        if (a.nslots > 0 || (SPZ && a.spin_part)) {
            __syncthreads();
            if ((int)t < a.nslots) {
                double v = 0.0;
                for (int ww = 0; ww < NW; ww++) v += s_red[ww][t];
                a.partials[(uint64_t)t * a.ntiles + tile] = v;
            }
            if (SPZ && a.spin_part && t < kTF) {
                double v = 0.0;
                for (int ww = 0; ww < NW; ww++) v += s_spin[ww][t];
                a.spin_part[(uint64_t)t * a.ntiles + tile] = v;
            }
        }
        if constexpr (!PERSIST) break;
        tile += gridDim.x;
        if (tile < a.ntiles) __syncthreads();  // LDS reuse by the next tile
    } while (tile < a.ntiles);
}

// Full-tile general-layer passes: layout count, real or complex matrices, nontemporal hints.
template <typename Real, int T, int R, int NS, int GMB, int NTM, int GC = 1, int GR = 2>
static void launch_gen_fast(const PassArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    if constexpr (GC == 1) {
        if (a.gen_unit) {  // unit-diagonal layers: the GEN = 3 / 4 kernels
            launch_gen_fast<Real, T, R, NS, GMB, NTM, 3, 4>(a, grid, block, st);
            return;
        }
    }
    const bool rm = a.gen_real != 0;
    // three or more layouts with complex matrices on complex128 amplitudes need the whole
    // register file (one workgroup per CU)
    constexpr int MB = (sizeof(Real) == 8 && GC == 1) ? 1 : GMB;
    // complex64 unit layers with two layouts: held to the 128 registers of two workgroups per CU, which
    // they exceed by two (spilled) since their phase may apply single-qubit diagonals (PT_DIAG); ten
    // Eq. AQA4 steps, n = 27: 14.1 -> 11.6 ms
    constexpr int MB2 = (sizeof(Real) == 4 && GC == 3) ? 4 : GMB;
    if (a.nlayouts == 1) {
        if (rm) hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, GMB, false, true, 1, NTM, false, false, GR>), grid, block,
                                   0, st, a);
        else hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, GMB, false, true, 1, NTM, false, false, GC>), grid, block, 0,
                                st, a);
    } else if (a.nlayouts == 2) {
        if (rm) hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, GMB, false, true, 2, NTM, false, false, GR>), grid, block,
                                   0, st, a);
        else hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MB2, false, true, 2, NTM, false, false, GC>), grid, block, 0,
                                st, a);
    } else if (a.kc34 && a.nlayouts == 3) {  // straight-line walk
        if (rm) hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, GMB, false, true, 3, NTM, false, false, GR>), grid, block,
                                   0, st, a);
        else hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MB, false, true, 3, NTM, false, false, GC>), grid, block, 0,
                                st, a);
    } else {
        if (rm) hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, GMB, false, true, 0, NTM, false, false, GR>), grid, block,
                                   0, st, a);
        else hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MB, false, true, 0, NTM, false, false, GC>), grid, block, 0,
                                st, a);
    }
}

// Passes of the two one-vector adjoint sweeps: QFM = 1 mixer-only passes (quadratic forms),
// QFM = 2 passes that also form zeta or the E form at their POINT, QFM = 3 the first pass of
// the zeta_+ sweep, which also reduces norm, <H_C> and P_gs (each part that is not needed
// is left out: kernels with all of them spill).
template <typename Real, int T, int R, int NS, int MINB, int QFM>
static int launch_qf(const PassArgs& a, bool fast, dim3 grid, dim3 block, hipStream_t st) {
    constexpr int PMB = MINB > 2 ? 2 : MINB;
    if (!fast && !a.libm) {  // states smaller than one tile
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, PMB, true, true, 0, 0, false, false, 0, QFM>), grid, block, 0, st,
                           a);
    } else if (!fast) {  // phase angles beyond kTileMaxAngle off the energy grid: library sincos
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, 1, true, false, 0, 0, false, false, 0, QFM>), grid, block, 0, st,
                           a);
    } else if (a.nlayouts == 1) {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 1, 0, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else if (a.nlayouts == 2 && a.nt == 3) {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 2, 3, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else if (a.nlayouts == 2) {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 2, 0, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else if (sizeof(Real) == 4 && a.nlayouts == 3 && a.nt == 3) {
        // complex64: straight-line walk (the layout loop spills more there)
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 3, 3, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else if (sizeof(Real) == 4 && a.nlayouts == 3) {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 3, 0, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else if (a.nt == 3) {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 0, 3, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    } else {
        hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, MINB, false, true, 0, 0, false, false, 0, QFM>), grid, block, 0,
                           st, a);
    }
    return (int)hipGetLastError();
}

// Slot counts: one-vector passes carry up to 8 reduction slots (fused AQA
// steps); two-vector passes need at most 4 (3 for the turnaround reductions
// + 1 gradient slot, or 3 gradient slots).
template <typename Real, int T, int R, int NV, int NS, int MINB>
static int run_pass(const PassArgs& a, void* stream) {
    // persistent grids exist for the one-vector fast paths with >= 2 layouts
    const bool pers = NV == 1 && a.grid > 0 && (uint64_t)a.grid < a.ntiles && a.nlayouts >= 2 && a.phantom == 0 &&
                      !a.libm;
    const unsigned nwg = pers ? (unsigned)a.grid : (unsigned)a.ntiles;
    const dim3 grid(nwg), block(1 << (T - R));
    hipStream_t st = (hipStream_t)stream;
    const bool fast = a.phantom == 0 && !a.libm;
    // general-layer kernels exist for 13-bit complex128 and 14-bit complex64 tiles
    if constexpr (NV == 1 && ((sizeof(Real) == 8 && T == 13) || (sizeof(Real) == 4 && T == 14))) {
        if (a.gmat) {  // general single-qubit layers (real matrices: half the arithmetic)
            // general kernels need more registers than the four-waves-per-SIMD budget
            constexpr int GMB = MINB > 2 ? 2 : MINB;
            if (fast && !a.spin_part) {
                if (a.nt == 3)
                    launch_gen_fast<Real, T, R, NS, GMB, 3>(a, grid, block, st);
                else
                    launch_gen_fast<Real, T, R, NS, GMB, 0>(a, grid, block, st);
            } else if (a.gen_unit) {
                hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, 1, true, false, 0, 0, false, true, 3>), grid, block,
                                   0, st, a);
            } else {
                hipLaunchKernelGGL((k_pass<Real, T, R, 1, NS, 1, true, false, 0, 0, false, true, 1>), grid, block,
                                   0, st, a);
            }
            return (int)hipGetLastError();
        }
    }
    if (a.gmat) return (int)hipErrorInvalidValue;
    // passes of the two one-vector adjoint sweeps (quadratic forms, zeta, E forms) exist for
    // the default one-vector tiles: 13-bit complex128 and 14-bit complex64 with four waves per SIMD
    constexpr bool kQF = NV == 1 && ((sizeof(Real) == 8 && T == 13) || (sizeof(Real) == 4 && T == 14 && MINB == 4));
    if (a.qf && !kQF) return (int)hipErrorInvalidValue;
    if constexpr (kQF) {
        if (a.qf == 1) return launch_qf<Real, T, R, NS, MINB, 1>(a, fast, grid, block, st);
        if (a.qf == 2) return launch_qf<Real, T, R, NS, MINB, 2>(a, fast, grid, block, st);
        if (a.qf == 3) return launch_qf<Real, T, R, NS, MINB, 3>(a, fast, grid, block, st);
    }
    if (fast) {
        // one or two layouts: straight-line walks; three or more: a loop keeps
        // the register pressure below the two-workgroups-per-CU limit
        // (nontemporal variants for passes over long contiguous runs)
        if constexpr (NV == 1) {
            if (a.spin_part) {
                // passes that also sum the spin expectations: straight-line walks fit the plain
                // kernels' register budget (the layout loop spills 200-280 B per thread in it; with
                // half the workgroups per CU instead, the n = 23 complex64 passes took 61-73 us, now 37-41)
                constexpr int SMB = MINB > 2 ? 2 : MINB;
                const bool nts = a.nt == 3;
                if (a.nlayouts == 1)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 1, 0, false, true>), grid, block,
                                       0, st, a);
                else if (a.nlayouts == 2 && nts)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 2, 3, false, true>), grid, block,
                                       0, st, a);
                else if (a.nlayouts == 2)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 2, 0, false, true>), grid, block,
                                       0, st, a);
                else if (a.nlayouts == 3 && nts)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 3, 3, false, true>), grid, block,
                                       0, st, a);
                else if (a.nlayouts == 3)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 3, 0, false, true>), grid, block,
                                       0, st, a);
                else
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, SMB, false, true, 0, 0, false, true>), grid, block,
                                       0, st, a);
                return (int)hipGetLastError();
            }
            if (pers) {
                if (a.nlayouts == 2)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 2, 0, true>), grid, block, 0, st,
                                       a);
                else if (a.nt == 3)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 0, 3, true>), grid, block, 0, st,
                                       a);
                else
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 0, 0, true>), grid, block, 0, st,
                                       a);
                return (int)hipGetLastError();
            }
        }
        if constexpr (NV == 2) {
            // two-vector passes (one workgroup per CU, the whole register file): three and
            // four layouts as straight-line walks
            if (a.kc34 && a.nlayouts == 3) {
                if (a.nt == 3)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 3, 3>), grid, block, 0, st, a);
                else
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 3>), grid, block, 0, st, a);
                return (int)hipGetLastError();
            }
            if (a.kc34 && a.nlayouts == 4) {
                if (a.nt == 3)
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 4, 3>), grid, block, 0, st, a);
                else
                    hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 4>), grid, block, 0, st, a);
                return (int)hipGetLastError();
            }
        }
        if (a.nlayouts == 1)
            hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 1>), grid, block, 0, st, a);
        else if (a.nlayouts == 2 && a.nt == 3)
            hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 2, 3>), grid, block, 0, st, a);
        else if (a.nlayouts == 2)
            hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 2>), grid, block, 0, st, a);
        else if (a.nt == 3)
            hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 0, 3>), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, MINB, false, true, 0>), grid, block, 0, st, a);
    } else if (!a.libm) {
        // states smaller than one tile (phantom bits): correctness over occupancy
        constexpr int PMB = MINB > 2 ? 2 : MINB;
        hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, PMB, true, true, 0>), grid, block, 0, st, a);
    } else {
        // large phase angles off the energy grid: the library's sincos needs more registers;
        // one workgroup per CU leaves it the whole file
        hipLaunchKernelGGL((k_pass<Real, T, R, NV, NS, 1, true, false, 0>), grid, block, 0, st, a);
    }
    return (int)hipGetLastError();
}

}  // namespace svk
