// gfx950 kernels for states that do not fill the chip with the large tiles of
// sv_kernels.hip: compact tile programs on 2^10 .. 2^13 amplitudes per
// workgroup, the per-instance energy table they read, and the second stage of
// their reductions.
//
// What bounds such a pass is latency, not bandwidth (the state sits in L2 or
// the last-level cache): kernel start, table reads, the serial chain of
// butterflies and exchanges of one workgroup, and instruction fetch, since
// every workgroup runs its code once.  So the tiles are small enough to reach
// every CU, all the layout arithmetic is done in registers instead of read
// from tables, the energy comes from a table of E(z) (R + 1 reads per thread),
// phase factors are computed in place instead of by a launch of their own, and
// the code is a loop over ops and layouts (one copy of each op's code).
// Measured against the large tiles: n = 12 complex64, p = 4 (one launch) 93 ->
// 19 us per evaluation, n = 20 complex64, p = 8 255 -> 114 us, n = 21 real
// couplings, p = 3 164 -> 86 us, n = 17 gradient, p = 4 436 -> 138 us.  Cycle
// stamps of one workgroup (n = 12, double precision in registers): a mixer round
// 900, a swap of two lane bits 500, an exchange 1500, a phase from the table
// 2300 (in place 2700), a reduction 2300; start and loads 2100.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sv_device.h"
#include "sv_internal.h"

namespace svk {

// E(z) of every basis state (Eq. HC), one thread per state: a compensated sum,
// so that the table holds E(z) rounded once whatever the number of terms.
__global__ void __launch_bounds__(256) k_energy_table(const IsingDev is, double* __restrict__ E, uint64_t N) {
    const uint64_t z = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0, e = 0.0;
    auto add = [&](double x) {
        const double t = s + x, b = t - s;
        e += (s - (t - b)) + (x - b);
        s = t;
    };
    for (int i = 0; i < is.n; i++) add(((z >> i) & 1) ? is.h[i] : -is.h[i]);
    for (int k = 0; k < is.m; k++) {
        const uint64_t same = ~((z >> is.ei[k]) ^ (z >> is.ej[k])) & 1ull;
        add(same ? is.J[k] : -is.J[k]);
    }
    if (z < N) E[z] = s + e;
}

int launch_energy_table(const IsingDev& is, double* E, void* stream) {
    const uint64_t N = 1ull << is.n;
    hipLaunchKernelGGL(k_energy_table, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, (hipStream_t)stream, is, E, N);
    return (int)hipGetLastError();
}

// Products with the fused operations spelt out, so that every variant of the
// kernel rounds alike.
template <typename X>
__device__ __forceinline__ X mul_re(X ar, X ai, X br, X bi) {
    return fma(ar, br, -(ai * bi));
}
template <typename X>
__device__ __forceinline__ X mul_im(X ar, X ai, X br, X bi) {
    return fma(ar, bi, ai * br);
}

// Workgroup sums of N per-thread values in a fixed order, handed to
// put(i, sum) by thread i (any thread for one wave).
template <int N, int NW, typename Put>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*s_red)[kTF], Put put) {
    static_assert(N <= kTF, "reduction row");
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < N; i++) v[i] = wave_sum(v[i]);
    if constexpr (NW == 1) {
        if (t == 0)
#pragma unroll
            for (int i = 0; i < N; i++) put(i, v[i]);
    } else {
        if ((t & 63) == 0)
#pragma unroll
            for (int i = 0; i < N; i++) s_red[t >> 6][i] = v[i];
        __syncthreads();
        if (t < N) {
            double x = 0.0;
            for (int w = 0; w < NW; w++) x += s_red[w][t];
            put(t, x);
        }
        __syncthreads();
    }
}

// LDS slot of a tile-local index (T <= 16): the higher nibbles folded into the lowest one, and the
// slot bits of one index bit (both linear over XOR).
__device__ __forceinline__ uint32_t tile_slot(uint32_t u) { return u ^ (((u >> 4) ^ (u >> 8) ^ (u >> 12)) & 15u); }
__device__ __forceinline__ uint32_t tile_slot_bit(int p) { return (1u << p) | (p >= 4 ? 1u << (p & 3) : 0u); }

// Exchanges lane bit B (4 or 5) of a wave with the choice of register: the lanes of a with the bit
// set take those of b with it clear, and the other way round.
template <int B>
__device__ __forceinline__ void lane_swap(uint32_t& a, uint32_t& b) {
    const auto x = B == 4 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                          : __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = x[0];
    b = x[1];
}
template <int B>
__device__ __forceinline__ void lane_swap(float& a, float& b) {
    uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    lane_swap<B>(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int B>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
    lane_swap<B>(xl, yl);
    lane_swap<B>(xh, yh);
    a = __longlong_as_double((long long)((uint64_t)xh << 32 | xl));
    b = __longlong_as_double((long long)((uint64_t)yh << 32 | yl));
}

// One tile program.  Real: stored amplitudes; Acc: amplitudes in registers and
// LDS; 2^T amplitudes per workgroup, 2^R per thread and vector, NV vectors.
// Layout j holds tile bits [b, b + 4) in registers, q and q + 1 in lane bits 4
// and 5, and the others in the rest of the thread index, in order.  A layout
// with butterflies on q and q + 1 swaps them with register slots 2 and 3 by
// permlane swaps (an eighth of an exchange through LDS), so that the next
// exchange leaves from, or arrives in, the swapped form; points, loads and
// stores see the plain one.  FEAT: 0 uniform mixers, phases and the energy
// reduction; 1 also the forms of the adjoint sweeps; 2 also general layers and
// spin sums (each left out where it is not needed: registers and code size);
// 3 as 0, with the library's sine and cosine for phase angles beyond
// kTileMaxAngle; 4 real general layers and nothing else (twelve Hadamard layers
// in complex128: n = 13 162 -> 122 us, n = 18 222 -> 186 us, n = 21 312 -> 248 us
// against the complex form; 127, 191 and 274 us on the large tiles.  Within
// variant 2 they gave 129, 198 and 275 us, and its double-precision kernels
// spilled more: complex layers at n = 21 2 % slower).
// OCC: waves per SIMD the registers are allotted for.
template <typename Real, typename Acc, int T, int R, int NV, int FEAT, int OCC>
__global__ void __launch_bounds__(1 << (T - R), OCC) k_tile(const TileArgs a) {
    using V2 = typename V2T<Real>::type;
    using A2 = typename V2T<Acc>::type;
    constexpr int NT = 1 << (T - R);
    constexpr int NR = 1 << R;
    constexpr int NW = NT / 64;
    static_assert(NT >= 64 && R == 4, "whole waves, 16 amplitudes per thread");
    __shared__ A2 xbuf[1 << T];
    __shared__ double s_red[NW][kTF];
    __shared__ A2 s_lut[kTileLut];  // phase factors of a grid-valued instance

    // every scalar of the header at once (the compiler would fetch them block by block, a memory
    // round trip each)
    asm volatile("" ::"s"(a.psi), "s"(a.lam), "s"(a.src), "s"(a.E), "s"(a.part), "s"(a.c), "s"(a.lo), "s"(a.g));
    asm volatile("" ::"s"(a.phantom), "s"(a.nlayouts), "s"(a.lbpack), "s"(a.act), "s"(a.load),
                 "s"(a.store), "s"(a.need_e), "s"(a.nops), "s"(a.dual), "s"(a.lut_n), "s"(a.lut_step), "s"(a.amp0));
    const uint32_t t = threadIdx.x;
    auto cis = [](double x) {
        if constexpr (FEAT == 3) {
            double sn, cs;
            sincos(x, &sn, &cs);
            return make_double2(cs, -sn);
        } else {
            return cis_neg(x);
        }
    };
    // the op list is read where it lies (a dynamic index into a by-value
    // argument would copy it to scratch memory)
    const SV_CONST TileArgs* ka = (const SV_CONST TileArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    struct {
        uint32_t w0, parts;
        int aux;
        double a, b;
    } op0 = {ka->ops[0].w0, ka->ops[0].parts, ka->ops[0].aux, ka->ops[0].a, ka->ops[0].b};
    asm volatile("" ::"s"(op0.w0), "s"(op0.parts), "s"(op0.aux), "s"(op0.a), "s"(op0.b));
    const uint64_t tile = a.dual ? 0 : blockIdx.x;
    const bool second = a.dual && blockIdx.x != 0;
    const TileGeom tg{a.c, a.lo, a.g};
    const uint64_t base = tg.base(tile);
    const int K = a.nlayouts;
    const uint32_t ph = a.phantom;
    double* const part = a.part + (second ? (uint64_t)a.dual_cols * a.ntiles : 0ull);

    auto lbase = [&](int j) { return (int)((a.lbpack >> (8 * j)) & 15u); };
    auto lpair = [&](int j) { return (int)((a.lbpack >> (8 * j + 4)) & 15u); };
    // tile bits of the thread index but lane bits 4 and 5, and of all of it
    auto trest = [&](int b, int q) {
        const uint32_t y = (t & 15u) | ((t >> 6) << 4);
        const int g1 = min(b, q), g2 = max(b, q), w1 = b < q ? R : 2, w2 = b < q ? 2 : R;
        const uint32_t z = (y & ((1u << g1) - 1u)) | ((y >> g1) << (g1 + w1));
        return (z & ((1u << g2) - 1u)) | ((z >> g2) << (g2 + w2));
    };
    const uint32_t tl = (t >> 4) & 3u;
    auto tpart = [&](int j) { return trest(lbase(j), lpair(j)) | tl << lpair(j); };
    auto swaps = [&](int j) { return ((a.act >> (8 * j)) & 0x30u) != 0u; };
    int cur = 0;
    int ab = lbase(0);
    uint32_t thr = tpart(0);

    // Byte offsets of 32 bits (the states here hold less than 2^28 bytes); register r = i ^ (i >> 1)
    // is reached by one XOR from register (i - 1) ^ ((i - 1) >> 1).
    constexpr uint32_t ES = (uint32_t)sizeof(V2);
    auto goff = [&](uint32_t u) { return (uint32_t)tg.gmap(u & ~ph); };
    const uint32_t base32 = (uint32_t)base;

    // ---- load in layout 0
    Acc vr[NV][NR], vi[NV][NR];
    {
        uint32_t gb[R];
#pragma unroll
        for (int k = 0; k < R; k++) gb[k] = goff(1u << (ab + k)) * ES;
#pragma unroll
        for (int v = 0; v < NV; v++) {
            const char* __restrict__ src =
                reinterpret_cast<const char*>(v == 1 ? (const void*)a.lam : (a.src ? a.src : (const void*)a.psi));
            if ((a.load >> v) & 1) {
                uint32_t off = (base32 | goff(thr)) * ES;
#pragma unroll
                for (int i = 0; i < NR; i++) {
                    if (i > 0) off ^= gb[__builtin_ctz(i)];
                    const int r = i ^ (i >> 1);
                    const V2 x = *reinterpret_cast<const V2*>(src + off);
                    vr[v][r] = x.x;
                    vi[v][r] = x.y;
                }
            } else {
                const Acc x0 = (v == 0 && (a.load & 4)) ? (Acc)a.amp0 : (Acc)0;
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    vr[v][r] = x0;
                    vi[v][r] = 0;
                }
            }
            if (ph != 0u) {  // states smaller than the tile
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    const bool valid = ((thr | ((uint32_t)r << ab)) & ph) == 0u;
                    vr[v][r] = valid ? vr[v][r] : (Acc)0;
                    vi[v][r] = valid ? vi[v][r] : (Acc)0;
                }
            }
        }
    }
    // energies of the thread's register 0 and of the registers one bit away from
    // it, for the layouts that hold a point op: E(r) = E(0) + sum_k r_k d_k + Q(r);
    // lane r also takes Q(r)
    double ev[2][R + 1], ql[2];
#pragma unroll
    for (int s = 0; s < 2; s++) {
#pragma unroll
        for (int k = 0; k <= R; k++) ev[s][k] = 0.0;
        ql[s] = 0.0;
        if ((a.need_e >> s) & 1) {
            const int b = lbase(s ? K - 1 : 0);
            const uint32_t u = tpart(s ? K - 1 : 0);
            const char* __restrict__ E = reinterpret_cast<const char*>(a.E);
            const uint32_t o = (base32 | goff(u)) * 8u;
            ev[s][0] = *reinterpret_cast<const double*>(E + o);
#pragma unroll
            for (int k = 0; k < R; k++)
                ev[s][1 + k] = *reinterpret_cast<const double*>(E + (o ^ (goff(1u << (b + k)) * 8u)));
            ql[s] = ka->Q[s][t & (NR - 1)];
        }
    }

    double pend[NV];  // uniform scale every register of vector v still has to be multiplied by
#pragma unroll
    for (int v = 0; v < NV; v++) pend[v] = 1.0;

    // register slots 2 and 3 <-> lane bits 4 and 5
    auto swap45 = [&]() {
#pragma unroll
        for (int v = 0; v < NV; v++)
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (!(r & 4)) {
                    lane_swap<4>(vr[v][r], vr[v][r | 4]);
                    lane_swap<4>(vi[v][r], vi[v][r | 4]);
                }
            }
#pragma unroll
        for (int v = 0; v < NV; v++)
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (!(r & 8)) {
                    lane_swap<5>(vr[v][r], vr[v][r | 8]);
                    lane_swap<5>(vi[v][r], vi[v][r | 8]);
                }
            }
    };
    // LDS exchange into layout j, between the swapped forms of layouts that swap.  A thread writes
    // only the slots it read last, so one barrier (between writes and reads) is enough.
    auto exchange = [&](int j) {
        const bool ws = swaps(cur), wd = swaps(j);
        const int nb = lbase(j), sq = lpair(cur), dq = lpair(j);
        constexpr uint32_t SZ = (uint32_t)sizeof(A2);
        uint32_t bs[R], bd[R];
#pragma unroll
        for (int k = 0; k < R; k++) {
            bs[k] = tile_slot_bit(k >= 2 && ws ? sq + k - 2 : ab + k) * SZ;
            bd[k] = tile_slot_bit(k >= 2 && wd ? dq + k - 2 : nb + k) * SZ;
        }
        const uint32_t nrest = trest(nb, dq);
        const uint32_t s0 = tile_slot((thr & ~(3u << sq)) | tl << (ws ? ab + 2 : sq)) * SZ;
        const uint32_t d0 = tile_slot(nrest | tl << (wd ? nb + 2 : dq)) * SZ;
        char* xb = reinterpret_cast<char*>(xbuf);
#pragma unroll
        for (int v = 0; v < NV; v++) {
            if (v > 0) __syncthreads();  // the first vector's reads
            uint32_t ad = s0;
#pragma unroll
            for (int i = 0; i < NR; i++) {
                if (i > 0) ad ^= bs[__builtin_ctz(i)];
                const int r = i ^ (i >> 1);
                A2 x;
                x.x = vr[v][r];
                x.y = vi[v][r];
                *reinterpret_cast<A2*>(xb + ad) = x;
            }
            __syncthreads();
            ad = d0;
#pragma unroll
            for (int i = 0; i < NR; i++) {
                if (i > 0) ad ^= bd[__builtin_ctz(i)];
                const int r = i ^ (i >> 1);
                const A2 x = *reinterpret_cast<const A2*>(xb + ad);
                vr[v][r] = x.x;
                vi[v][r] = x.y;
            }
        }
        cur = j;
        ab = nb;
        thr = nrest | tl << dq;
    };

    // the next op is fetched while one runs
    uint32_t nw0 = op0.w0;
    uint32_t nparts = op0.parts;
    int naux = op0.aux;
    double na = op0.a, nb_ = op0.b;
#pragma unroll 1
    for (int oi = 0; oi < a.nops; oi++) {
        const uint32_t w0 = nw0;
        const int kind = (int)(w0 & 255u), fl = (int)(w0 >> 8);
        const double opa = na, opb = nb_;
        const int part0 = (int)(int16_t)(nparts & 0xffffu), part2 = (int)nparts >> 16, aux = naux;
        {
            const SV_CONST TileOp* nx = &ka->ops[oi + 1 < a.nops ? oi + 1 : oi];
            nw0 = nx->w0;
            nparts = nx->parts;
            naux = nx->aux;
            na = nx->a;
            nb_ = nx->b;
        }
        auto put_at = [&](int col) {
            return [&, col](int i, double x) { part[(uint64_t)(col + i) * a.ntiles + tile] = x; };
        };
        if (kind == OP_MIX) {
            const bool fwd = cur == 0;
            double gsum = 0.0;
            const Acc tq = (Acc)opa;
            // butterflies of register slots K0 .. 3; slot 0 or 2 holds tile bit p0 or p2
            auto round = [&](auto k0, uint32_t act, int p0, int p2) {
                constexpr int K0 = decltype(k0)::value;
                if (FEAT == 4) {
                    // real matrices: half the arithmetic of the general form
                    const SV_CONST double* M = (const SV_CONST double*)(a.gmat + (uint64_t)aux * kGenBlock);
#pragma unroll
                    for (int k = K0; k < R; k++) {
                        if (!((act >> k) & 1)) continue;
                        const SV_CONST double* m = M + 8 * (k < 2 ? p0 + k : p2 + k - 2);
                        const Acc a0 = (Acc)m[0], b0 = (Acc)m[2], c0 = (Acc)m[4], d0 = (Acc)m[6];
#pragma unroll
                        for (int r = 0; r < NR; r++) {
                            if (r & (1 << k)) continue;
                            const int r2 = r | (1 << k);
                            const Acc ur = vr[0][r], ui = vi[0][r], wr = vr[0][r2], wi = vi[0][r2];
                            vr[0][r] = fma(a0, ur, b0 * wr);
                            vi[0][r] = fma(a0, ui, b0 * wi);
                            vr[0][r2] = fma(c0, ur, d0 * wr);
                            vi[0][r2] = fma(c0, ui, d0 * wi);
                        }
                    }
                    return;
                }
                if (FEAT == 2 && (fl & MIX_GEN)) {
                    // general single-qubit layer: (u, v) <- (m00 u + m01 v, m10 u + m11 v)
                    const SV_CONST double* M = (const SV_CONST double*)(a.gmat + (uint64_t)aux * kGenBlock);
#pragma unroll
                    for (int k = K0; k < R; k++) {
                        if (!((act >> k) & 1)) continue;
                        const SV_CONST double* m = M + 8 * (k < 2 ? p0 + k : p2 + k - 2);
                        const Acc a0 = (Acc)m[0], a1 = (Acc)m[1], b0 = (Acc)m[2], b1 = (Acc)m[3];
                        const Acc c0 = (Acc)m[4], c1 = (Acc)m[5], d0 = (Acc)m[6], d1 = (Acc)m[7];
#pragma unroll
                        for (int r = 0; r < NR; r++) {
                            if (r & (1 << k)) continue;
                            const int r2 = r | (1 << k);
                            const Acc ur = vr[0][r], ui = vi[0][r], wr = vr[0][r2], wi = vi[0][r2];
                            vr[0][r] = fma(a0, ur, fma(-a1, ui, fma(b0, wr, -b1 * wi)));
                            vi[0][r] = fma(a0, ui, fma(a1, ur, fma(b0, wi, b1 * wr)));
                            vr[0][r2] = fma(c0, ur, fma(-c1, ui, fma(d0, wr, -d1 * wi)));
                            vi[0][r2] = fma(c0, ui, fma(c1, ur, fma(d0, wi, d1 * wr)));
                        }
                    }
                    return;
                }
#pragma unroll
                for (int k = K0; k < R; k++) {
                    // a slot that is not active here runs identity butterflies (t = 0): a branch
                    // would copy the amplitude registers at its join
                    const bool on = (act >> k) & 1;
                    const Acc tk = on ? tq : (Acc)0;
                    if (on && NV == 2 && FEAT == 1 && (fl & MIX_GBETA)) {
                        // Im(conj(lam_a) psi_b) + Im(conj(lam_b) psi_a), summed in FP64
                        double gb = 0.0;
#pragma unroll
                        for (int r = 0; r < NR; r++) {
                            if (r & (1 << k)) continue;
                            const int r2 = r | (1 << k);
                            const Acc q = vr[NV - 1][r] * vi[0][r2] - vi[NV - 1][r] * vr[0][r2] +
                                          vr[NV - 1][r2] * vi[0][r] - vi[NV - 1][r2] * vr[0][r];
                            gb += (double)q;
                        }
                        gsum += gb * pend[0] * pend[NV - 1];
                    }
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        const bool mine = NV == 1 || (fl & (1 << v)) != 0;
                        const Acc tv = mine ? tk : (Acc)0;
#pragma unroll
                        for (int r = 0; r < NR; r++) {
                            if (r & (1 << k)) continue;
                            const int r2 = r | (1 << k);
                            butterfly<Acc>(vr[v][r], vi[v][r], vr[v][r2], vi[v][r2], tv);
                        }
                        pend[v] *= (on && mine) ? opb : 1.0;
                    }
                }
                if (FEAT == 1 && NV == 1 && (fl & MIX_GBETA)) {
                    // quadratic forms 2 Re(conj(a) b) of the pairs of every active slot, from the
                    // values after the round (a butterfly leaves the form of every qubit unchanged)
                    double g2[2] = {0.0, 0.0};
#pragma unroll
                    for (int k = K0; k < R; k++) {
                        if (!((act >> k) & 1)) continue;
#pragma unroll
                        for (int r = 0; r < NR; r++) {
                            if (r & (1 << k)) continue;
                            const int r2 = r | (1 << k);
                            g2[k & 1] = fma((double)vr[0][r], (double)vr[0][r2], g2[k & 1]);
                            g2[k & 1] = fma((double)vi[0][r], (double)vi[0][r2], g2[k & 1]);
                        }
                    }
                    gsum += 2.0 * (g2[0] + g2[1]) * pend[0] * pend[0];
                }
            };
            using S0 = std::integral_constant<int, 0>;
            using S2 = std::integral_constant<int, 2>;
#pragma unroll 1
            for (int step = 0; step < K; step++) {
                const int j = fwd ? step : K - 1 - step;
                const uint32_t act = (a.act >> (8 * j)) & 255u;
                const bool sw = (act & 0x30u) != 0u;
                if (step > 0) {
                    exchange(j);
                    if (sw) {  // the layout a mixer ends in
                        round(S2{}, act >> 2, 0, lpair(j));
                        swap45();
                    }
                }
                round(S0{}, act & 15u, ab, ab + 2);
                if (step == 0 && sw) {  // the layout it begins in
                    swap45();
                    round(S2{}, act >> 2, 0, lpair(j));
                    if (K == 1) swap45();
                }
            }
            if (FEAT == 1 && (fl & MIX_GBETA)) {
                double gv[1] = {gsum};
                block_sums<1, NW>(gv, s_red, put_at(part0));
            }
            continue;
        }
        if constexpr (FEAT == 4) continue;
        // ---- OP_POINT in the current layout (0 or K - 1)
        const int es = cur == 0 ? 0 : 1;
        double e0 = es ? ev[1][0] : ev[0][0], d[R];
#pragma unroll
        for (int k = 0; k < R; k++) d[k] = (es ? ev[1][1 + k] : ev[0][1 + k]) - e0;
        // per-register loop in Gray-code order (E changes by +-d[k]), f(r, E(r))
        auto each = [&](auto f) {
            double e_run = e0;
#pragma unroll
            for (int i = 0; i < NR; i++) {
                const int r = i ^ (i >> 1);
                if (i > 0) {
                    const int k = __builtin_ctz(i);
                    e_run += ((r >> k) & 1) ? d[k] : -d[k];
                }
                f(r, e_run + lane_value(es ? ql[1] : ql[0], r));
            }
        };
        if (fl & (PT_REDUCE | PT_SPINZ)) {
            double rv[3] = {0.0, 0.0, 0.0};
            double Sk[R];
#pragma unroll
            for (int k = 0; k < R; k++) Sk[k] = 0.0;
            each([&](int r, double e) {
                const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                const double p2 = fma(pr, pr, pi * pi);
                rv[0] += p2;
                rv[1] = fma(e, p2, rv[1]);
                if (fabs(e - a.emin) <= a.etol) rv[2] += p2;
                if constexpr (FEAT == 2)
#pragma unroll
                    for (int k = 0; k < R; k++) Sk[k] += ((r >> k) & 1) ? p2 : -p2;
            });
            const double s2 = pend[0] * pend[0];
            const double nrm = rv[0] * s2;
            if (FEAT == 2 && (fl & PT_SPINZ)) {
                // entry l < T: sum of |psi|^2 s_l over the tile, entry T: sum of |psi|^2
                // (tile bit l is register bit l - ab or a bit of thr)
                double sv[T + 1];
#pragma unroll
                for (int l = 0; l < T; l++) {
                    const int k = l - ab;
                    double x = ((thr >> l) & 1u) ? nrm : -nrm;
#pragma unroll
                    for (int q = 0; q < R; q++)
                        if (k == q) x = Sk[q] * s2;
                    sv[l] = x;
                }
                sv[T] = nrm;
                const int ncol = a.spin_cols;
                block_sums<T + 1, NW>(sv, s_red, [&](int i, double x) {
                    if (i < ncol) part[(uint64_t)(aux + i) * a.ntiles + tile] = x;
                });
            }
            if (fl & PT_REDUCE) {
#pragma unroll
                for (int i = 0; i < 3; i++) rv[i] *= s2;
                block_sums<3, NW>(rv, s_red, put_at(part0));
            }
        }
        if constexpr (NV == 2) {
            if (fl & PT_LAM_INIT) {
                each([&](int r, double e) {
                    vr[1][r] = (Acc)(e * (double)vr[0][r]);
                    vi[1][r] = (Acc)(e * (double)vi[0][r]);
                });
                pend[1] = pend[0];
            }
            if (fl & PT_GGAMMA) {
                double gv[1] = {0.0};
                each([&](int r, double e) {
                    const Acc q = vr[1][r] * vi[0][r] - vi[1][r] * vr[0][r];
                    gv[0] += e * (double)q;
                });
                gv[0] *= pend[0] * pend[1];
                block_sums<1, NW>(gv, s_red, put_at(part2));
            }
        } else if constexpr (FEAT == 1) {
            if (fl & PT_ZETA) {
                const double zt = second ? -opb : opb;
                each([&](int r, double e) {
                    const double te = zt * e;
                    const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                    vr[0][r] = (Acc)fma(-te, pi, pr);
                    vi[0][r] = (Acc)fma(te, pr, pi);
                });
            }
            if (fl & PT_EFORM) {
                double gv[1] = {0.0};
                each([&](int r, double e) {
                    const double pr = (double)vr[0][r], pi = (double)vi[0][r];
                    gv[0] = fma(e, fma(pr, pr, pi * pi), gv[0]);
                });
                gv[0] *= pend[0] * pend[0];
                block_sums<1, NW>(gv, s_red, put_at(part2));
            }
        }
        // Every phase also takes the pending scale, so that it does not pile up over the passes of a
        // program that runs in one launch (cos(beta) per qubit and mixer: single precision overflows
        // after some 20 layers of 13 qubits).  The vectors of an adjoint sweep carry the same scale
        // from PT_LAM_INIT on; a ratio other than 1 goes into lambda.
        double psc = 1.0;
        if (fl & (PT_PHASE_PSI | PT_PHASE_LAM)) {
            psc = pend[0];
            if constexpr (NV == 2) {
                const Acc q = (Acc)(pend[1] / psc);
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    vr[1][r] *= q;
                    vi[1][r] *= q;
                }
                pend[1] = 1.0;
            }
            pend[0] = 1.0;
        }
        if ((fl & (PT_PHASE_PSI | PT_PHASE_LAM)) && a.lut_n > 0) {
            // Energies on the grid (2 i - lut_n + 1) / q, 0 <= i < lut_n: the factors of all of them,
            // with the pending scale, in LDS; then one look-up per amplitude (220 instructions per
            // thread and phase instead of 540).
            __syncthreads();  // the look-ups of the phase before
            for (int i = (int)t; i < a.lut_n; i += NT) {
                const double2 f = cis(opa * ((double)(2 * i - a.lut_n + 1) * a.lut_step));
                A2 x;
                x.x = (Acc)(f.x * psc);
                x.y = (Acc)(f.y * psc);
                s_lut[i] = x;
            }
            const double hq = 0.5 / a.lut_step;
            constexpr int LS = (int)sizeof(A2);
            int run = (int)fma(e0, hq, 0.5 * (double)(a.lut_n - 1)) * LS;
            const int qi = (int)((es ? ql[1] : ql[0]) * hq) * LS;
            int di[R];
#pragma unroll
            for (int k = 0; k < R; k++) di[k] = (int)(d[k] * hq) * LS;
            __syncthreads();
            const char* lut = reinterpret_cast<const char*>(s_lut);
#pragma unroll
            for (int i = 0; i < NR; i++) {
                const int r = i ^ (i >> 1);
                if (i > 0) {
                    const int k = __builtin_ctz(i);
                    run += ((r >> k) & 1) ? di[k] : -di[k];
                }
                const A2 c = *reinterpret_cast<const A2*>(lut + (run + __builtin_amdgcn_readlane(qi, r)));
#pragma unroll
                for (int v = 0; v < NV; v++) {
                    const Acc xr = vr[v][r], xi = vi[v][r];
                    vr[v][r] = mul_re(xr, xi, c.x, c.y);
                    vi[v][r] = mul_im(xr, xi, c.x, c.y);
                }
            }
        } else if (fl & (PT_PHASE_PSI | PT_PHASE_LAM)) {
            // e^{-i gamma E(r)} = e^{-i gamma E(0)} prod_k e^{-i gamma r_k d_k} e^{-i gamma Q(r)};
            // lane r of every wave forms the factor of Q(r), which all lanes then read
            const double2 qf = cis(opa * (es ? ql[1] : ql[0]));
            double2 gk[R];
#pragma unroll
            for (int k = 0; k < R; k++) gk[k] = cis(opa * d[k]);
            double2 run = cis(opa * e0);
            run.x *= psc;
            run.y *= psc;
#pragma unroll
            for (int i = 0; i < NR; i++) {
                const int r = i ^ (i >> 1);
                if (i > 0) {
                    const int k = __builtin_ctz(i);
                    const double gx = gk[k].x, gy = ((r >> k) & 1) ? gk[k].y : -gk[k].y;
                    run = make_double2(mul_re(run.x, run.y, gx, gy), mul_im(run.x, run.y, gx, gy));
                }
                const double qx = lane_value(qf.x, r), qy = lane_value(qf.y, r);
                const Acc cr = (Acc)mul_re(run.x, run.y, qx, qy), ci = (Acc)mul_im(run.x, run.y, qx, qy);
#pragma unroll
                for (int v = 0; v < NV; v++) {
                    const Acc xr = vr[v][r], xi = vi[v][r];
                    vr[v][r] = mul_re(xr, xi, cr, ci);
                    vi[v][r] = mul_im(xr, xi, cr, ci);
                }
            }
        }
    }

    // ---- store, in layout 0 (the last layout holds the lowest tile bits in registers)
    if (cur != 0 && a.store != 0) {
        if (swaps(cur)) swap45();
        exchange(0);
        if (swaps(0)) swap45();
    }
    {
        uint32_t gb[R];
#pragma unroll
        for (int k = 0; k < R; k++) gb[k] = goff(1u << (ab + k)) * ES;
#pragma unroll
        for (int v = 0; v < NV; v++) {
            if (!((a.store >> v) & 1)) continue;
            char* __restrict__ dst = reinterpret_cast<char*>(v == 0 ? a.psi : a.lam);
            const Acc sc = (Acc)pend[v];
            uint32_t off = (base32 | goff(thr)) * ES;
            if (ph == 0u) {
#pragma unroll
                for (int i = 0; i < NR; i++) {
                    if (i > 0) off ^= gb[__builtin_ctz(i)];
                    const int r = i ^ (i >> 1);
                    V2 x;
                    x.x = (Real)(vr[v][r] * sc);
                    x.y = (Real)(vi[v][r] * sc);
                    *reinterpret_cast<V2*>(dst + off) = x;
                }
            } else {
#pragma unroll
                for (int r = 0; r < NR; r++) {
                    const uint32_t ur = (uint32_t)r << ab;
                    if (((thr | ur) & ph) != 0u) continue;
                    V2 x;
                    x.x = (Real)(vr[v][r] * sc);
                    x.y = (Real)(vi[v][r] * sc);
                    *reinterpret_cast<V2*>(dst + (off ^ (goff(ur) * ES))) = x;
                }
            }
        }
    }
}

template <typename Real, typename Acc, int NV, int FEAT>
static int run_tile(int T, const TileArgs& a, hipStream_t st) {
    const dim3 grid(a.dual ? 2u : (unsigned)a.ntiles);
    // Double-precision variants with forms, general layers or spin sums need 280 registers.  Up to 256
    // tiles, at most one wave per SIMD runs anyway and may have them (within 256 they spill 44:
    // gradients n = 10 51.9 -> 45.9 us, n = 17 144 -> 138 us, n = 20 233 -> 211 us, observed runs
    // n = 17 74.5 -> 69 us); 512 tiles need two waves (n = 21 gradient 325 us, with one 359 us).
    constexpr int W = FEAT > 0 && sizeof(Acc) == 8 ? 1 : 2;
    switch (T) {
        case 10: hipLaunchKernelGGL((k_tile<Real, Acc, 10, 4, NV, FEAT, W>), grid, dim3(64), 0, st, a); break;
        case 11: hipLaunchKernelGGL((k_tile<Real, Acc, 11, 4, NV, FEAT, W>), grid, dim3(128), 0, st, a); break;
        case 12:
            if (a.ntiles <= 256)
                hipLaunchKernelGGL((k_tile<Real, Acc, 12, 4, NV, FEAT, W>), grid, dim3(256), 0, st, a);
            else
                hipLaunchKernelGGL((k_tile<Real, Acc, 12, 4, NV, FEAT, 2>), grid, dim3(256), 0, st, a);
            break;
        case 13: hipLaunchKernelGGL((k_tile<Real, Acc, 13, 4, NV, FEAT, 2>), grid, dim3(512), 0, st, a); break;
        default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

template <typename Real, typename Acc>
static int run_tile_feat(int T, const TileArgs& a, hipStream_t st) {
    if (a.feat == 0) return run_tile<Real, Acc, 1, 0>(T, a, st);
    if (a.feat == 3) return run_tile<Real, Acc, 1, 3>(T, a, st);
    if (a.feat == 4) return run_tile<Real, Acc, 1, 4>(T, a, st);
    return a.feat == 1 ? run_tile<Real, Acc, 1, 1>(T, a, st) : run_tile<Real, Acc, 1, 2>(T, a, st);
}

int launch_tile(int dtype, int nv, int T, const TileArgs& a, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (a.nops < 0 || a.nops > kMaxTileOps || a.nlayouts < 1 || a.nlayouts > kMaxLayouts || a.feat < 0 || a.feat > 4)
        return (int)hipErrorInvalidValue;
    if (nv == 2) return dtype == 1 ? run_tile<float, float, 2, 1>(T, a, st) : (int)hipErrorInvalidValue;
    if (dtype == 2) return run_tile_feat<double, double>(T, a, st);
    // one workgroup that runs a whole program keeps the amplitudes in double precision
    return a.resident ? run_tile_feat<float, double>(T, a, st) : run_tile_feat<float, float>(T, a, st);
}

// Second stage of the reductions of a program, one workgroup per result: result
// i sums its columns of the partial sums ([column][tile]) in a
// fixed order; a column may be signed by one bit of the tile index
// (spin expectations of qubits outside the tile).
__global__ void __launch_bounds__(256) k_gather(const GatherArgs a) {
    __shared__ double sh[4];
    const SV_CONST GatherArgs* ka = (const SV_CONST GatherArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    const int i = blockIdx.x, t = threadIdx.x;
    double v = 0.0;
    const uint32_t s0 = ka->first[i], s1 = ka->first[i + 1];
    for (uint32_t s = s0; s < s1; s++) {
        const uint32_t seg = ka->seg[s];
        const double* __restrict__ col = a.part + (uint64_t)(seg & 0xffffffu) * a.ntiles;
        const uint32_t sb = seg >> 24;  // 255: unsigned
#pragma unroll 4
        for (uint32_t w = t; w < a.ntiles; w += 256) {
            const double x = col[w];
            v += (sb != 255u && !((w >> sb) & 1u)) ? -x : x;
        }
    }
    v = wave_sum(v);
    if ((t & 63) == 0) sh[t >> 6] = v;
    __syncthreads();
    if (t == 0) a.out[i] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

int launch_gather(const GatherArgs& a, int n, void* stream) {
    hipLaunchKernelGGL(k_gather, dim3((unsigned)n), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace svk
