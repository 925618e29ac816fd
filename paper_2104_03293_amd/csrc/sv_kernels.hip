// gfx950 kernels of libsv: tile passes over the state vector, ground-state
// enumeration and deterministic second-stage reductions.
//
// A tile pass streams 2^T amplitudes per workgroup from HBM into registers
// (2^R per thread), runs a short program of ops on them and streams them
// back.  MIX applies exp(-i beta sigma^x_q) to every active qubit q of the
// tile as a 2-component update on register-local pairs (Eq.
// twocomponentupdates); qubits that are thread bits in the current layout are
// made register-local by an LDS exchange into the next layout.  POINT works
// per amplitude with the Ising energy E(z) of Eq. HC, built from the bits of z
// as  E = E_fixed + sum_l g_l s_l + (couplings inside the tile)  where E_fixed
// and the fields g_l seen by the tile bits are computed once per workgroup.
#include <hip/hip_runtime.h>

#include "sv_device.h"
#include "sv_internal.h"

namespace svk {

// Per-tile part of E(z) for one tile (one wave): E_fixed (fields and couplings
// among the bits outside the tile) and g_l = h_{P[l]} + sum of couplings from
// tile bit l to the fixed bits, written to the tile's row of the field table.
// Deterministic order.
__device__ void tile_fields_row(const IsingDev& is, const GeoBuf* geo, const TileGeom& tg, uint64_t base, int T,
                                double* __restrict__ row) {
    const int lane = threadIdx.x & 63;
    double part = 0.0;
    for (int i = lane; i < is.n; i += 64)
        if (!tg.in_tile(i)) part += is.h[i] * spin_z(base, i);
    for (int k = lane; k < is.m; k += 64) {
        const int i = is.ei[k], j = is.ej[k];
        if (!tg.in_tile(i) && !tg.in_tile(j)) part += is.J[k] * spin_z(base, i) * spin_z(base, j);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) part += __shfl_xor(part, off);
    if (lane == kTF - 1) row[lane] = part;
    if (lane < kTF - 1) {
        const int P = lane < T ? geo->P[lane] : -1;
        double gv = 0.0;
        if (P >= 0) {
            gv = is.h[P];
            for (int q = is.adj_ptr[P]; q < is.adj_ptr[P + 1]; q++) {
                const int j = is.adj_nbr[q];
                if (!tg.in_tile(j)) gv += is.adj_J[q] * spin_z(base, j);
            }
        }
        row[lane] = gv;
    }
}

// Field table of an instance for one tile geometry, one wave per tile.
__global__ void __launch_bounds__(256) k_tile_fields(const TfArgs a) {
    const TileGeom tg{a.c, a.lo, a.g};
    const uint64_t stride = (uint64_t)gridDim.x * 4;
    for (uint64_t w = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); w < a.ntiles; w += stride)
        tile_fields_row(a.is, a.geo, tg, tg.base(w), a.T, a.tf + w * kTF);
}

// Phase tables of one call: qph[r] = exp(-i gamma Q[r]) and, for instances whose
// energies lie on the grid Z / q (integer or half-integer coefficients),
// lut[m + L] = exp(-i gamma m / q), m = -L..L.  One workgroup per job.
struct TableJobs {
    TableJob j[64];
};

__global__ void __launch_bounds__(256) k_tables(const TableJobs jobs, double2* __restrict__ out) {
    const TableJob jb = jobs.j[blockIdx.x];
    for (int r = threadIdx.x; r < jb.nr; r += 256) {
        double sn, cs;
        sincos(jb.gamma * jb.Q[r], &sn, &cs);
        out[jb.qph_off + r] = make_double2(cs, -sn);
    }
    if (jb.L >= 0) {
        for (int m = threadIdx.x; m <= 2 * jb.L; m += 256) {
            double sn, cs;
            sincos(jb.gamma * ((double)(m - jb.L) * jb.qinv), &sn, &cs);
            out[jb.lut_off + m] = make_double2(cs, -sn);
        }
    }
}

// Column sums of partials[nslots][nrows] in a fixed order: out[dst[s]] (+)= sum.
// Two launches: kReduceBlocks workgroups each sum a contiguous run of rows
// (strided per thread, then a tree) into stage[block][slot]; one workgroup then
// adds the blocks' sums in a tree.  The order depends only on nrows.
struct SlotDst {
    int d[kMaxSlots];
};

__global__ void __launch_bounds__(256) k_reduce_rows(const double* __restrict__ partials, uint64_t nrows, int nslots,
                                                     double* __restrict__ stage) {
    __shared__ double sh[kMaxSlots][256];
    const int t = threadIdx.x;
    const uint64_t per = (nrows + gridDim.x - 1) / gridDim.x;
    const uint64_t r0 = (uint64_t)blockIdx.x * per;
    const uint64_t r1 = r0 + per < nrows ? r0 + per : nrows;
    double v[kMaxSlots];
#pragma unroll
    for (int q = 0; q < kMaxSlots; q++) v[q] = 0.0;
    for (uint64_t i = r0 + t; i < r1; i += 256)
#pragma unroll
        for (int q = 0; q < kMaxSlots; q++)
            if (q < nslots) v[q] += partials[q * nrows + i];
#pragma unroll
    for (int q = 0; q < kMaxSlots; q++) sh[q][t] = v[q];
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w)
#pragma unroll
            for (int q = 0; q < kMaxSlots; q++) sh[q][t] += sh[q][t + w];
        __syncthreads();
    }
    if (t < nslots) stage[blockIdx.x * kMaxSlots + t] = sh[t][0];
}

__global__ void __launch_bounds__(256) k_reduce_slots(const double* __restrict__ stage, int nblocks, int nslots,
                                                      SlotDst dst, int accumulate, double* __restrict__ out) {
    __shared__ double sh[256];
    const int t = threadIdx.x;
    for (int q = 0; q < nslots; q++) {
        sh[t] = t < nblocks ? stage[t * kMaxSlots + q] : 0.0;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if (t < w) sh[t] += sh[t + w];
            __syncthreads();
        }
        if (t == 0) {
            const int d = dst.d[q];
            out[d] = accumulate ? out[d] + sh[0] : sh[0];
        }
        __syncthreads();
    }
}

// <sigma^z_i> from the per-tile spin partials, one workgroup per qubit in a fixed
// order: a qubit held by tile bit l sums entry l over the tiles; any other qubit
// is fixed within a tile, so it sums s_i(tile) times the tile's norm entry.
__global__ void __launch_bounds__(256) k_spin_reduce(const SpinArgs a) {
    __shared__ double sh[256];
    const int i = blockIdx.x;
    const int t = threadIdx.x;
    int l = -1;
    for (int q = 0; q < a.T; q++)
        if (a.qubit[q] == i) l = q;
    const TileGeom tg{a.c, a.lo, a.g};
    double v = 0.0;
    for (uint64_t w = t; w < a.ntiles; w += 256) {
        v += l >= 0 ? a.part[(uint64_t)l * a.ntiles + w] : spin_z(tg.base(w), i) * a.part[(kTF - 1) * a.ntiles + w];
    }
    sh[t] = v;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if (t < s) sh[t] += sh[t + s];
        __syncthreads();
    }
    if (t == 0) a.out[i] = sh[0];
}

int launch_spin_reduce(const SpinArgs& a, void* stream) {
    hipLaunchKernelGGL(k_spin_reduce, dim3((unsigned)a.n), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// Brute-force enumeration of E(z) over all basis states, tile by tile in layout 0.
template <int T, int R>
__global__ void __launch_bounds__(1 << (T - R)) k_ground(const GroundArgs a) {
    constexpr int NT = 1 << (T - R);
    constexpr int NR = 1 << R;
    constexpr int NW = NT / 64;
    constexpr int RLO = (R + 1) / 2;
    constexpr int RHI = R - RLO;
    __shared__ double s_g[kTF];
    __shared__ double s_e[NW];
    __shared__ unsigned long long s_c[NW], s_a[NW];

    const uint32_t t = threadIdx.x;
    const uint64_t tile = blockIdx.x;
    CGeoBuf* __restrict__ geo = (CGeoBuf*)a.geo;
    const TileGeom tg{a.c, a.lo, a.g};
    const uint64_t base = tg.base(tile);
    if (t < kTF) s_g[t] = a.tf[tile * kTF + t];
    __syncthreads();

    CGeoLayout* L = &geo->L[0];
    const uint32_t thr_u = thread_index_bits<T - R>(t, L->tmask);
    const uint64_t thr_goff = tg.gmap(thr_u);
    double f[R];
    const double e0 = thread_energy<R, T - R>(L, geo, t, s_g, f);
    double elo[1 << RLO], ehi[1 << RHI];
    elo[0] = e0;
#pragma unroll
    for (int k = 0; k < RLO; k++)
#pragma unroll
        for (int r = 0; r < (1 << k); r++) elo[r | (1 << k)] = elo[r] + 2.0 * f[k];
    ehi[0] = 0.0;
#pragma unroll
    for (int k = 0; k < RHI; k++)
#pragma unroll
        for (int r = 0; r < (1 << k); r++) ehi[r | (1 << k)] = ehi[r] + 2.0 * f[RLO + k];

    double emin = INFINITY;
    unsigned long long cnt = 0, first = ~0ull;
#pragma unroll
    for (int r = 0; r < NR; r++) {
        const uint32_t u = thr_u | L->reg_u[r];
        if ((u & a.phantom) != 0u) continue;
        const double e = elo[r & ((1 << RLO) - 1)] + ehi[r >> RLO] + L->Q[r];
        if (a.mode == 0) {
            emin = fmin(emin, e);
        } else if (fabs(e - a.emin) <= a.etol) {
            const unsigned long long z = base | thr_goff | L->reg_goff[r];
            cnt++;
            first = z < first ? z : first;
        }
    }
    const int lane = t & 63, w = t >> 6;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        emin = fmin(emin, __shfl_xor(emin, off));
        cnt += __shfl_xor(cnt, off);
        const unsigned long long o = __shfl_xor(first, off);
        first = o < first ? o : first;
    }
    if (lane == 0) {
        s_e[w] = emin;
        s_c[w] = cnt;
        s_a[w] = first;
    }
    __syncthreads();
    if (t == 0) {
        double e = s_e[0];
        unsigned long long c2 = s_c[0], f2 = s_a[0];
        for (int ww = 1; ww < NW; ww++) {
            e = fmin(e, s_e[ww]);
            c2 += s_c[ww];
            f2 = s_a[ww] < f2 ? s_a[ww] : f2;
        }
        if (a.mode == 0) {
            a.part_e[tile] = e;
        } else {
            a.part_cnt[tile] = c2;
            a.part_arg[tile] = f2;
        }
    }
}

__global__ void __launch_bounds__(256) k_ground_finish(const GroundArgs a, double* out_e,
                                                       unsigned long long* out_cnt,
                                                       unsigned long long* out_arg) {
    __shared__ double se[256];
    __shared__ unsigned long long sc[256], sa[256];
    const int t = threadIdx.x;
    double e = INFINITY;
    unsigned long long c = 0, f = ~0ull;
    for (uint64_t i = t; i < a.ntiles; i += 256) {
        if (a.mode == 0) {
            e = fmin(e, a.part_e[i]);
        } else {
            c += a.part_cnt[i];
            f = a.part_arg[i] < f ? a.part_arg[i] : f;
        }
    }
    se[t] = e;
    sc[t] = c;
    sa[t] = f;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) {
            se[t] = fmin(se[t], se[t + w]);
            sc[t] += sc[t + w];
            sa[t] = sa[t + w] < sa[t] ? sa[t + w] : sa[t];
        }
        __syncthreads();
    }
    if (t == 0) {
        if (a.mode == 0) {
            *out_e = se[0];
        } else {
            *out_cnt = sc[0];
            *out_arg = sa[0];
        }
    }
}

// ----------------------------------------------------------------------------- dispatch
// Tile shapes.  complex128: T = 13 (128 KiB tiles).  complex64: T = 14 for
// one-vector programs; adjoint programs use T = 13 for both vectors, the
// largest two-vector tile whose kernel fits the register file.
Shape shape_for(int dtype, int nv, bool grad) {
    if (dtype == 2) return nv == 1 ? Shape{13, 5} : Shape{13, 4};
    if (!grad) return Shape{14, 5};
    return nv == 1 ? Shape{13, 5} : Shape{13, 4};
}

int launch_pass(int dtype, int nv, int T, int R, const PassArgs& a, void* stream) {
    if (nv == 2 && a.nslots > 4) return (int)hipErrorInvalidValue;
    if (a.nlayouts < 1 || a.nlayouts > kMaxLayouts) return (int)hipErrorInvalidValue;
    if (dtype == 2) return nv == 1 ? launch_pass_c128(T, a, stream) : launch_pass_c128_pair(a, stream);
    return nv == 1 ? launch_pass_c64(T, a, stream) : launch_pass_c64_pair(T, R, a, stream);
}

// Streaming ceiling of a tile geometry: every workgroup loads its tile (2^T
// amplitudes, the pass's lane order: thread t holds tile-local indices
// t + r 2^(T-R)) with nontemporal loads and stores it back unchanged, in the
// passes' XCD-aware tile order.  No arithmetic.
template <typename V2, int T, int R, int MINB>
__global__ void __launch_bounds__(1 << (T - R), MINB) k_stream(V2* __restrict__ p, const StreamArgs a) {
    constexpr int NT = 1 << (T - R);
    constexpr int NR = 1 << R;
    uint64_t tile = blockIdx.x;
    if (a.xcd > 0) {
        const int kb = 2 + a.xcd;
        if ((a.ntiles & ((1ull << kb) - 1ull)) == 0 && gridDim.x == a.ntiles)
            tile = (uint64_t)(blockIdx.x & ((1u << kb) - 1u)) * (a.ntiles >> kb) + (blockIdx.x >> kb);
    }
    const TileGeom tg{a.c, a.lo, a.g};
    V2* __restrict__ q = p + tg.base(tile);
    V2 v[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) v[r] = ld_nt(q + tg.gmap(threadIdx.x + (uint32_t)r * NT));
    // XOR with a mask that is zero at run time: the stores cannot be proven to
    // write back what was loaded, so the compiler keeps them
#pragma unroll
    for (int r = 0; r < NR; r++) {
        if constexpr (sizeof(v[r].x) == 8) {
            v[r].x = __longlong_as_double(__double_as_longlong(v[r].x) ^ (long long)a.mask);
            v[r].y = __longlong_as_double(__double_as_longlong(v[r].y) ^ (long long)a.mask);
        } else {
            v[r].x = __int_as_float(__float_as_int(v[r].x) ^ (int)a.mask);
            v[r].y = __int_as_float(__float_as_int(v[r].y) ^ (int)a.mask);
        }
    }
#pragma unroll
    for (int r = 0; r < NR; r++) st_nt(q + tg.gmap(threadIdx.x + (uint32_t)r * NT), v[r]);
}

int launch_stream(int dtype, void* p, const StreamArgs& a, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (dtype == 2)
        hipLaunchKernelGGL((k_stream<double2, 13, 5, 2>), dim3((unsigned)a.ntiles), dim3(256), 0, st,
                           (double2*)p, a);
    else
        hipLaunchKernelGGL((k_stream<float2, 14, 5, 4>), dim3((unsigned)a.ntiles), dim3(512), 0, st,
                           (float2*)p, a);
    return (int)hipGetLastError();
}

int launch_tables(const TableJob* jobs, int njobs, double2* out, void* stream) {
    for (int s = 0; s < njobs; s += 64) {
        TableJobs tj;
        const int cnt = njobs - s < 64 ? njobs - s : 64;
        for (int i = 0; i < cnt; i++) tj.j[i] = jobs[s + i];
        hipLaunchKernelGGL(k_tables, dim3(cnt), dim3(256), 0, (hipStream_t)stream, tj, out);
        const int e = (int)hipGetLastError();
        if (e) return e;
    }
    return 0;
}

int launch_reduce_slots(const double* partials, uint64_t nrows, int nslots, const int* dst, int accumulate,
                        double* out, double* stage, void* stream) {
    SlotDst d;
    for (int s = 0; s < kMaxSlots; s++) d.d[s] = s < nslots ? dst[s] : 0;
    const uint64_t want = (nrows + 2047) / 2048;  // about 2048 rows per workgroup
    const int nb = (int)(want < (uint64_t)kReduceBlocks ? (want > 0 ? want : 1) : kReduceBlocks);
    hipLaunchKernelGGL(k_reduce_rows, dim3(nb), dim3(256), 0, (hipStream_t)stream, partials, nrows, nslots, stage);
    hipLaunchKernelGGL(k_reduce_slots, dim3(1), dim3(256), 0, (hipStream_t)stream, stage, nb, nslots, d, accumulate,
                       out);
    return (int)hipGetLastError();
}

int launch_tile_fields(const TfArgs& a, void* stream) {
    const uint64_t blocks = (a.ntiles + 3) / 4;
    const unsigned grid = (unsigned)(blocks < 65536 ? blocks : 65536);
    hipLaunchKernelGGL(k_tile_fields, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_ground(int dtype, const GroundArgs& a, void* stream) {
    if (dtype == 2)
        hipLaunchKernelGGL((k_ground<13, 5>), dim3((unsigned)a.ntiles), dim3(256), 0, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL((k_ground<14, 5>), dim3((unsigned)a.ntiles), dim3(512), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_ground_finish(const GroundArgs& a, double* out_e, uint64_t* out_cnt, uint64_t* out_arg,
                         void* stream) {
    hipLaunchKernelGGL(k_ground_finish, dim3(1), dim3(256), 0, (hipStream_t)stream, a, out_e,
                       (unsigned long long*)out_cnt, (unsigned long long*)out_arg);
    return (int)hipGetLastError();
}

}  // namespace svk

// ============================================================================ batch scan
// p = 1 landscape over many small instances (Sec. III.C.1, Fig. 5): for each
// instance i and grid point (gamma_a, beta_b), psi = exp(-i beta_b H_D)
// exp(-i gamma_a H_C) |+>, then <H_C> and the ground-state probability.
namespace svk {

// Energy tables E_i(z) for every instance (Eq. HC), one thread per basis state;
// integer-valued instances also get the 16-bit table index E(z) - lut_lo.
__global__ void __launch_bounds__(256) k_batch_energy(const BatchArgs a) {
    const int i = blockIdx.y;
    const BatchInst in = a.inst[i];
    const uint64_t N = 1ull << in.n;
    for (uint64_t z = (uint64_t)blockIdx.x * 256 + threadIdx.x; z < N; z += (uint64_t)gridDim.x * 256) {
        double e = 0.0;
        for (int q = 0; q < in.n; q++) e += a.h[in.hoff + q] * (((z >> q) & 1) ? 1.0 : -1.0);
        for (int k = 0; k < in.m; k++) {
            const int u = a.ei[in.coff + k], v = a.ej[in.coff + k];
            const double su = ((z >> u) & 1) ? 1.0 : -1.0, sv = ((z >> v) & 1) ? 1.0 : -1.0;
            e += a.J[in.coff + k] * su * sv;
        }
        a.etab[in.eoff + z] = e;
        if (in.lut_n > 0) a.eidx[in.eoff + z] = (uint16_t)((int)e - in.lut_lo);
    }
}

// Minimum of each energy table (one workgroup per instance).
__global__ void __launch_bounds__(256) k_batch_emin(const BatchArgs a, BatchInst* inst) {
    __shared__ double sh[256];
    const int i = blockIdx.x;
    const BatchInst in = a.inst[i];
    const uint64_t N = 1ull << in.n;
    double e = INFINITY;
    for (uint64_t z = threadIdx.x; z < N; z += 256) e = fmin(e, a.etab[in.eoff + z]);
    sh[threadIdx.x] = e;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] = fmin(sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) inst[i].emin = sh[0];
}

constexpr int kBatchUnroll = 4;  // table entries in flight per thread

// One workgroup per CU holds the LDS state, with NTH threads (complex128: four
// waves, its register blocks need more than the 256 registers that two waves
// per SIMD leave; complex64: four or eight).
template <typename Real>
struct BatchCfg {
    static constexpr int G = sizeof(Real) == 4 ? 4 : 3;  // LDS swizzle width
};

__device__ __forceinline__ uint32_t bswz(uint32_t z, int G) { return lds_swizzle(z, G); }

// Hides a per-thread value from loop-invariant code motion: the block addresses
// derived from it are then formed next to their use instead of being hoisted out
// of the slice and beta loops and kept live (and spilled) across them.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// exp(-i beta sigma^x) / cos(beta) on the NB index bits of 2^NB register values,
// t = tan(beta): the pair (a, b) becomes (a - i t b, b - i t a).  The scan applies
// the factor cos(beta)^{2n} to the reduced sums instead of to every amplitude.
template <typename Real, int NB>
__device__ __forceinline__ void reg_mix(typename V2T<Real>::type (&v)[1 << NB], Real t) {
#pragma unroll
    for (int k = 0; k < NB; k++) {
#pragma unroll
        for (int r = 0; r < (1 << NB); r++) {
            if (r & (1 << k)) continue;
            const int r2 = r | (1 << k);
            const Real ar = v[r].x, ai = v[r].y, br = v[r2].x, bi = v[r2].y;
            v[r].x = ar + t * bi;
            v[r].y = ai - t * br;
            v[r2].x = br + t * ai;
            v[r2].y = bi - t * ar;
        }
    }
}

// exp(-i beta sigma^x) / cos(beta) on every qubit of an LDS-resident state of 2^nb
// elements (bits 0..nb-1), in register blocks of 5 bits; t = tan(beta).
template <typename Real, int NTH>
__device__ void lds_mixer(typename V2T<Real>::type* st, int nb, Real t) {
    using V2 = typename V2T<Real>::type;
    constexpr int G = BatchCfg<Real>::G;
    const int nblk = (nb + 4) / 5;
    uint32_t done = 0;
    for (int j = 0; j < nblk; j++) {
        const int a0 = min(5 * j, nb - 5);
        uint32_t act = 0;
        for (int k = 0; k < 5; k++)
            if (!((done >> (a0 + k)) & 1u)) act |= 1u << k;
        done |= 31u << a0;
        const uint32_t nq = 1u << (nb - 5);
        for (uint32_t q = threadIdx.x; q < nq; q += NTH) {
            const uint32_t zb = (q & ((1u << a0) - 1u)) | ((q >> a0) << (a0 + 5));
            const uint32_t bz = bswz(zb, G);
            V2 v[32];
#pragma unroll
            for (int r = 0; r < 32; r++) v[r] = st[bz ^ bswz((uint32_t)r << a0, G)];
#pragma unroll
            for (int k = 0; k < 5; k++) {
                if (!((act >> k) & 1u)) continue;
#pragma unroll
                for (int r = 0; r < 32; r++) {
                    if (r & (1 << k)) continue;
                    const int r2 = r | (1 << k);
                    const Real ar = v[r].x, ai = v[r].y, br = v[r2].x, bi = v[r2].y;
                    v[r].x = ar + t * bi;
                    v[r].y = ai - t * br;
                    v[r2].x = br + t * ai;
                    v[r2].y = bi - t * ar;
                }
            }
#pragma unroll
            for (int r = 0; r < 32; r++) st[bz ^ bswz((uint32_t)r << a0, G)] = v[r];
        }
        __syncthreads();
    }
}

// Persistent scan: workgroups take (instance, gamma) units from a queue, largest
// n first, and evaluate every beta of the grid for that unit.  Integer-valued
// instances read 16-bit table indices (E(z) - lut_lo) and take the phase
// 2^{-n/2} exp(-i gamma E) from an LDS table; the others read E(z) in FP64 and
// take sincos.  Table reads are issued kBatchUnroll at a time per thread.
// SLOTS = false drops the slot code (registers for the LDS-resident path only):
// the variant for queues that hold only units with n <= S.
template <typename Real, int NTH, int S, int LUTN, int MINW = 1, bool SLOTS = true>
__global__ void __launch_bounds__(NTH, MINW) k_batch_scan(const BatchArgs a) {
    using V2 = typename V2T<Real>::type;
    constexpr int G = BatchCfg<Real>::G;
    constexpr int U = kBatchUnroll;
    static_assert(S >= 10 && S <= 15, "slice rounds assume 10 <= S <= 15");
    __shared__ V2 st[1 << S];
    __shared__ V2 lut[LUTN];  // 2^{-n/2} exp(-i gamma E), rounded once to the storage type
    __shared__ double red[NTH / 64][2];
    __shared__ int s_unit;
    const int t = threadIdx.x;
    V2* slot = reinterpret_cast<V2*>(a.scratch) + (uint64_t)blockIdx.x * a.scratch_elems;

    for (;;) {
        if (t == 0) s_unit = (int)atomicAdd(a.counter, 1u);
        __syncthreads();
        const int u = s_unit;
        __syncthreads();
        if (u >= a.nunits) break;  // every wave of the workgroup sees the same u
        const BatchInst in = a.inst[a.unit_inst[u]];
        const double gam = a.gammas[a.unit_gam[u]];
        const int n = in.n;
        const double amp0 = exp2(-0.5 * n);
        const double* E = a.etab + in.eoff;
        const uint16_t* X = a.eidx + in.eoff;
        const bool intE = in.lut_n > 0;
        const int xmin = intE ? (int)in.emin - in.lut_lo : 0;  // table index of the ground energy
        if (intE) {
            for (int m = t; m < in.lut_n; m += NTH) {
                double sn, cs;
                sincos(gam * (double)(in.lut_lo + m), &sn, &cs);
                lut[m].x = (Real)(amp0 * cs);
                lut[m].y = (Real)(-amp0 * sn);
            }
            __syncthreads();
        }
        // phase state 2^{-n/2} exp(-i gamma E(z)) for U consecutive-stride entries z0 + j NTH
        auto phi_block = [&](uint64_t base, uint32_t z0, uint32_t lim, V2 (&out)[U]) {
            if (intE) {
                uint16_t x[U];
#pragma unroll
                for (int j = 0; j < U; j++) {
                    const uint32_t z = z0 + j * NTH;
                    x[j] = z < lim ? X[base + z] : (uint16_t)0;
                }
#pragma unroll
                for (int j = 0; j < U; j++) out[j] = lut[x[j]];
            } else {
                double e[U];
#pragma unroll
                for (int j = 0; j < U; j++) {
                    const uint32_t z = z0 + j * NTH;
                    e[j] = z < lim ? E[base + z] : 0.0;
                }
                // one sincos at a time (each needs many temporaries)
#pragma unroll 1
                for (int j = 0; j < U; j++) {
                    double sn, cs;
                    sincos(gam * e[j], &sn, &cs);
                    out[j].x = (Real)(amp0 * cs);
                    out[j].y = (Real)(-amp0 * sn);
                }
            }
        };
        // <H_C> and P_gs terms of U entries
        // (amplitude j sits at index z0 + j NTH; its energy is that of index (z0 + j NTH) ^ fl)
        auto obs_block = [&](uint64_t base, uint32_t z0, uint32_t lim, uint32_t fl, const V2 (&v)[U], double& r_e,
                             double& r_p) {
            if (intE) {
                uint16_t x[U];
#pragma unroll
                for (int j = 0; j < U; j++) {
                    const uint32_t z = z0 + j * NTH;
                    x[j] = z < lim ? X[base + (z ^ fl)] : (uint16_t)0;
                }
#pragma unroll
                for (int j = 0; j < U; j++) {
                    if (z0 + j * NTH >= lim) continue;
                    const double p2 = (double)v[j].x * v[j].x + (double)v[j].y * v[j].y;
                    r_e += (double)(in.lut_lo + (int)x[j]) * p2;
                    if ((int)x[j] == xmin) r_p += p2;
                }
            } else {
                double e[U];
#pragma unroll
                for (int j = 0; j < U; j++) {
                    const uint32_t z = z0 + j * NTH;
                    e[j] = z < lim ? E[base + (z ^ fl)] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < U; j++) {
                    if (z0 + j * NTH >= lim) continue;
                    const double p2 = (double)v[j].x * v[j].x + (double)v[j].y * v[j].y;
                    r_e += e[j] * p2;
                    if (fabs(e[j] - in.emin) <= in.etol) r_p += p2;
                }
            }
        };
        for (int b = 0; b < a.nb; b++) {
            // beta -> beta + pi multiplies the state by (-1)^n, and beta -> beta + pi/2
            // applies -i sigma^x to every qubit, which moves the amplitude of z to the
            // complement of z.  So beta is reduced to |beta| <= pi/4, the mixers run in
            // the tangent form (|tan| <= 1), the tables are read at z ^ fl, and the sums
            // take the factor cos(beta)^{2n} at the end.
            double bb = remainder(a.betas[b], M_PI);
            uint32_t fl = 0u;
            if (fabs(bb) > 0.25 * M_PI) {
                bb -= copysign(0.5 * M_PI, bb);
                fl = (uint32_t)((1ull << n) - 1ull);
            }
            const Real tq = (Real)tan(bb);
            double r_e = 0.0, r_p = 0.0;
            if (n <= S) {
                const uint32_t N = 1u << n;
                for (uint32_t z0 = t; z0 < N; z0 += NTH * U) {
                    V2 v[U];
                    phi_block(0, z0, N, v);
#pragma unroll
                    for (int j = 0; j < U; j++)
                        if (z0 + j * NTH < N) st[bswz(z0 + j * NTH, G)] = v[j];
                }
                __syncthreads();
                if (n >= 5) {
                    lds_mixer<Real, NTH>(st, n, tq);
                } else {
                    if (t == 0) {  // tiny states: plain pair loops
                        for (int q = 0; q < n; q++)
                            for (uint32_t z = 0; z < N; z++) {
                                if ((z >> q) & 1u) continue;
                                V2& x = st[bswz(z, G)];
                                V2& y = st[bswz(z | (1u << q), G)];
                                const Real ar = x.x, ai = x.y, br = y.x, bi = y.y;
                                x.x = ar + tq * bi;
                                x.y = ai - tq * br;
                                y.x = br + tq * ai;
                                y.y = bi - tq * ar;
                            }
                    }
                    __syncthreads();
                }
                for (uint32_t z0 = t; z0 < N; z0 += NTH * U) {
                    V2 v[U];
#pragma unroll
                    for (int j = 0; j < U; j++) {
                        const uint32_t z = z0 + j * NTH;
                        if (z < N) v[j] = st[bswz(z, G)];
                        else v[j].x = v[j].y = (Real)0;
                    }
                    obs_block(0, z0, N, fl, v, r_e, r_p);
                }
            } else if constexpr (SLOTS) {
                // low S bits slice by slice, written to this workgroup's slot: bits
                // S-5..S-1 in registers as the phases are formed, bits 0..4 in LDS,
                // bits 5..S-6 on the way from LDS to the slot
                const int nh = n - S;
                constexpr int LB = S - 5;
                constexpr int MB = S - 10;
                for (uint32_t sl = 0; sl < (1u << nh); sl++) {
                    const uint64_t off = (uint64_t)sl << S;
                    if (!intE) {
                        for (uint32_t z0 = t; z0 < (1u << S); z0 += NTH * U) {
                            V2 v[U];
                            phi_block(off, z0, 1u << S, v);
#pragma unroll
                            for (int j = 0; j < U; j++) st[bswz(z0 + j * NTH, G)] = v[j];
                        }
                        __syncthreads();
                    }
                    const uint16_t* Xs = X + off;  // uniform bases, 32-bit lane offsets
                    V2* Ss = slot + off;
                    for (uint32_t l = t; l < (1u << LB); l += NTH) {
                        const uint32_t bl = opaque(bswz(l, G));
                        V2 v[32];
                        if (intE) {
                            uint16_t x[32];
#pragma unroll
                            for (int r = 0; r < 32; r++) x[r] = Xs[l | ((uint32_t)r << LB)];
#pragma unroll
                            for (int r = 0; r < 32; r++) v[r] = lut[x[r]];
                        } else {
#pragma unroll
                            for (int r = 0; r < 32; r++) v[r] = st[bl ^ bswz((uint32_t)r << LB, G)];
                        }
                        reg_mix<Real, 5>(v, tq);
#pragma unroll
                        for (int r = 0; r < 32; r++) st[bl ^ bswz((uint32_t)r << LB, G)] = v[r];
                    }
                    __syncthreads();
                    for (uint32_t q = t; q < (1u << LB); q += NTH) {
                        const uint32_t bq = opaque(bswz(q << 5, G));
                        V2 v[32];
#pragma unroll
                        for (int r = 0; r < 32; r++) v[r] = st[bq ^ bswz((uint32_t)r, G)];
                        reg_mix<Real, 5>(v, tq);
#pragma unroll
                        for (int r = 0; r < 32; r++) st[bq ^ bswz((uint32_t)r, G)] = v[r];
                    }
                    __syncthreads();
                    for (uint32_t g = t; g < (1u << (S - MB)); g += NTH) {
                        const uint32_t zb = (g & 31u) | ((g >> 5) << (5 + MB));
                        const uint32_t bz = opaque(bswz(zb, G));
                        V2 v[1 << MB];
#pragma unroll
                        for (int r = 0; r < (1 << MB); r++) v[r] = st[bz ^ bswz((uint32_t)r << 5, G)];
                        reg_mix<Real, MB>(v, tq);
#pragma unroll
                        for (int r = 0; r < (1 << MB); r++) Ss[zb | ((uint32_t)r << 5)] = v[r];
                    }
                    __syncthreads();
                }
                // high bits: each thread holds the 2^nh amplitudes of one low index
                for (uint32_t l0 = t; l0 < (1u << S); l0 += NTH) {
                    const uint32_t l = opaque(l0);
                    V2 v[32];
#pragma unroll
                    for (int r = 0; r < 32; r++)
                        if (r < (1 << nh)) v[r] = slot[((uint32_t)r << S) | l];
#pragma unroll
                    for (int k = 0; k < 5; k++) {
                        if (k >= nh) continue;
#pragma unroll
                        for (int r = 0; r < 32; r++) {
                            if ((r & (1 << k)) || r >= (1 << nh)) continue;
                            const int r2 = r | (1 << k);
                            const Real ar = v[r].x, ai = v[r].y, br = v[r2].x, bi = v[r2].y;
                            v[r].x = ar + tq * bi;
                            v[r].y = ai - tq * br;
                            v[r2].x = br + tq * ai;
                            v[r2].y = bi - tq * ar;
                        }
                    }
                    if (intE) {
#pragma unroll
                        for (int r0 = 0; r0 < 32; r0 += U) {
                            uint16_t x[U];
#pragma unroll
                            for (int j = 0; j < U; j++)
                                x[j] = r0 + j < (1 << nh) ? X[(((uint32_t)(r0 + j) << S) | l) ^ fl] : (uint16_t)0;
#pragma unroll
                            for (int j = 0; j < U; j++) {
                                const int r = r0 + j;
                                if (r >= (1 << nh)) continue;
                                const double p2 = (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
                                r_e += (double)(in.lut_lo + (int)x[j]) * p2;
                                if ((int)x[j] == xmin) r_p += p2;
                            }
                        }
                    } else {
#pragma unroll
                        for (int r = 0; r < 32; r++) {
                            if (r >= (1 << nh)) continue;
                            const double p2 = (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
                            const double e = E[(((uint32_t)r << S) | l) ^ fl];
                            r_e += e * p2;
                            if (fabs(e - in.emin) <= in.etol) r_p += p2;
                        }
                    }
                }
                __syncthreads();  // slot reads done before the next beta overwrites it
            }
            // fixed-order workgroup sum
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                r_e += __shfl_xor(r_e, off);
                r_p += __shfl_xor(r_p, off);
            }
            if ((t & 63) == 0) {
                red[t >> 6][0] = r_e;
                red[t >> 6][1] = r_p;
            }
            __syncthreads();
            if (t == 0) {
                double se = 0.0, sp = 0.0;
                for (int w = 0; w < NTH / 64; w++) {
                    se += red[w][0];
                    sp += red[w][1];
                }
                const double cb = cos(bb), sc = pow(cb * cb, (double)n);  // the deferred cos(beta)^{2n}
                const uint64_t o = ((uint64_t)a.unit_inst[u] * a.ng + a.unit_gam[u]) * a.nb + b;
                a.out_e[o] = se * sc;
                a.out_p[o] = sp * sc;
            }
            __syncthreads();
        }
    }
}

int launch_batch_energy(const BatchArgs& a, int max_n, void* stream) {
    const unsigned gx = (unsigned)std::max(1, std::min(1024, (1 << max_n) / 256));
    hipLaunchKernelGGL(k_batch_energy, dim3(gx, a.ninst), dim3(256), 0, (hipStream_t)stream, a);
    int e = (int)hipGetLastError();
    if (e) return e;
    hipLaunchKernelGGL(k_batch_emin, dim3(a.ninst), dim3(256), 0, (hipStream_t)stream, a,
                       const_cast<BatchInst*>(a.inst));
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------- sliced states
// States larger than the LDS tile (n > S) go through a slab of a few hundred MB
// that stays in the last-level cache between two kernels, instead of a
// per-workgroup slot of 2^n amplitudes that streams through HBM:
//   k_batch_slices  one workgroup per (state, slice of 2^S amplitudes): phase
//                   state of the slice, mixer on the low S bits, slice -> slab;
//   k_batch_columns one workgroup per (state, block of 2^S amplitudes taken as
//                   2^(S - nh) columns of the 2^nh high-bit values): mixer on
//                   the high bits, <H_C> and P_gs partial sums;
//   k_batch_finish  one thread per state: its partials in a fixed order, times
//                   the deferred cos(beta)^{2n}.
// Mixer in the tangent form on |beta| <= pi/4 as in k_batch_scan; fl flips the
// table index where beta was moved by pi/2.
__device__ __forceinline__ double batch_reduce_beta(double beta, int n, uint32_t& fl) {
    double bb = remainder(beta, M_PI);
    fl = 0u;
    if (fabs(bb) > 0.25 * M_PI) {
        bb -= copysign(0.5 * M_PI, bb);
        fl = (uint32_t)((1ull << n) - 1ull);
    }
    return bb;
}

// <H_C> and P_gs of state s of a launch (qubits n, first unit u0, first group
// state base): its 2^nh partial sums in a fixed order, times cos(beta)^{2n}.
__device__ void batch_finish_state(const BatchArgs& a, int nh, int n, int u0, int64_t base, const double* part,
                                   int s) {
    const int64_t g = base + s;
    const int u = u0 + (int)(g / a.nb);
    const int b = (int)(g % a.nb);
    uint32_t fl;
    const double bb = batch_reduce_beta(a.betas[b], n, fl);
    double se = 0.0, sp = 0.0;
    const double* P = part + ((uint64_t)s << nh) * 2;
    for (int k = 0; k < (1 << nh); k++) {
        se += P[2 * k];
        sp += P[2 * k + 1];
    }
    const double cb = cos(bb), sc = pow(cb * cb, (double)n);  // the deferred cos(beta)^{2n}
    const uint64_t o = ((uint64_t)a.unit_inst[u] * a.ng + a.unit_gam[u]) * a.nb + b;
    a.out_e[o] = se * sc;
    a.out_p[o] = sp * sc;
}

// B: bits of a register block (5: 2^13 slices in rounds of 5, 5 and 3 bits; 4: 2^12
// slices in three rounds of 4 bits)
template <typename Real, int NTH, int S, int LUTN, int MINW, int B = 5>
__global__ void __launch_bounds__(NTH, MINW) k_batch_slices(const BatchArgs a) {
    using V2 = typename V2T<Real>::type;
    constexpr int G = BatchCfg<Real>::G;
    constexpr int U = kBatchUnroll;
    constexpr int NB = 1 << B;
    constexpr int LB = S - B;
    constexpr int MB = S - 2 * B;
    static_assert(MB >= 1 && MB <= B, "slice rounds assume B < S - B <= 2 B");
    static_assert((1 << S) % (NTH * kBatchUnroll) == 0, "phase loop assumes whole blocks");
    __shared__ V2 st[1 << S];
    __shared__ V2 lut[LUTN];  // 2^{-n/2} exp(-i gamma E), rounded once to the storage type
    const int t = threadIdx.x;
    const int n = a.s_n;
    const int nh = n - S;
    const uint32_t nsl = (uint32_t)a.s_count << nh;
    if (blockIdx.x >= nsl) {  // trailing workgroups: the previous launch's states
        const int fs = (int)(blockIdx.x - nsl) * NTH + t;
        if (fs < a.f_count) batch_finish_state(a, a.f_nh, a.f_n, a.f_u0, a.f_base, a.f_part, fs);
        return;
    }
    const uint32_t s = blockIdx.x >> nh;
    const uint32_t sl = blockIdx.x & ((1u << nh) - 1u);
    const int64_t g = a.s_base + s;
    const int u = a.s_u0 + (int)(g / a.nb);
    const int b = (int)(g % a.nb);
    const BatchInst in = a.inst[a.unit_inst[u]];
    const double gam = a.gammas[a.unit_gam[u]];
    const double amp0 = exp2(-0.5 * n);
    const bool intE = in.lut_n > 0;
    uint32_t fl;
    const Real tq = (Real)tan(batch_reduce_beta(a.betas[b], n, fl));
    const uint64_t off = in.eoff + ((uint64_t)sl << S);
    V2* __restrict__ Ss = reinterpret_cast<V2*>(a.slab) + ((uint64_t)s << n) + ((uint64_t)sl << S);
    if (intE) {
        for (int m = t; m < in.lut_n; m += NTH) {
            double sn, cs;
            sincos(gam * (double)(in.lut_lo + m), &sn, &cs);
            lut[m].x = (Real)(amp0 * cs);
            lut[m].y = (Real)(-amp0 * sn);
        }
    } else {
        const double* E = a.etab + off;
        for (uint32_t z0 = t; z0 < (1u << S); z0 += NTH * U) {
            double e[U];
#pragma unroll
            for (int j = 0; j < U; j++) e[j] = E[z0 + j * NTH];
#pragma unroll 1
            for (int j = 0; j < U; j++) {
                double sn, cs;
                sincos(gam * e[j], &sn, &cs);
                V2 v;
                v.x = (Real)(amp0 * cs);
                v.y = (Real)(-amp0 * sn);
                st[bswz(z0 + j * NTH, G)] = v;
            }
        }
    }
    __syncthreads();
    // bits S-B..S-1 in registers as the phases are formed
    const uint16_t* Xs = a.eidx + off;
    for (uint32_t l = t; l < (1u << LB); l += NTH) {
        const uint32_t bl = opaque(bswz(l, G));
        V2 v[NB];
        if (intE) {
            uint16_t x[NB];
#pragma unroll
            for (int r = 0; r < NB; r++) x[r] = Xs[l | ((uint32_t)r << LB)];
#pragma unroll
            for (int r = 0; r < NB; r++) v[r] = lut[x[r]];
        } else {
#pragma unroll
            for (int r = 0; r < NB; r++) v[r] = st[bl ^ bswz((uint32_t)r << LB, G)];
        }
        reg_mix<Real, B>(v, tq);
#pragma unroll
        for (int r = 0; r < NB; r++) st[bl ^ bswz((uint32_t)r << LB, G)] = v[r];
    }
    __syncthreads();
    // bits 0..B-1
    for (uint32_t q = t; q < (1u << LB); q += NTH) {
        const uint32_t bq = opaque(bswz(q << B, G));
        V2 v[NB];
#pragma unroll
        for (int r = 0; r < NB; r++) v[r] = st[bq ^ bswz((uint32_t)r, G)];
        reg_mix<Real, B>(v, tq);
#pragma unroll
        for (int r = 0; r < NB; r++) st[bq ^ bswz((uint32_t)r, G)] = v[r];
    }
    __syncthreads();
    // bits B..S-B-1 on the way from LDS to the slab
    for (uint32_t gq = t; gq < (1u << (S - MB)); gq += NTH) {
        const uint32_t zb = (gq & (NB - 1u)) | ((gq >> B) << (B + MB));
        const uint32_t bz = opaque(bswz(zb, G));
        V2 v[1 << MB];
#pragma unroll
        for (int r = 0; r < (1 << MB); r++) v[r] = st[bz ^ bswz((uint32_t)r << B, G)];
        reg_mix<Real, MB>(v, tq);
#pragma unroll
        for (int r = 0; r < (1 << MB); r++) Ss[zb | ((uint32_t)r << B)] = v[r];
    }
}

template <typename Real, int NTH, int S, int NH>
__global__ void __launch_bounds__(NTH) k_batch_columns(const BatchArgs a) {
    using V2 = typename V2T<Real>::type;
    constexpr int U = kBatchUnroll;
    constexpr int NV = 1 << NH;  // high-bit values of one column
    __shared__ double red[NTH / 64][2];
    const int t = threadIdx.x;
    const int n = S + NH;
    const uint32_t s = blockIdx.x >> NH;
    const uint32_t cb = blockIdx.x & (NV - 1u);
    const int64_t g = a.s_base + s;
    const int u = a.s_u0 + (int)(g / a.nb);
    const int b = (int)(g % a.nb);
    const BatchInst in = a.inst[a.unit_inst[u]];
    const bool intE = in.lut_n > 0;
    const int xmin = intE ? (int)in.emin - in.lut_lo : 0;  // table index of the ground energy
    uint32_t fl;
    const Real tq = (Real)tan(batch_reduce_beta(a.betas[b], n, fl));
    const V2* __restrict__ Sv = reinterpret_cast<const V2*>(a.slab) + ((uint64_t)s << n);
    const uint16_t* X = a.eidx + in.eoff;
    const double* E = a.etab + in.eoff;
    constexpr uint32_t ncol = 1u << (S - NH);  // columns of this workgroup
    const uint32_t c0 = cb << (S - NH);
    double r_e = 0.0, r_p = 0.0;
    for (uint32_t lc = t; lc < ncol; lc += NTH) {
        const uint32_t l = opaque(c0 + lc);
        V2 v[NV];
#pragma unroll
        for (int r = 0; r < NV; r++) v[r] = Sv[((uint32_t)r << S) | l];
        reg_mix<Real, NH>(v, tq);
        if (intE) {
#pragma unroll
            for (int r0 = 0; r0 < NV; r0 += U) {
                constexpr int W = NV < U ? NV : U;
                uint16_t x[W];
#pragma unroll
                for (int j = 0; j < W; j++) x[j] = X[(((uint32_t)(r0 + j) << S) | l) ^ fl];
#pragma unroll
                for (int j = 0; j < W; j++) {
                    const int r = r0 + j;
                    const double p2 = (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
                    r_e += (double)(in.lut_lo + (int)x[j]) * p2;
                    if ((int)x[j] == xmin) r_p += p2;
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < NV; r++) {
                const double p2 = (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
                const double e = E[(((uint32_t)r << S) | l) ^ fl];
                r_e += e * p2;
                if (fabs(e - in.emin) <= in.etol) r_p += p2;
            }
        }
    }
    // fixed-order workgroup sum
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        r_e += __shfl_xor(r_e, o);
        r_p += __shfl_xor(r_p, o);
    }
    if ((t & 63) == 0) {
        red[t >> 6][0] = r_e;
        red[t >> 6][1] = r_p;
    }
    __syncthreads();
    if (t == 0) {
        double se = 0.0, sp = 0.0;
        for (int w = 0; w < NTH / 64; w++) {
            se += red[w][0];
            sp += red[w][1];
        }
        a.part[2 * (uint64_t)blockIdx.x] = se;
        a.part[2 * (uint64_t)blockIdx.x + 1] = sp;
    }
}

// Six high bits (64 values per column): each column is held by a lane pair, 32
// values per lane; row bits 0-4 in registers, row bit 5 across the pair (both
// members take x <- x - i t x_partner).
template <typename Real, int S>
__global__ void __launch_bounds__(128) k_batch_columns_pair(const BatchArgs a) {
    using V2 = typename V2T<Real>::type;
    constexpr int U = kBatchUnroll;
    constexpr int NH = 6;
    constexpr int NTH = 128;
    static_assert(S - NH == 6, "a block of 64 columns per 128 threads");
    __shared__ double red[NTH / 64][2];
    const int t = threadIdx.x;
    const int n = S + NH;
    const uint32_t s = blockIdx.x >> NH;
    const uint32_t cb = blockIdx.x & ((1u << NH) - 1u);
    const int64_t g = a.s_base + s;
    const int u = a.s_u0 + (int)(g / a.nb);
    const int b = (int)(g % a.nb);
    const BatchInst in = a.inst[a.unit_inst[u]];
    const bool intE = in.lut_n > 0;
    const int xmin = intE ? (int)in.emin - in.lut_lo : 0;  // table index of the ground energy
    uint32_t fl;
    const Real tq = (Real)tan(batch_reduce_beta(a.betas[b], n, fl));
    const V2* __restrict__ Sv = reinterpret_cast<const V2*>(a.slab) + ((uint64_t)s << n);
    const uint16_t* X = a.eidx + in.eoff;
    const double* E = a.etab + in.eoff;
    const uint32_t h = (uint32_t)t & 1u;  // upper or lower 32 rows
    const uint32_t l = opaque((cb << (S - NH)) + ((uint32_t)t >> 1));
    const uint32_t r0 = h << 5;
    V2 v[32];
#pragma unroll
    for (int j = 0; j < 32; j++) v[j] = Sv[((r0 + (uint32_t)j) << S) | l];
    reg_mix<Real, 5>(v, tq);
#pragma unroll
    for (int j = 0; j < 32; j++) {
        const Real pr = __shfl_xor(v[j].x, 1), pi = __shfl_xor(v[j].y, 1);
        v[j].x = fma(tq, pi, v[j].x);
        v[j].y = fma(-tq, pr, v[j].y);
    }
    double r_e = 0.0, r_p = 0.0;
    if (intE) {
#pragma unroll
        for (int j0 = 0; j0 < 32; j0 += U) {
            uint16_t x[U];
#pragma unroll
            for (int j = 0; j < U; j++) x[j] = X[(((r0 + (uint32_t)(j0 + j)) << S) | l) ^ fl];
#pragma unroll
            for (int j = 0; j < U; j++) {
                const V2 w = v[j0 + j];
                const double p2 = (double)w.x * w.x + (double)w.y * w.y;
                r_e += (double)(in.lut_lo + (int)x[j]) * p2;
                if ((int)x[j] == xmin) r_p += p2;
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < 32; j++) {
            const double p2 = (double)v[j].x * v[j].x + (double)v[j].y * v[j].y;
            const double e = E[(((r0 + (uint32_t)j) << S) | l) ^ fl];
            r_e += e * p2;
            if (fabs(e - in.emin) <= in.etol) r_p += p2;
        }
    }
    // fixed-order workgroup sum
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        r_e += __shfl_xor(r_e, o);
        r_p += __shfl_xor(r_p, o);
    }
    if ((t & 63) == 0) {
        red[t >> 6][0] = r_e;
        red[t >> 6][1] = r_p;
    }
    __syncthreads();
    if (t == 0) {
        a.part[2 * (uint64_t)blockIdx.x] = red[0][0] + red[1][0];
        a.part[2 * (uint64_t)blockIdx.x + 1] = red[0][1] + red[1][1];
    }
}

template <typename Real, int S>
static int launch_batch_columns(const BatchArgs& a, unsigned grid, hipStream_t st) {
    switch (a.s_n - S) {
        case 1: hipLaunchKernelGGL((k_batch_columns<Real, 256, S, 1>), dim3(grid), dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_batch_columns<Real, 256, S, 2>), dim3(grid), dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL((k_batch_columns<Real, 256, S, 3>), dim3(grid), dim3(256), 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_batch_columns<Real, 256, S, 4>), dim3(grid), dim3(256), 0, st, a); break;
        case 5: hipLaunchKernelGGL((k_batch_columns<Real, 256, S, 5>), dim3(grid), dim3(256), 0, st, a); break;
        case 6:
            if constexpr (S == 12) {
                hipLaunchKernelGGL((k_batch_columns_pair<Real, S>), dim3(grid), dim3(128), 0, st, a);
                break;
            }
            return (int)hipErrorInvalidValue;
        default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

__global__ void __launch_bounds__(256) k_batch_finish(const BatchArgs a) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s < a.f_count) batch_finish_state(a, a.f_nh, a.f_n, a.f_u0, a.f_base, a.f_part, s);
}

// Slice bits of the sliced path: complex128 states in 2^12-amplitude slices (72 KiB of
// LDS, two workgroups per CU; the column kernels then hold 2 to 6 high bits), complex64
// ones in 2^13 slices.
int batch_slice_bits(int dtype, int) { return dtype == 2 ? 12 : 13; }

int launch_batch_sliced(int dtype, const BatchArgs& a, int wide, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    const int S = batch_slice_bits(dtype, a.s_n);
    if (batch_lds_bits(dtype, wide) != 13 || a.s_n <= 13 || a.s_n > S + (S == 12 ? 6 : 5) || a.s_count < 1)
        return (int)hipErrorInvalidValue;
    const unsigned grid = (unsigned)a.s_count << (a.s_n - S);
    const unsigned fin = a.f_count > 0 ? (unsigned)((a.f_count + 255) / 256) : 0u;  // 256-thread workgroups
    if (dtype == 2)
        hipLaunchKernelGGL((k_batch_slices<double, 256, 12, 512, 2, 4>), dim3(grid + fin), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_batch_slices<float, 256, 13, 1024, 2>), dim3(grid + fin), dim3(256), 0, st, a);
    int e = (int)hipGetLastError();
    if (e) return e;
    return dtype == 2 ? launch_batch_columns<double, 12>(a, grid, st) : launch_batch_columns<float, 13>(a, grid, st);
}

int launch_batch_finish(const BatchArgs& a, void* stream) {
    if (a.f_count < 1) return 0;
    hipLaunchKernelGGL(k_batch_finish, dim3((unsigned)((a.f_count + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       a);
    return (int)hipGetLastError();
}

// Variants: complex128 2^13-amplitude LDS states, four waves (wide = 0) or eight (wide = 1);
// complex64 2^14 states with eight
// waves (wide = 1) or four (wide = 0), one workgroup per CU; complex64 2^13 states with four
// waves (wide = 2), two workgroups per CU.  Phase tables hold 1024 entries.
int batch_lds_bits(int dtype, int wide) { return dtype == 2 ? 13 : (wide == 2 ? 13 : 14); }
int batch_lut_cap(int dtype, int) { return dtype == 2 ? 512 : 1024; }  // complex128: the 2^12-slice kernel's table

int launch_batch_scan(int dtype, const BatchArgs& a, int grid, int wide, void* stream) {
    if (a.scratch_elems == 0 && ((dtype == 2 && wide == 1) || (dtype != 2 && wide == 2))) {  // LDS-resident units only
        if (dtype == 2)
            hipLaunchKernelGGL((k_batch_scan<double, 512, 13, 1024, 1, false>), dim3(grid), dim3(512), 0,
                               (hipStream_t)stream, a);
        else
            hipLaunchKernelGGL((k_batch_scan<float, 256, 13, 1024, 2, false>), dim3(grid), dim3(256), 0,
                               (hipStream_t)stream, a);
        return (int)hipGetLastError();
    }
    if (dtype == 2 && wide == 1)
        hipLaunchKernelGGL((k_batch_scan<double, 512, 13, 1024>), dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
    else if (dtype == 2)
        hipLaunchKernelGGL((k_batch_scan<double, 256, 13, 1024>), dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    else if (wide == 1)
        hipLaunchKernelGGL((k_batch_scan<float, 512, 14, 1024>), dim3(grid), dim3(512), 0, (hipStream_t)stream, a);
    else if (wide == 2)
        hipLaunchKernelGGL((k_batch_scan<float, 256, 13, 1024, 2>), dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL((k_batch_scan<float, 256, 14, 1024>), dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace svk
