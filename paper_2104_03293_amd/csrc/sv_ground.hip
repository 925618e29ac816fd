// Ground states: of small states from their energy table (k_ground_table), of
// instances on an energy grid by enumeration over an independent set: k spins without couplings among each other are, given the
// other r = n - k, each at its own best value, so
//   min_z E(z) = min_x ( E_rest(x) - sum_i |F_i(x)| ),   F_i = h_i + sum_j J_ij s_j(x),
// over the 2^r settings x of the rest; a setting at the minimum stands for
// 2^{number of F_i = 0} states, and its smallest index takes bit 0 wherever
// F_i >= 0.  Energies are integers (in units of 1/q), so the minimum, the number
// of states at it and the first of them are those of the full enumeration.
//
// Bound by integer arithmetic: 5 operations per term and setting, terms read
// from LDS once per four settings.  n = 31, 62 couplings (r = 19): 15 us, against
// 2.27 ms for the two passes of the tile enumeration over all states.
#include <hip/hip_runtime.h>

#include "sv_device.h"
#include "sv_internal.h"

namespace svk {

// sum of c (-1)^{parity(x & mask)} over terms [t0, t1) for the settings x .. x + 3
__device__ __forceinline__ void add_terms(const int2* s_t, int t0, int t1, uint32_t x, int (&e)[4]) {
    for (int k = t0; k < t1; k++) {
        const uint32_t mask = (uint32_t)s_t[k].x;
        const int c = s_t[k].y;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int p = -(int)(__popc((x + j) & mask) & 1u);  // 0 or -1
            e[j] += (c ^ p) - p;
        }
    }
}

// Combined (energy, count, first) of one workgroup in thread 0.
struct GroundBest {
    int e;
    unsigned long long cnt, first;
};
__device__ __forceinline__ void ground_merge(GroundBest& b, const GroundBest& o) {
    if (o.e < b.e) {
        b = o;
    } else if (o.e == b.e) {
        b.cnt += o.cnt;
        b.first = o.first < b.first ? o.first : b.first;
    }
}

template <int NW>
__device__ void ground_block(GroundBest& b, GroundBest* s_b) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        GroundBest o;
        o.e = __shfl_xor(b.e, off);
        o.cnt = __shfl_xor(b.cnt, off);
        o.first = __shfl_xor(b.first, off);
        ground_merge(b, o);
    }
    if ((threadIdx.x & 63) == 0) s_b[threadIdx.x >> 6] = b;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < NW; w++) ground_merge(b, s_b[w]);
}

__global__ void __launch_bounds__(256) k_ground_sets(const GroundSetArgs a) {
    __shared__ int2 s_t[kMaxGroundTerms];
    __shared__ int s_min[4];
    __shared__ GroundBest s_b[4];
    const int t = threadIdx.x;
    for (int k = t; k < a.nterms; k += 256) s_t[k] = a.terms[k];
    __syncthreads();
    GroundBest best{0x7fffffff, 0ull, ~0ull};
    const uint64_t nset = 1ull << a.r;
    for (uint64_t x0 = (uint64_t)blockIdx.x * 1024; x0 < nset; x0 += (uint64_t)gridDim.x * 1024) {
        const uint32_t x = (uint32_t)(x0 + 4 * t);
        const bool in = x0 + 4 * t < nset;
        int e[4] = {a.e0, a.e0, a.e0, a.e0};
        add_terms(s_t, 0, a.first[0], x, e);
        int f[4];
        for (int i = 0; i < a.k; i++) {
#pragma unroll
            for (int j = 0; j < 4; j++) f[j] = a.h[i];
            add_terms(s_t, a.first[i], a.first[i + 1], x, f);
#pragma unroll
            for (int j = 0; j < 4; j++) e[j] -= abs(f[j]);
        }
        int m = in ? min(min(e[0], e[1]), min(e[2], e[3])) : 0x7fffffff;
        // the step's minimum; only settings at it (and not above the best so far) are looked at again
        int lo = m;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) lo = min(lo, __shfl_xor(lo, off));
        if ((t & 63) == 0) s_min[t >> 6] = lo;
        __syncthreads();
        lo = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
        __syncthreads();
        if (lo > best.e) continue;
        if (lo < best.e) best = GroundBest{lo, 0ull, ~0ull};  // every thread keeps the same energy
        if (m != lo) continue;
        for (int j = 0; j < 4; j++) {
            if (e[j] != lo) continue;
            // count and smallest index of setting x + j
            unsigned long long z = 0ull;
            const uint32_t xj = x + (uint32_t)j;
            for (int b = 0; b < a.r; b++) z |= (unsigned long long)((xj >> b) & 1u) << a.rest[b];
            int zeros = 0;
            for (int i = 0; i < a.k; i++) {
                int fi = a.h[i];
                for (int k = a.first[i]; k < a.first[i + 1]; k++) {
                    const int p = -(int)(__popc(xj & (uint32_t)s_t[k].x) & 1u);
                    fi += (s_t[k].y ^ p) - p;
                }
                zeros += fi == 0;
                if (fi < 0) z |= 1ull << a.spin[i];
            }
            best.cnt += 1ull << zeros;
            best.first = z < best.first ? z : best.first;
        }
    }
    ground_block<4>(best, s_b);
    if (t == 0) {
        a.part_e[blockIdx.x] = best.e;
        a.part_c[2 * blockIdx.x] = best.cnt;
        a.part_c[2 * blockIdx.x + 1] = best.first;
    }
}

__global__ void __launch_bounds__(256) k_ground_sets_finish(const GroundSetArgs a, int nblocks) {
    __shared__ GroundBest s_b[4];
    GroundBest best{0x7fffffff, 0ull, ~0ull};
    for (int i = threadIdx.x; i < nblocks; i += 256)
        ground_merge(best, GroundBest{a.part_e[i], a.part_c[2 * i], a.part_c[2 * i + 1]});
    ground_block<4>(best, s_b);
    if (threadIdx.x == 0) {
        a.out[0] = (unsigned long long)(long long)best.e;
        a.out[1] = best.cnt;
        a.out[2] = best.first;
    }
}

// Small states: minimum, number of states at it (within tol) and the first of them from the energy
// table that the small tiles read, one workgroup.  Bound by its latency (16 loads in series with two
// reductions, in the shadow of the call's allocations and copy).
__global__ void __launch_bounds__(1024) k_ground_table(const double* __restrict__ E, uint32_t N, double tol, double* out) {
    __shared__ double s_m[16];
    __shared__ uint32_t s_c[16], s_f[16];
    const uint32_t t = threadIdx.x;
    double m = INFINITY;
    for (uint32_t z = t; z < N; z += 1024) m = fmin(m, E[z]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmin(m, __shfl_xor(m, off));
    if ((t & 63) == 0) s_m[t >> 6] = m;
    __syncthreads();
    for (int w = 0; w < 16; w++) m = fmin(m, s_m[w]);
    uint32_t cnt = 0, first = 0xffffffffu;
    for (uint32_t z = t; z < N; z += 1024)
        if (fabs(E[z] - m) <= tol) {
            cnt++;
            first = min(first, z);
        }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        cnt += __shfl_xor(cnt, off);
        first = min(first, (uint32_t)__shfl_xor(first, off));
    }
    if ((t & 63) == 0) {
        s_c[t >> 6] = cnt;
        s_f[t >> 6] = first;
    }
    __syncthreads();
    if (t != 0) return;
    for (int w = 1; w < 16; w++) {
        cnt += s_c[w];
        first = min(first, s_f[w]);
    }
    out[0] = m;
    out[1] = (double)cnt;
    out[2] = (double)first;
}

int launch_ground_table(const double* E, int n, double tol, double* out, void* stream) {
    hipLaunchKernelGGL(k_ground_table, dim3(1), dim3(1024), 0, (hipStream_t)stream, E, 1u << n, tol, out);
    return (int)hipGetLastError();
}

int launch_ground_sets(const GroundSetArgs& a, int nblocks, void* stream) {
    hipLaunchKernelGGL(k_ground_sets, dim3((unsigned)nblocks), dim3(256), 0, (hipStream_t)stream, a);
    hipLaunchKernelGGL(k_ground_sets_finish, dim3(1), dim3(256), 0, (hipStream_t)stream, a, nblocks);
    return (int)hipGetLastError();
}

}  // namespace svk
