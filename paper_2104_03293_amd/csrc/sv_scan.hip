// Landscape scan of p = 1 circuits (Sec. III.C.1, Fig. 5) without evolving a
// state per grid point, for instances whose energies lie on a grid Z / q.
//
// Energy.  With s = sin 2 beta, c = cos 2 beta and the phase state
// |phi> = exp(-i gamma H_C) |+>, rotating sigma^z by the mixer gives
//   <H_C>(gamma, beta) = s A + c s B + s^2 C,
//   A = sum_i h_i <W_i>,  B = sum_ij J_ij <W_i Z_j + Z_i W_j>,  C = sum_ij J_ij <W_i W_j>,
// W = -i Z X, and every expectation in |phi> is an average over independent
// neighbour spins, i.e. a product of cosines:
//   <W_i>     = sin(2 g h_i) prod_k cos(2 g J_ik),
//   <W_i Z_j> = sin(2 g J_ij) cos(2 g h_i) prod_{k != j} cos(2 g J_ik),
//   <W_i W_j> = (cos(2 g (h_i - h_j)) prod_k cos(2 g (J_ik - J_jk))
//                - cos(2 g (h_i + h_j)) prod_k cos(2 g (J_ik + J_jk))) / 2,  k != i, j.
// So a gamma costs O(n m) and a grid point O(1).
//
// Ground-state probability.  The amplitude of z depends on phi only through its
// sums over the spheres of Hamming distance d around z:
//   <z| exp(-i beta H_D) |phi> = sum_d cos^{n-d}(beta) (-i sin beta)^d A_d(gamma),
//   A_d = 2^{-n/2} sum_e N_z(d, e) exp(-i gamma e),
// N_z(d, e) = number of states at distance d from z with energy e: one pass over
// 2^n table indices per ground state, whatever the size of the grid.
//
// The direct scan (k_batch_* in sv_kernels.hip) mixes 2^n amplitudes for every
// grid point; it remains for instances off the grid, and for those with more
// ground states than grid points, where the histograms would cost more.
// 128 instances of 10 to 18 qubits on a 32 x 32 grid: 29.7 -> 0.53 ms a call (0.9-1.1 ms where every
// call brings new instances), of which 0.17 ms are kernels (bound by the index pass and the LDS atomics
// of the histograms) and the rest copies of the results, allocations and the two waits for the host.
#include <hip/hip_runtime.h>

#include "sv_device.h"
#include "sv_internal.h"

namespace svk {

constexpr int kScanPer = 8;  // basis states per thread of k_scan_index

// Table index q E(z) - lo of every basis state, and the smallest and largest
// index of each instance.  The terms are staged in LDS (a scalar load per term
// would put a memory round trip into every step of the loop); a thread's eight
// states share all terms but those of bits 0..2.
__global__ void __launch_bounds__(256) k_scan_index(const ScanArgs a) {
    __shared__ int hs[kScanMaxN];
    __shared__ int4 cs[kScanMaxN * (kScanMaxN - 1) / 2];
    const uint32_t i = blockIdx.x / a.bpi, b = blockIdx.x % a.bpi;
    const ScanInst in = a.inst[i];
    const uint32_t N = 1u << in.n;
    if (b * 256 * kScanPer >= N) return;
    const int32_t* cq = a.cq + 3 * (uint64_t)in.coff;
    if ((int)threadIdx.x < in.n) hs[threadIdx.x] = a.hq[in.hoff + threadIdx.x];
    for (int k = threadIdx.x; k < in.m; k += 256)
        cs[k] = make_int4(min(cq[3 * k], cq[3 * k + 1]), max(cq[3 * k], cq[3 * k + 1]), cq[3 * k + 2], 0);
    __syncthreads();
    int lo = 0x7fffffff, hi = -1;
    uint16_t* X = a.x + in.xoff;
    for (uint32_t z0 = (b * 256 + threadIdx.x) * kScanPer; z0 < N; z0 += a.bpi * 256 * kScanPer) {
        int e0 = -in.lo, f[3] = {0, 0, 0}, c01 = 0, c02 = 0, c12 = 0;
        for (int k = 0; k < in.n; k++) {
            const int h = hs[k];
            if (k == 0) f[0] += h;
            else if (k == 1) f[1] += h;
            else if (k == 2) f[2] += h;
            else e0 += ((z0 >> k) & 1u) ? h : -h;
        }
        for (int k = 0; k < in.m; k++) {
            const int u = cs[k].x, v = cs[k].y, J = cs[k].z;
            if (u > 2) {
                e0 += (((z0 >> u) ^ (z0 >> v)) & 1u) ? -J : J;
            } else if (v > 2) {
                const int x = ((z0 >> v) & 1u) ? J : -J;
                if (u == 0) f[0] += x;
                else if (u == 1) f[1] += x;
                else f[2] += x;
            } else if (v == 1) {
                c01 += J;
            } else if (u == 0) {
                c02 += J;
            } else {
                c12 += J;
            }
        }
        union {
            uint16_t h[kScanPer];
            uint4 v;
        } o;
#pragma unroll
        for (int j = 0; j < kScanPer; j++) {
            const int s0 = (j & 1) ? 1 : -1, s1 = (j & 2) ? 1 : -1, s2 = (j & 4) ? 1 : -1;
            const int e = e0 + s0 * f[0] + s1 * f[1] + s2 * f[2] + s0 * s1 * c01 + s0 * s2 * c02 + s1 * s2 * c12;
            o.h[j] = (uint16_t)e;
            if (z0 + j >= N) continue;
            lo = min(lo, e);
            hi = max(hi, e);
        }
        *reinterpret_cast<uint4*>(X + z0) = o.v;  // every instance's table holds a multiple of eight entries
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
    }
    if ((threadIdx.x & 63) == 0 && hi >= 0) {
        atomicMin(&a.stat[3 * i], lo);
        atomicMax(&a.stat[3 * i + 1], hi);
    }
}

// Ground states of each instance in ascending order (the first zcap of them)
// and their number, one workgroup per instance: 8192 indices a step, the step's
// matches placed by a prefix sum where there are any.
__global__ void __launch_bounds__(1024) k_scan_ground(const ScanArgs a) {
    __shared__ int s_wave[16];
    const int i = blockIdx.x, t = threadIdx.x;
    const ScanInst in = a.inst[i];
    const uint32_t N = 1u << in.n;
    const uint16_t* X = a.x + in.xoff;
    const int xmin = a.stat[3 * i];
    int total = 0;
    for (uint32_t b = 0; b < N; b += 8192u) {  // the same trips for every thread
        const uint32_t z0 = b + (uint32_t)t * 8u;
        uint32_t m = 0u;
        if (z0 < N) {
            const uint4 w = *reinterpret_cast<const uint4*>(X + z0);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (z0 + j < N && (int)((ws[j >> 1] >> (16 * (j & 1))) & 0xffffu) == xmin) m |= 1u << j;
        }
        if (!__syncthreads_or((int)m)) continue;
        const int cnt = __popc(m);
        int inc = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o);
            if ((t & 63) >= o) inc += y;
        }
        if ((t & 63) == 63) s_wave[t >> 6] = inc;
        __syncthreads();
        int at = total + inc - cnt;
        for (int w = 0; w < 16; w++) {
            if (w < (t >> 6)) at += s_wave[w];
            total += s_wave[w];
        }
        for (int j = 0; j < 8; j++)
            if ((m >> j) & 1u) {
                if (at < in.zcap) a.z[in.zoff + at] = z0 + j;
                at++;
            }
        __syncthreads();  // s_wave is free again
    }
    if (t == 0) a.stat[3 * i + 2] = total;
}

// A, B, C of the energy for every gamma, one wave per (instance, gamma).
__global__ void __launch_bounds__(256) k_scan_coef(const ScanArgs a) {
    __shared__ int Jm[kScanMaxN * kScanMaxN];
    __shared__ int hs[kScanMaxN];
    __shared__ double tc[4][64], ts[4][64];  // cos, sin(2 gamma k / q), one row per wave
    const uint32_t i = blockIdx.x / a.gpb, gb = blockIdx.x % a.gpb;
    const ScanInst in = a.inst[i];
    const int n = in.n, t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int32_t* hq = a.hq + in.hoff;
    const int32_t* cq = a.cq + 3 * (uint64_t)in.coff;
    const double qi = 1.0 / in.q;
    const int64_t gi = (int64_t)gb * 4 + w;
    const double g2 = gi < a.ng ? 2.0 * a.gammas[gi] : 0.0;
    sincos(g2 * (lane * qi), &ts[w][lane], &tc[w][lane]);
    for (int k = t; k < n * n; k += 256) Jm[k] = 0;
    if (t < n) hs[t] = hq[t];
    __syncthreads();
    for (int k = t; k < in.m; k += 256) {
        Jm[cq[3 * k] * n + cq[3 * k + 1]] = cq[3 * k + 2];
        Jm[cq[3 * k + 1] * n + cq[3 * k]] = cq[3 * k + 2];
    }
    __syncthreads();
    if (gi >= a.ng) return;
    // cos and sin of 2 gamma k / q: from the table for the small multiples
    auto ck = [&](int k) {
        k = abs(k);
        return k < 64 ? tc[w][k] : cos(g2 * (k * qi));
    };
    auto sk = [&](int k) {
        const int m = abs(k);
        const double x = m < 64 ? ts[w][m] : sin(g2 * (m * qi));
        return k < 0 ? -x : x;
    };
    double A = 0.0, B = 0.0, C = 0.0;
    for (int u = lane; u < n; u += 64) {
        if (hs[u] == 0) continue;
        double p = sk(hs[u]);
        for (int k = 0; k < n; k++)
            if (Jm[u * n + k] != 0) p *= ck(Jm[u * n + k]);
        A = fma(hs[u] * qi, p, A);
    }
    for (int e = lane; e < in.m; e += 64) {
        const int u = cq[3 * e], v = cq[3 * e + 1], J = cq[3 * e + 2];
        if (J == 0) continue;
        double pu = ck(hs[u]), pv = ck(hs[v]), pm = ck(hs[u] - hs[v]), pp = ck(hs[u] + hs[v]);
        for (int k = 0; k < n; k++) {
            if (k == u || k == v) continue;
            const int x = Jm[u * n + k], y = Jm[v * n + k];
            if (x != 0) pu *= ck(x);
            if (y != 0) pv *= ck(y);
            if (x != 0 || y != 0) {
                pm *= ck(x - y);
                pp *= ck(x + y);
            }
        }
        B = fma(J * qi, sk(J) * (pu + pv), B);
        C = fma(0.5 * (J * qi), pm - pp, C);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        A += __shfl_xor(A, o);
        B += __shfl_xor(B, o);
        C += __shfl_xor(C, o);
    }
    if (lane == 0) {
        double* out = a.coef + ((uint64_t)i * a.ng + gi) * 3;
        out[0] = A;
        out[1] = B;
        out[2] = C;
    }
}

// Sphere sums A_d(gamma) of one ground state per workgroup: the histogram
// N_z(d, e) in LDS (integer counts: the order of the atomics does not matter),
// then one (gamma, d) pair per thread, a polynomial in exp(-i gamma / q)
// evaluated from the middle of the energy range outwards.
__global__ void __launch_bounds__(512) k_scan_amps(const ScanArgs a) {
    extern __shared__ uint32_t hist[];
    const int t = threadIdx.x;
    const int64_t u = a.u0 + blockIdx.x;
    const int i = a.uinst[u];
    const ScanInst in = a.inst[i];
    const int n = in.n;
    const uint32_t N = 1u << n;
    const int xlo = a.stat[3 * i], ne = a.stat[3 * i + 1] - xlo + 1;
    const uint32_t z = a.z[in.zoff + (u - a.uoff[i])];
    for (int k = t; k < (n + 1) * ne; k += 512) hist[k] = 0u;
    __syncthreads();
    const uint16_t* X = a.x + in.xoff;
    if (N >= 8) {
#pragma unroll 2
        for (uint32_t b = (uint32_t)t * 8u; b < N; b += 512u * 8u) {
            const uint4 w = *reinterpret_cast<const uint4*>(X + b);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int e = (int)((ws[j >> 1] >> (16 * (j & 1))) & 0xffffu) - xlo;
                atomicAdd(&hist[__popc((b + j) ^ z) * ne + e], 1u);
            }
        }
    } else if ((uint32_t)t < N) {
        atomicAdd(&hist[__popc((uint32_t)t ^ z) * ne + ((int)X[t] - xlo)], 1u);
    }
    __syncthreads();
    const double amp0 = exp2(-0.5 * n);
    double2* out = a.amps + (uint64_t)blockIdx.x * a.gc * (kScanMaxN + 1);
    const int mid = ne >> 1;
    for (int k = t; k < a.gc * (n + 1); k += 512) {
        const int gl = k / (n + 1), d = k % (n + 1);
        const double gam = a.gammas[a.g0 + gl];
        const uint32_t* h = hist + d * ne;
        double sn, cs;
        sincos(gam / in.q, &sn, &cs);
        // w = exp(-i gamma / q): entries above mid in powers of w, those below in powers of conj(w)
        double pr = 0.0, pi = 0.0, mr = 0.0, mi = 0.0;
        for (int e = ne - 1; e > mid; e--) {
            const double x = pr + (double)h[e];
            pr = fma(x, cs, pi * sn);
            pi = fma(pi, cs, -x * sn);
        }
        for (int e = 0; e < mid; e++) {
            const double x = mr + (double)h[e];
            mr = fma(x, cs, -mi * sn);
            mi = fma(mi, cs, x * sn);
        }
        const double sr = (pr + mr) + (double)h[mid], si = pi + mi;
        // times exp(-i gamma E_mid) 2^{-n/2}
        sincos(gam * ((double)(in.lo + xlo + mid) / in.q), &sn, &cs);
        out[(uint64_t)gl * (kScanMaxN + 1) + d] =
            make_double2(amp0 * fma(sr, cs, si * sn), amp0 * fma(si, cs, -sr * sn));
    }
}

// <H_C> and P_gs of the grid points of one (instance, gamma) per workgroup, from
// the coefficients and the sphere sums of the units of this launch: eight threads
// per beta take every eighth ground state (the few instances with many of them
// would otherwise run the whole kernel's length in one thread).
__global__ void __launch_bounds__(256) k_scan_out(const ScanArgs a) {
    const uint32_t bl = blockIdx.x / (uint32_t)a.gc;
    const int gl = (int)(blockIdx.x % (uint32_t)a.gc);
    const int i = a.oinst[a.o0 + bl];
    const ScanInst in = a.inst[i];
    const int64_t gi = a.g0 + gl;
    const int64_t uo = a.uoff[i];
    const int64_t ua = max(uo, a.u0), ub = min(uo + (int64_t)a.stat[3 * i + 2], a.u0 + a.ucount);
    const int n = in.n, zl = threadIdx.x & 7;
    const double* q = a.coef + ((uint64_t)i * a.ng + gi) * 3;
    for (int b0 = 0; b0 < a.nb; b0 += 32) {
        const int b = b0 + (threadIdx.x >> 3);
        const double beta = a.betas[min(b, a.nb - 1)];
        double sn, cs;
        sincos(beta, &sn, &cs);
        // sum_d cos^{n-d} (-i sin)^d A_d: the larger of the two factored out, Horner in the ratio
        const bool fc = fabs(cs) >= fabs(sn);
        const double r = fc ? -sn / cs : cs / sn;
        double P = 0.0;
        for (int64_t u = ua + zl; u < ub; u += 8) {
            const double2* A = a.amps + ((uint64_t)(u - a.u0) * a.gc + gl) * (kScanMaxN + 1);
            double x = 0.0, y = 0.0;
#pragma unroll 4
            for (int k = 0; k <= n; k++) {  // times i r, plus the next: downwards from A_n, or upwards from A_0
                const double2 v = A[fc ? n - k : k];
                const double xr = fma(-y, r, v.x);
                y = fma(x, r, v.y);
                x = xr;
            }
            P += fma(x, x, y * y);
        }
#pragma unroll
        for (int o = 4; o >= 1; o >>= 1) P += __shfl_xor(P, o);
        if (zl != 0 || b >= a.nb) continue;
        double sc = 1.0;
        for (int k = 0; k < n; k++) sc *= fc ? cs * cs : sn * sn;
        P *= sc;
        const uint64_t o = ((uint64_t)in.out * a.ng + gi) * a.nb + b;
        if (ua > uo) {
            a.out_p[o] += P;
        } else {
            a.out_p[o] = P;
            const double s2 = 2.0 * sn * cs, c2 = fma(cs, cs, -sn * sn);
            a.out_e[o] = s2 * (q[0] + c2 * q[1] + s2 * q[2]);
        }
    }
}

int launch_scan_tables(const ScanArgs& a, int ninst, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_scan_index, dim3((unsigned)ninst * a.bpi), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_scan_ground, dim3((unsigned)ninst), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(k_scan_coef, dim3((unsigned)ninst * a.gpb), dim3(256), 0, st, a);
    return (int)hipGetLastError();
}

int launch_scan_points(const ScanArgs& a, int nout, size_t lds, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_scan_amps, dim3((unsigned)a.ucount), dim3(512), lds, st, a);
    hipLaunchKernelGGL(k_scan_out, dim3((unsigned)nout * (unsigned)a.gc), dim3(256), 0, st, a);
    return (int)hipGetLastError();
}

}  // namespace svk
