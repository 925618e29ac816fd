// Device helpers shared by the kernel files: complex types, LDS swizzle, streaming
// accesses, tile geometry, wave sums and the pair butterfly.
#pragma once
#include <hip/hip_runtime.h>

#include "sv_internal.h"

namespace svk {

template <typename Real>
struct V2T;
template <>
struct V2T<double> {
    using type = double2;
};
template <>
struct V2T<float> {
    using type = float2;
};

// swizzle of a tile-local index into an LDS element index: bits >= G are folded
// into the low G bits so that 2^G consecutive lanes that differ in any G
// consecutive tile bits land in distinct 128-byte bank groups.
__device__ __forceinline__ uint32_t lds_swizzle(uint32_t u, int G) {
    uint32_t x = u >> G, f = 0;
#pragma unroll
    for (int i = 0; i < 6; i++) {
        f ^= x;
        x >>= G;
    }
    return u ^ (f & ((1u << G) - 1u));
}

// Streaming (nontemporal) accesses of one complex amplitude.
typedef double nd2 __attribute__((ext_vector_type(2)));
typedef float nf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 ld_nt(const double2* p) {
    const nd2 v = __builtin_nontemporal_load(reinterpret_cast<const nd2*>(p));
    return make_double2(v.x, v.y);
}
__device__ __forceinline__ float2 ld_nt(const float2* p) {
    const nf2 v = __builtin_nontemporal_load(reinterpret_cast<const nf2*>(p));
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ void st_nt(double2* p, double2 x) {
    nd2 v;
    v.x = x.x;
    v.y = x.y;
    __builtin_nontemporal_store(v, reinterpret_cast<nd2*>(p));
}
__device__ __forceinline__ void st_nt(float2* p, float2 x) {
    nf2 v;
    v.x = x.x;
    v.y = x.y;
    __builtin_nontemporal_store(v, reinterpret_cast<nf2*>(p));
}

// Tables that no kernel writes while it reads them (tile geometries, phase
// tables) are read through the constant address space: the compiler may then
// use scalar loads for their wave-uniform entries even after the kernel's own
// stores to the state, instead of one vector load per entry.
#define SV_CONST __attribute__((address_space(4)))
typedef const SV_CONST GeoBuf CGeoBuf;
typedef const SV_CONST GeoLayout CGeoLayout;
// entry i of a constant-space complex table (component loads: the vector type's
// operators take generic references)
__device__ __forceinline__ double2 ctab(const SV_CONST double* t, int i) {
    return make_double2(t[2 * i], t[2 * i + 1]);
}

__device__ __forceinline__ double spin_u(uint32_t u, int l) { return ((u >> l) & 1u) ? 1.0 : -1.0; }
__device__ __forceinline__ double spin_z(uint64_t z, int i) { return ((z >> i) & 1ull) ? 1.0 : -1.0; }

// Tile-local index of the thread part: thread-id bit j goes to the j-th set
// bit of the layout's (wave-uniform) thread mask.  No memory access.
template <int NTB>
__device__ __forceinline__ uint32_t thread_index_bits(uint32_t t, uint32_t tmask) {
    uint32_t u = 0, m = tmask;
#pragma unroll
    for (int j = 0; j < NTB; j++) {
        const uint32_t l = (uint32_t)__builtin_ctz(m);
        m &= m - 1u;
        u |= ((t >> j) & 1u) << l;
    }
    return u;
}

struct TileGeom {
    int c, lo, g;
    __device__ __forceinline__ bool in_tile(int i) const { return i < c || (i >= lo && i < lo + g); }
    __device__ __forceinline__ uint64_t gmap(uint32_t u) const {
        return (uint64_t)(u & ((1u << c) - 1u)) | ((uint64_t)(u >> c) << lo);
    }
    __device__ __forceinline__ uint64_t base(uint64_t w) const {
        const int nlow = lo - c;
        return ((w & ((1ull << nlow) - 1ull)) << c) | ((w >> nlow) << (lo + g));
    }
};

// Thread part of E for layout L: returns e0 = E at register index 0 and the
// register-bit fields f[k], so that E(r) = e0 + sum_{k: r_k = 1} 2 f[k] + Q[r].
// s_g holds the tile's g_l (l < T) and E_fixed (entry kTF - 1).  The couplings
// inside the tile that involve thread bits come from the layout's per-thread
// table (one coalesced load per row).
template <int R, int NTB>
__device__ __forceinline__ double thread_energy(CGeoLayout* L, CGeoBuf* geo, uint32_t t,
                                                const double* s_g, double (&f)[R]) {
    constexpr int NT = 1 << NTB;
    const uint32_t off = L->thr_off;
    const SV_CONST double* __restrict__ tab = reinterpret_cast<const SV_CONST double*>(geo) + off + t;
    double eth = s_g[kTF - 1];
    uint32_t m = L->tmask;
#pragma unroll
    for (int j = 0; j < NTB; j++) {
        const int l = __builtin_ctz(m);
        m &= m - 1u;
        const double gl = s_g[l];
        eth += ((t >> j) & 1u) ? gl : -gl;
    }
    if (off != 0) eth += tab[0];
    const uint32_t rbp = L->rbpack;
#pragma unroll
    for (int k = 0; k < R; k++) {
        double fv = s_g[(rbp >> (4 * k)) & 15u];
        if (off != 0) fv += tab[(1 + k) * NT];
        f[k] = fv;
        eth -= fv;
    }
    return eth;
}

// Value of x in lane r (the same r in every lane), as a scalar.
__device__ __forceinline__ double lane_value(double x, int r) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), r);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), r);
    return __longlong_as_double(((long long)hi << 32) | (long long)lo);
}

// Wave sum, the same in every lane: within rows of 16 by DPP moves (lane ^ 1, lane ^ 2, mirrored
// halves, mirrored row), then the four rows as scalars.  A third of the latency of six
// cross-lane reads through LDS.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return v + __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm 1 0 3 2
    v = dpp_add<0x4E>(v);   // quad_perm 2 3 0 1
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
    return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Wave-level sum of a per-lane value, added by lane 0 to this wave's row of the
// per-workgroup reduction array.
template <int NS>
__device__ __forceinline__ void wave_add(double (*s_red)[NS], int slot, double v) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6][slot] += v;
}

// (cos x, -sin x) for |x| <= kTileMaxAngle (the host sends programs with larger
// phase angles to kernels that call the library function).  Two-term reduction by pi/2 with fused
// multiply-adds (x - k hi(pi/2) is exact for |x| <= 2^16: both are multiples of
// 2^-52 and the difference is below 1) and Taylor polynomials on [-pi/4, pi/4]
// (first dropped terms: 8e-20 for the sine, 2e-18 for the cosine).
__device__ __forceinline__ double2 cis_neg(double x) {
    const double k = rint(x * 0.63661977236758134);
    const double r = fma(-k, 6.123233995736766e-17, fma(-k, 1.5707963267948966, x));
    const double z = r * r;
    double s = 1.0 / 355687428096000.0, c = 1.0 / 20922789888000.0;
    s = fma(s, z, -1.0 / 1307674368000.0);
    c = fma(c, z, -1.0 / 87178291200.0);
    s = fma(s, z, 1.0 / 6227020800.0);
    c = fma(c, z, 1.0 / 479001600.0);
    s = fma(s, z, -1.0 / 39916800.0);
    c = fma(c, z, -1.0 / 3628800.0);
    s = fma(s, z, 1.0 / 362880.0);
    c = fma(c, z, 1.0 / 40320.0);
    s = fma(s, z, -1.0 / 5040.0);
    c = fma(c, z, -1.0 / 720.0);
    s = fma(s, z, 1.0 / 120.0);
    c = fma(c, z, 1.0 / 24.0);
    s = fma(s, z, -1.0 / 6.0);
    s = fma(s * z, r, r);
    const double h = 0.5 * z, w = 1.0 - h;  // 1 - z/2 + z^2 c with the rounding error of 1 - z/2 put back
    c = w + fma(z * z, c, (1.0 - w) - h);
    const int q = (int)k;
    const double cs = (q & 1) ? s : c, sn = (q & 1) ? c : s;
    return make_double2(((q + 1) & 2) ? -cs : cs, (q & 2) ? sn : -sn);
}

__device__ __forceinline__ double2 cmul(double2 x, double2 y) {
    return make_double2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x);
}

// One pair butterfly of exp(-i beta sigma^x) without its cos(beta) factor:
// (u, v) <- (u - i t v, v - i t u), t = tan(beta).
template <typename Real>
__device__ __forceinline__ void butterfly(Real& ar, Real& ai, Real& br, Real& bi, Real t) {
    const Real nar = fma(t, bi, ar), nai = fma(-t, br, ai);
    const Real nbr = fma(t, ai, br), nbi = fma(-t, ar, bi);
    ar = nar;
    ai = nai;
    br = nbr;
    bi = nbi;
}

}  // namespace svk
