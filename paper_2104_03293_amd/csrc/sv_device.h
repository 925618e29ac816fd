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

// Wave-level sum of a per-lane value (fixed butterfly order), added by lane 0
// to this wave's row of the per-workgroup reduction array.
template <int NS>
__device__ __forceinline__ void wave_add(double (*s_red)[NS], int slot, double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6][slot] += v;
}

// Value of x in lane r (the same r in every lane), as a scalar.
__device__ __forceinline__ double lane_value(double x, int r) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), r);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), r);
    return __longlong_as_double(((long long)hi << 32) | (long long)lo);
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
