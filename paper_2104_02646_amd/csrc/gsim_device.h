// Device helpers shared by the HIP kernels of libgsim (templated on the scalar
// type): 3-vectors, scalar math overloads, global loads and stores through
// address space 1, and the ground contact model with its adjoint.
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

namespace gsim {
namespace {

// ------------------------------------------------------------------ math ---
template <typename T>
struct V3 {
    T x, y, z;
};

template <typename T> __device__ __forceinline__ V3<T> mk3(T x, T y, T z) { return V3<T>{x, y, z}; }
template <typename T> __device__ __forceinline__ V3<T> operator+(V3<T> a, V3<T> b) { return mk3(a.x + b.x, a.y + b.y, a.z + b.z); }
template <typename T> __device__ __forceinline__ V3<T> operator-(V3<T> a, V3<T> b) { return mk3(a.x - b.x, a.y - b.y, a.z - b.z); }
template <typename T> __device__ __forceinline__ V3<T> operator-(V3<T> a) { return mk3(-a.x, -a.y, -a.z); }
template <typename T> __device__ __forceinline__ V3<T> operator*(V3<T> a, T s) { return mk3(a.x * s, a.y * s, a.z * s); }
template <typename T> __device__ __forceinline__ V3<T>& operator+=(V3<T>& a, V3<T> b) { a = a + b; return a; }
template <typename T> __device__ __forceinline__ V3<T>& operator-=(V3<T>& a, V3<T> b) { a = a - b; return a; }
template <typename T> __device__ __forceinline__ T dot(V3<T> a, V3<T> b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
template <typename T> __device__ __forceinline__ V3<T> cross(V3<T> a, V3<T> b) {
    return mk3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
template <typename T> __device__ __forceinline__ V3<T> zero3() { return mk3(T(0), T(0), T(0)); }

__device__ __forceinline__ float gsqrt(float a) { return sqrtf(a); }
__device__ __forceinline__ double gsqrt(double a) { return sqrt(a); }
__device__ __forceinline__ float gsin(float a) { return sinf(a); }
__device__ __forceinline__ double gsin(double a) { return sin(a); }
__device__ __forceinline__ float gcos(float a) { return cosf(a); }
__device__ __forceinline__ double gcos(double a) { return cos(a); }
__device__ __forceinline__ float gabs(float a) { return fabsf(a); }
__device__ __forceinline__ double gabs(double a) { return fabs(a); }
__device__ __forceinline__ float gatan2(float y, float x) { return atan2f(y, x); }
__device__ __forceinline__ double gatan2(double y, double x) { return atan2(y, x); }

__device__ __forceinline__ float gfma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double gfma(double a, double b, double c) { return fma(a, b, c); }
// Vector arithmetic with every rounding written out (contraction off, fused multiply-adds
// explicit): the tets, the contact and the particle update use it, so that each kernel
// that evaluates them, however its loads and branches are arranged, gets the same bits.
template <typename T>
__device__ __forceinline__ V3<T> fma3(V3<T> a, T s, V3<T> c) {
    return mk3(gfma(a.x, s, c.x), gfma(a.y, s, c.y), gfma(a.z, s, c.z));
}
template <typename T>
__device__ __forceinline__ V3<T> mul3(V3<T> a, T s) {
#pragma clang fp contract(off)
    return mk3(a.x * s, a.y * s, a.z * s);
}
template <typename T>
__device__ __forceinline__ V3<T> add3(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
    return mk3(a.x + b.x, a.y + b.y, a.z + b.z);
}
template <typename T>
__device__ __forceinline__ V3<T> sub3(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
    return mk3(a.x - b.x, a.y - b.y, a.z - b.z);
}
// a s + b t + c r, the first product fused into the rounded second, then the third
template <typename T>
__device__ __forceinline__ V3<T> lin3(V3<T> a, T s, V3<T> b, T t, V3<T> c, T r) {
    return fma3(c, r, fma3(a, s, mul3(b, t)));
}
template <typename T>
__device__ __forceinline__ T fdot(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
    return gfma(a.z, b.z, gfma(a.x, b.x, a.y * b.y));
}
template <typename T>
__device__ __forceinline__ V3<T> fcross(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
    return mk3(gfma(a.y, b.z, -(a.z * b.y)), gfma(a.z, b.x, -(a.x * b.z)), gfma(a.x, b.y, -(a.y * b.x)));
}

// --------------------------------------------------------- lane network ---
// Lane exchanges in the vector units, by 32-bit halves for doubles.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Exchanges lanes 32-63 of a with lanes 0-31 of b (HALF), or in each half its upper 16 lanes
// of a with its lower 16 of b.
template <bool HALF>
__device__ __forceinline__ void swap_rows(uint32_t& a, uint32_t& b) {
    if constexpr (HALF) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
// a + (a of the other half-wave) in lanes 0-31 and the same of b in lanes 32-63 (HALF; else
// by the two 16-lane rows of each half).
template <bool HALF>
__device__ __forceinline__ float swap_add(float a, float b) {
    uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    swap_rows<HALF>(x, y);
    return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
}
template <bool HALF>
__device__ __forceinline__ double swap_add(double a, double b) {
    const uint64_t p = __builtin_bit_cast(uint64_t, a), q = __builtin_bit_cast(uint64_t, b);
    uint32_t xl = (uint32_t)p, xh = (uint32_t)(p >> 32), yl = (uint32_t)q, yh = (uint32_t)(q >> 32);
    swap_rows<HALF>(xl, yl);
    swap_rows<HALF>(xh, yh);
    return __builtin_bit_cast(double, ((uint64_t)xh << 32) | xl) + __builtin_bit_cast(double, ((uint64_t)yh << 32) | yl);
}
__device__ __forceinline__ float lane_of(float x, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_of(double x, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sums of N values over the wavefront's 64 lanes; every lane gets every total.  All
// lanes must be active.  Four values share a register after the half-wave and the row
// exchange (value 4k in row 0, 4k + 2 in row 1, 4k + 1 in row 2, 4k + 3 in row 3); the
// sum over a row's 16 lanes is a fixed tree (lanes 8, 4, 2, 1 apart).
template <typename T, int N>
__device__ __forceinline__ void wave_sum(T v[N]) {
    constexpr int H = (N + 1) / 2, Q = (N + 3) / 4;
    T h[2 * Q];
#pragma unroll
    for (int i = 0; i < H; ++i) h[i] = swap_add<true>(v[2 * i], 2 * i + 1 < N ? v[2 * i + 1] : T(0));
    if constexpr (H < 2 * Q) h[2 * Q - 1] = T(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T r = swap_add<false>(h[2 * i], h[2 * i + 1]);
        r += dpp<0x128>(r);  // row_ror:8
        r += dpp<0x124>(r);  // row_ror:4 (lanes 8 apart are equal by now)
        r += dpp<0x4e>(r);   // quad_perm [2, 3, 0, 1]
        r += dpp<0xb1>(r);   // quad_perm [1, 0, 3, 2]
        const int row[4] = {0, 32, 16, 48};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (4 * i + k < N) v[4 * i + k] = lane_of(r, row[k]);
    }
}

// Device-memory accesses through address space 1: pointers read out of the
// launch tables are generic, and generic (flat) loads both count against the
// LDS wait counter and may alias LDS, which would order every record load
// before the next LDS barrier.  Global loads do neither.
template <typename T> __device__ __forceinline__ T gld(const T* p, int64_t i) {
    return ((const __attribute__((address_space(1))) T*)p)[i];
}
template <typename T> __device__ __forceinline__ void gst(T* p, int64_t i, T v) {
    ((__attribute__((address_space(1))) T*)p)[i] = v;
}
// Accesses at a uniform base (the same in every lane: a tile's first item) plus a
// lane's 32-bit byte offset: the base stays in scalar registers and one offset register
// serves every array of the tile, so no address arithmetic runs on the vector units.
template <typename T> __device__ __forceinline__ T gldo(const T* base, uint32_t off) {
    return *(const __attribute__((address_space(1))) T*)((const __attribute__((address_space(1))) char*)base + off);
}
template <typename T> __device__ __forceinline__ void gsto(T* base, uint32_t off, T v) {
    *(__attribute__((address_space(1))) T*)((__attribute__((address_space(1))) char*)base + off) = v;
}
template <typename T> __device__ __forceinline__ V3<T> ld3(const T* __restrict__ p, int64_t n, int64_t i) {
    return mk3(gld(p, i), gld(p, n + i), gld(p, 2 * n + i));
}
template <typename T> __device__ __forceinline__ void st3(T* __restrict__ p, int64_t n, int64_t i, V3<T> a) {
    gst(p, i, a.x);
    gst(p, n + i, a.y);
    gst(p, 2 * n + i, a.z);
}
template <typename T> __device__ __forceinline__ V3<T> ld3o(const T* p, int64_t n, uint32_t off) {
    return mk3(gldo(p, off), gldo(p + n, off), gldo(p + 2 * n, off));
}
template <typename T> __device__ __forceinline__ void st3o(T* p, int64_t n, uint32_t off, V3<T> a) {
    gsto(p, off, a.x);
    gsto(p + n, off, a.y);
    gsto(p + 2 * n, off, a.z);
}

// ------------------------------------------------------------- contact ---
// gap = n.x - d; C = -gap when gap < 0; lambda_n = k_e C + k_d Cdot, Cdot = -n.v;
// f_n = lambda_n n; u_t = v - (n.v) n; stick if k_f |u_t| <= mu_f |lambda_n|:
// f_f = -k_f u_t; otherwise f_f = -mu_f |lambda_n| u_t / |u_t|.
// The deformable kernels pass the gap itself (the rest gap of the particle plus
// n.u for its displacement u, so that no absolute coordinate is rounded); the
// rigid kernels pass a world point through the overloads below.
template <typename T>
__device__ __forceinline__ V3<T> contact_force_gap(T gap, V3<T> v, const T pl[4], const T c[4]) {
#pragma clang fp contract(off)
    const V3<T> n = mk3(pl[0], pl[1], pl[2]);
    if (!(gap < T(0))) return zero3<T>();
    const T C = -gap;
    const T vn = fdot(n, v);
    const T lam = gfma(c[0], C, -(c[1] * vn));
    const V3<T> ut = fma3(n, -vn, v);
    const T s = gsqrt(fdot(ut, ut));
    const T lim = c[3] * (lam < T(0) ? -lam : lam);
    V3<T> ff;
    if (c[2] * s <= lim) ff = mul3(ut, -c[2]);
    else ff = mul3(ut, -lim / s);
    return fma3(n, lam, ff);
}

// Adjoint of contact_force_gap for the force adjoint fb: adds to xb (through
// d gap / dx = n), vb and the contact-parameter gradients gc (k_e, k_d, k_f,
// mu_f); returns the force.
template <typename T>
__device__ __forceinline__ V3<T> contact_adjoint_gap(T gap, V3<T> v, const T pl[4], const T c[4], V3<T> fb, V3<T>& xb,
                                                     V3<T>& vb, T gc[4]) {
#pragma clang fp contract(off)
    const V3<T> n = mk3(pl[0], pl[1], pl[2]);
    if (!(gap < T(0))) return zero3<T>();
    const T C = -gap;
    const T vn = fdot(n, v);
    const T lam = gfma(c[0], C, -(c[1] * vn));
    const V3<T> ut = fma3(n, -vn, v);
    const T s = gsqrt(fdot(ut, ut));
    const T sg = lam < T(0) ? T(-1) : T(1);
    const T lim = c[3] * lam * sg;
    T lamb = fdot(fb, n);
    V3<T> utb;
    V3<T> ff;
    if (c[2] * s <= lim) {
        ff = mul3(ut, -c[2]);
        utb = mul3(fb, -c[2]);
        gc[2] -= fdot(ut, fb);
    } else {
        const T is = T(1) / s;
        const V3<T> th = mul3(ut, is);
        ff = mul3(th, -lim);
        const T limb = -fdot(th, fb);
        const V3<T> thb = mul3(fb, -lim);
        utb = mul3(fma3(th, -fdot(th, thb), thb), is);
        gc[3] = gfma(lam * sg, limb, gc[3]);
        lamb = gfma(c[3] * sg, limb, lamb);
    }
    vb = add3(vb, fma3(n, -fdot(n, utb), utb));
    gc[0] = gfma(C, lamb, gc[0]);
    gc[1] = gfma(-vn, lamb, gc[1]);
    xb = fma3(n, -(c[0] * lamb), xb);
    vb = fma3(n, -(c[1] * lamb), vb);
    return fma3(n, lam, ff);
}

template <typename T>
__device__ __forceinline__ V3<T> contact_force(V3<T> x, V3<T> v, const T pl[4], const T c[4]) {
    return contact_force_gap(dot(mk3(pl[0], pl[1], pl[2]), x) - pl[3], v, pl, c);
}
template <typename T>
__device__ __forceinline__ V3<T> contact_adjoint(V3<T> x, V3<T> v, const T pl[4], const T c[4], V3<T> fb, V3<T>& xb,
                                                 V3<T>& vb, T gc[4]) {
    return contact_adjoint_gap(dot(mk3(pl[0], pl[1], pl[2]), x) - pl[3], v, pl, c, fb, xb, vb, gc);
}

}  // namespace
}  // namespace gsim
