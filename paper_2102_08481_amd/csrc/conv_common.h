// Element, fragment and matrix-instruction helpers shared by the layer kernels (conv_igemm.hip, conv_large.h).
#pragma once
#include <type_traits>

#include "thia_internal.h"

namespace thia {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;


template <typename T>
__device__ inline void mma_step(f32x16_t& acc, const u32x4_t& a, const u32x4_t& b);

template <>
__device__ inline void mma_step<bf16_t>(f32x16_t& acc, const u32x4_t& a, const u32x4_t& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
}
template <>
__device__ inline void mma_step<float>(f32x16_t& acc, const u32x4_t& a, const u32x4_t& b) {
    // 16 bytes = 4 consecutive k per lane half; MFMA step j contracts k = {j, 4 + j} of the 8-wide group
    const f32x4_t fa = __builtin_bit_cast(f32x4_t, a), fb = __builtin_bit_cast(f32x4_t, b);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.x, fb.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.y, fb.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.z, fb.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa.w, fb.w, acc, 0, 0, 0);
}

__device__ inline float load_elem(const float* p) { return *p; }
__device__ inline float load_elem(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ inline void store_elem(float* p, float v) { *p = v; }
__device__ inline void store_elem(bf16_t* p, float v) { *p = (bf16_t)pack_bf16x2(v, 0.f); }

__device__ inline void load4(const float* p, float r[4]) {
    const f32x4_t v = *reinterpret_cast<const f32x4_t*>(p);
    r[0] = v.x; r[1] = v.y; r[2] = v.z; r[3] = v.w;
}
__device__ inline void load4(const bf16_t* p, float r[4]) {
    const u32x2_t v = *reinterpret_cast<const u32x2_t*>(p);
    r[0] = __uint_as_float(v.x << 16); r[1] = __uint_as_float(v.x & 0xffff0000u);
    r[2] = __uint_as_float(v.y << 16); r[3] = __uint_as_float(v.y & 0xffff0000u);
}
__device__ inline void store4(float* p, const float r[4]) {
    f32x4_t v = {r[0], r[1], r[2], r[3]};
    *reinterpret_cast<f32x4_t*>(p) = v;
}
__device__ inline void store4(bf16_t* p, const float r[4]) {
    u32x2_t v;
    v.x = pack_bf16x2(r[0], r[1]);
    v.y = pack_bf16x2(r[2], r[3]);
    *reinterpret_cast<u32x2_t*>(p) = v;
}

// 8 consecutive elements of T as one register bundle
template <typename T> struct Vec8;
template <> struct __attribute__((aligned(16))) Vec8<bf16_t> { u32x4_t v; };
template <> struct __attribute__((aligned(16))) Vec8<float> { f32x4_t lo, hi; };
__device__ inline void unpack8(const Vec8<bf16_t>& x, float r[8]) {
    const uint32_t w[4] = {x.v.x, x.v.y, x.v.z, x.v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) { r[2 * q] = __uint_as_float(w[q] << 16); r[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u); }
}
__device__ inline void unpack8(const Vec8<float>& x, float r[8]) {
    r[0] = x.lo.x; r[1] = x.lo.y; r[2] = x.lo.z; r[3] = x.lo.w; r[4] = x.hi.x; r[5] = x.hi.y; r[6] = x.hi.z; r[7] = x.hi.w;
}
__device__ inline void store8(bf16_t* p, const float r[8]) {
    u32x4_t v;
    v.x = pack_bf16x2(r[0], r[1]);
    v.y = pack_bf16x2(r[2], r[3]);
    v.z = pack_bf16x2(r[4], r[5]);
    v.w = pack_bf16x2(r[6], r[7]);
    *reinterpret_cast<u32x4_t*>(p) = v;
}
__device__ inline void store8(float* p, const float r[8]) {
    f32x4_t lo = {r[0], r[1], r[2], r[3]}, hi = {r[4], r[5], r[6], r[7]};
    *reinterpret_cast<f32x4_t*>(p) = lo;
    *reinterpret_cast<f32x4_t*>(p + 4) = hi;
}

// One bit per filter tap (ky kw + kx; kh kw <= 32) that lies inside the image, for the filter whose tap 0 is at (iy0, ix0).
// every_row: a bit at ky kw for each ky < kh.
__host__ __device__ inline uint32_t tap_mask(int iy0, int ix0, int H, int W, int kh, int kw, uint32_t every_row) {
    const int x0 = ix0 < 0 ? (-ix0 < kw ? -ix0 : kw) : 0, x1 = W - ix0 < kw ? W - ix0 : kw;
    const int y0 = iy0 < 0 ? (-iy0 < kh ? -iy0 : kh) : 0, y1 = H - iy0 < kh ? H - iy0 : kh;
    if (x1 <= x0 || y1 <= y0) return 0u;
    const uint32_t cols = (uint32_t)((1ull << x1) - (1ull << x0)), rows = (uint32_t)((1ull << (y1 * kw)) - (1ull << (y0 * kw)));
    return cols * (every_row & rows);   // (the columns once per row: no carries)
}

// Large tiles: the row of a block's first image from which the offsets of its input pixels count, oy0 being its first output row.
// (The first filter's row, before padding; with wide padding it may lie below the image, in front of which the next one begins.)
__host__ __device__ inline int large_first_row(int oy0, int stride, int H) { return oy0 * stride < H ? oy0 * stride : H; }

// compile-time loop: the body sees the index as a constant (keeps accumulator indices static)
template <int I, int N, typename F>
__device__ inline void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

}  // namespace thia
