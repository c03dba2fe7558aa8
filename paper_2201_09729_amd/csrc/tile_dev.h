// Device pieces of the tile kernels: bfloat16 words, conversions and the sums over the four
// spin lanes of a right-hand side.
#pragma once
#include "tile.h"

namespace dlma {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b16x8, a), __builtin_bit_cast(b16x8, b), c, 0, 0, 0);
}

// two numbers to one word, round to nearest even
__device__ __forceinline__ uint32_t pack16(float x, float y) {
    const f32x2 v = {x, y};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b16x2));
}
__device__ __forceinline__ float word_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float word_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// sum over the four spin lanes of a column (lanes n, n + 16, n + 32, n + 48)
__device__ __forceinline__ double sum_over_q(double v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

template <int CP> HD void wst3(const WSrc& s, uint32_t v, uint32_t u, u32x3 w) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_buffer_store_b96(w, s.r, (int)v, (int)u, CP);
#else
    (void)s; (void)v; (void)u; (void)w;
#endif
}
template <int CP> HD u32x3 wld3c(const WSrc& s, uint32_t v, uint32_t u) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_raw_buffer_load_b96(s.r, (int)v, (int)u, CP);
#else
    return wld3(s, v, u);
#endif
}

// words of one tile of a field
HD WSrc tile_src(uint32_t* f, int Vh, int tile) { return wsrc(f + (size_t)tile * Vh * 192, 768u * (uint32_t)Vh); }

}  // namespace dlma
