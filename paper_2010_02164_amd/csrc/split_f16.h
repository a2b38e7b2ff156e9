// fp32 values as pairs of fp16 for the fp32 projection (proj_f32.hip): the
// split, the layout of the pairs and one K chunk of their products.
#pragma once

#include "mfma_common.h"

namespace sb {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int SPLIT_K = 64;                        // K values per chunk
constexpr int SPLIT_CHUNK = SPLIT_K / 16 * 2048;   // bytes of a 32-row block's chunk: [4 steps][hi, lo][64 lanes][16 B]
constexpr float SPLIT_H_SCALE = 16384.0f;          // states are split after scaling by 2^14 (|h| <= 1)

// x = hi + lo / 2048, to one unit in the last of x's 24 bits or better.
__device__ __forceinline__ void split_f16(float x, _Float16 &hi, _Float16 &lo) {
  hi = (_Float16)x;
  lo = (_Float16)((x - (float)hi) * 2048.0f);
}

// Byte offset of value k of row r in the split states [R / 32][d / 16][hi, lo]
// [64 lanes][8 fp16]; the lo part follows 1024 bytes later.
__device__ __forceinline__ size_t split_state_off(int d, int r, int k) {
  return ((size_t)(r >> 5) * (d / 16) + (k >> 4)) * 2048 + ((((k >> 3) & 1) << 5) + (r & 31)) * 16 + (k & 7) * 2;
}

// One step (16 values of K): the sum of the high parts' products, and the
// cross terms, which are summed apart over a chunk and join the sum once.
__device__ __forceinline__ void split_step(u4 wh, u4 wl, u4 bh, u4 bl, f16v &tot, f16v &c) {
  tot = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, wh), __builtin_bit_cast(h8, bh), tot, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, wl), __builtin_bit_cast(h8, bh), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, wh), __builtin_bit_cast(h8, bl), c, 0, 0, 0);
}
__device__ __forceinline__ void split_flush(const f16v &c, f16v &tot) {
#pragma unroll
  for (int r = 0; r < 16; ++r) tot[r] = fmaf(c[r], 1.0f / 2048.0f, tot[r]);
}

// tot += W chunk (8 fragments af: hi, lo of 4 steps) x state chunk (fragments
// bs[0], bs[bstride], ...).
__device__ __forceinline__ void split_chunk(const u4 *af, const u4 *bs, int bstride, f16v &tot) {
  f16v c = {};
#pragma unroll
  for (int s = 0; s < 4; ++s) split_step(af[2 * s], af[2 * s + 1], bs[2 * s * bstride], bs[(2 * s + 1) * bstride], tot, c);
  split_flush(c, tot);
}

// The 16 vocabulary rows' scales of a lane (register r: row 8 (r / 4) + r % 4
// from `p`).
struct SplitScale {
  f4 s[4];
  __device__ explicit SplitScale(const float *p) {
#pragma unroll
    for (int g = 0; g < 4; ++g) s[g] = *reinterpret_cast<const f4 *>(p + 8 * g);
  }
  __device__ f16v apply(const f16v &t) const {
    f16v z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = t[r] * s[r >> 2][r & 3];
    return z;
  }
};

}  // namespace sb
