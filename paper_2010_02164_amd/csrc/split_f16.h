// fp32 values as pairs of fp16 for the fp32 projection (proj_f32.hip): the
// split, the layout of the pairs and one K chunk of their products.
#pragma once

#include "mfma_common.h"

namespace sb {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));

constexpr int SPLIT_K = 64;                        // K values per chunk
constexpr int SPLIT_CHUNK = SPLIT_K / 16 * 2048;   // bytes of a 32-row block's chunk: [4 steps][hi, lo][64 lanes][16 B]
constexpr float SPLIT_H_SCALE = 32768.0f;          // states are split after scaling by 2^15 (|h| <= 1)
constexpr float SPLIT_H_MIN = 1.0f / (1 << 29);    // smallest state that the pairs hold
constexpr float SPLIT_LO = 4096.0f;                // scale of the low parts

// x = hi + lo / 4096. x - hi has at most 13 significant bits, so the pair is x
// to one unit in the last of its 24 bits (exact for three values in four) for
// 2^-14 <= |x| <= 2^15; below that range it loses bits.
constexpr int SPLIT_OCTAVES = 29;
__device__ __forceinline__ void split_f16(float x, _Float16 &hi, _Float16 &lo) {
  hi = (_Float16)x;
  lo = (_Float16)((x - (float)hi) * SPLIT_LO);
}

// A product of pairs is off by up to 2^-21.2 of itself (the dropped lo lo' and
// the pairs' last unit), against 2^-24 on the fp32 MFMA; a sum of many products
// is off by less than there, because its running value is rounded less often.
// The two meet (2-norm against 64 bits, N(0, 1) weights, tanh states) at about
// 46 / 98 / 290 non-zero products for d = 64 / 256 / 1024.
__host__ __device__ constexpr int split_min_terms(int d) { return 32 + d / 4; }

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
  for (int r = 0; r < 16; ++r) tot[r] = fmaf(c[r], 1.0f / SPLIT_LO, tot[r]);
}

// tot += W chunk (8 fragments af: hi, lo of 4 steps) x state chunk (fragments
// bs[0], bs[bstride], ...).
__device__ __forceinline__ void split_chunk(const u4 *af, const u4 *bs, int bstride, f16v &tot) {
  f16v c = {};
#pragma unroll
  for (int s = 0; s < 4; ++s) split_step(af[2 * s], af[2 * s + 1], bs[2 * s * bstride], bs[(2 * s + 1) * bstride], tot, c);
  split_flush(c, tot);
}

// Whether a vocabulary tile's products are taken on the fp32 MFMA.
__device__ __forceinline__ bool split_tile_fp32(const DevState &st, int vt) {
  const int4 n = *reinterpret_cast<const int4 *>(st.w_nfar + 4 * vt);
  return (n.x | n.y | n.z | n.w) < 0;
}

// Whether a row's products are: r_far counts its states that are zero, once, and
// those below SPLIT_H_MIN, d times.
__device__ __forceinline__ bool split_row_fp32(const DevState &st, int row) {
  return st.r_far[row] > st.d - split_min_terms(st.d);
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

// z[b] += the far values of a 32-row vocabulary slice (entries f[0..n)) times
// row b's state (x + row[b]), one fused product each in list order. The caller's lane half h
// holds vocabulary rows 8 (r / 4) + 4 h + r % 4 of the slice in registers r.
// The states of four entries are loaded at a time (past the end the last
// entry's).
template <int NB>
__device__ __forceinline__ void add_far(const FarValue *f, int n, int h, const float *x, const uint32_t *row,
                                        f16v *z) {
  constexpr int U = 4;
#pragma unroll 1
  for (int i0 = 0; i0 < n; i0 += U) {
    int at[U];
    float w[U], hv[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const FarValue e = f[min(i0 + u, n - 1)];
      at[u] = __builtin_amdgcn_readfirstlane(e.at);
      w[u] = e.val;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int b = 0; b < NB; ++b) hv[u][b] = (x + (at[u] & 0xFFFF))[row[b]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u >= n) break;
      const int v = at[u] >> 16, reg = 4 * (v >> 3) + (v & 3);
      const bool mine = ((v >> 2) & 1) == h;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r == reg) {
#pragma unroll
          for (int b = 0; b < NB; ++b) z[b][r] = mine ? fmaf(w[u], hv[u][b], z[b][r]) : z[b][r];
        }
    }
  }
}

}  // namespace sb
