// Epilogue of the vocabulary projection, shared by its fp32 and bf16
// kernels: a 32 x 32 block of logits is folded into per-row (max, sum exp)
// and best keys, and a row's four 32-token slices of a 128-token tile into
// the tile's partial record.
#pragma once

#include "mfma_common.h"
#include "topk.h"
#include "wave.h"

namespace sb {

constexpr int TV = GEMM_BV;      // vocabulary rows per tile (4 slices x 32)
constexpr int TILE_BLOCKS = 4;   // 32-row batch blocks per tile, at most
constexpr int TILE_THREADS = 256;   // 4 waves, each 32 vocabulary rows of the tile
constexpr int FRAG = 1024;       // bytes of one wave-wide 16-byte-per-lane fragment

// Order of a step's tiles, of which XCD x takes the x-th eighth: groups of row
// tiles, in a group vocabulary tile major. A group's states (2 MB) stay in an
// XCD's 4 MB L2 while its share of the weights streams by; ungrouped, the
// states of a large step (10 MB for 5120 bf16 rows at d = 1024) are fetched
// again for every vocabulary tile. bf16, |V| = 32000, us, ungrouped / 1 / 2 /
// 3 MB: 5120 rows 512 / 485 / 465 / 479, 2560 rows 246 / 249 / 241 / 245;
// smaller steps and the fp32 ones are within 2 % of each other.
constexpr int GROUP_BYTES = 2 << 20;
struct TileOrder {
  int nvt, nra, group;
  __device__ TileOrder(int nvt, int nra, int row_tile_bytes) : nvt(nvt), nra(nra) {
    const int most = max(1, GROUP_BYTES / row_tile_bytes), groups = (nra + most - 1) / most;
    group = (nra + groups - 1) / groups;
  }
  __device__ void at(int t, int &vt, int &rt) const {
    const int rg = t / (nvt * group), rem = t - rg * nvt * group;
    const int n = min(group, nra - rg * group);
    vt = rem / n;
    rt = rg * group + rem - vt * n;
  }
};

// Lane-level epilogue of one 32-row block: lane holds batch row l32 of the
// block and the wave's vocabulary rows v0 + 32wv + 8*(reg/4) + 4h + reg%4
// (increasing with reg). Adds the EOS bias, folds the 16 logits into
// (max, sum exp) and a sorted best-KB key list, then combines lanes l and
// l+32 (same row), which end with identical results. KB = 4 takes a
// cheaper network than a full sort.
template <int KB>
__device__ __forceinline__ void block_lists(const f16v &z, int v0, int wv, int h, int V, float bias, float &m_out,
                                            float &s_out, TopK<KB> &tk) {
  float vals[16];
  if (v0 != 0 && v0 + TV <= V) {   // interior tile: no EOS bias, no rows past V
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) vals[reg] = z[reg];
  } else {
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) {
      const int v = v0 + 32 * wv + 8 * (reg >> 2) + 4 * h + (reg & 3);
      const float zz = v == 0 ? z[reg] + bias : z[reg];
      vals[reg] = v < V ? zz : -INFINITY;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < 16; ++q) m = fmaxf(m, vals[q]);
  float s = 0.0f;
  if (m > -INFINITY) {
#pragma unroll
    for (int q = 0; q < 16; ++q) s += __expf(vals[q] - m);
  }
  // The lane's 16 candidates as ranking keys, sorted by a network.
  cand_key keys[16];
#pragma unroll
  for (int reg = 0; reg < 16; ++reg) keys[reg] = make_key(vals[reg], v0 + 32 * wv + 8 * (reg >> 2) + 4 * h + (reg & 3));
  TopK<KB> mine;
  if constexpr (KB == 4) {
    top4_of_16(keys, mine);
  } else {
    bitonic_sort_desc<16>(keys);
#pragma unroll
    for (int q = 0; q < KB; ++q) mine.k[q] = keys[q];
  }
  TopK<KB> lo, hi;
#pragma unroll
  for (int q = 0; q < KB; ++q) stage64<5>(mine.k[q], lo.k[q], hi.k[q]);
  topk_merge(lo, hi);
  tk = lo;
  uint32_t ma, mb, sa, sb;
  stage32<5>(__float_as_uint(m), ma, mb);
  stage32<5>(__float_as_uint(s), sa, sb);
  m = __uint_as_float(ma);
  s = __uint_as_float(sa);
  lse_merge(m, s, __uint_as_float(mb), __uint_as_float(sb));
  m_out = m;
  s_out = s;
}

// Partial record of (row j, vocabulary tile vt): the merge of the four
// vocabulary slices' (max, sum exp, key list), read from LDS.
template <int KB>
__device__ __forceinline__ void write_record(const DevState &st, int j, int vt, const float *const *slices) {
  constexpr int PW = part_width(KB);
  float m = -INFINITY, s = 0.0f;
  TopK<KB> tk;
  topk_init(tk);
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const float *p = slices[x];
    TopK<KB> o;
    topk_load(o, p + 2);
    lse_merge(m, s, p[0], p[1]);
    topk_merge(tk, o);
  }
  float rec[PW];
  rec[0] = m;
  rec[1] = s;
  topk_store(rec + 2, tk);
#pragma unroll
  for (int x = 2 + 2 * KB; x < PW; ++x) rec[x] = 0.0f;
  u4 *out = reinterpret_cast<u4 *>(st.part + ((size_t)j * st.S + vt) * PW);
#pragma unroll
  for (int x = 0; x < PW / 4; ++x)
    out[x] = u4{__float_as_uint(rec[4 * x]), __float_as_uint(rec[4 * x + 1]), __float_as_uint(rec[4 * x + 2]),
                __float_as_uint(rec[4 * x + 3])};
}

// Epilogue of a tile of NB blocks (its row s + l is row(s, l), s the same in every
// lane; R or above past the last) of vocabulary tile vt, by a workgroup of 4 waves: wave wv's lane lists of its
// 32-token slice of each block (logits z(b)), then one thread per row merges the
// four slices. Ends with a barrier: LDS may be reused.
template <int KB, int NB, class Z, class Row>
__device__ __forceinline__ void tile_epilogue(const DevState &st, float (*xch)[32 * TILE_BLOCKS][part_width(KB)],
                                              Z &&z, int vt, int wv, int R, Row &&row) {
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int v0 = vt * TV;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int j = row(32 * b, l32);
    const float bias = (v0 == 0 && j < R) ? st.beta * (float)(st.r_t[j] - st.r_Lx[j]) : 0.0f;
    float m, s;
    TopK<KB> tk;
    block_lists<KB>(z(b), v0, wv, h, st.V, bias, m, s, tk);
    if (lane < 32) {
      float *p = xch[wv][32 * b + l32];
      p[0] = m;
      p[1] = s;
      topk_store(p + 2, tk);
    }
  }
  __syncthreads();
  if (tid < 32 * NB && row(0, tid) < R) {
    const float *sl[4] = {xch[0][tid], xch[1][tid], xch[2][tid], xch[3][tid]};
    write_record<KB>(st, row(0, tid), vt, sl);
  }
  __syncthreads();
}

}  // namespace sb
