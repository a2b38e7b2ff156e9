// fp32 vocabulary projection on the fp16 MFMA, fused with the EOS bias, the
// online log-sum-exp and the per-row partial top-k (the bf16 form of the same
// step is in proj.hip):
//   z = W_out h,  z[0] += beta (t - L_x)      [R,d] x [V,d]^T
//
// The fp32 MFMA peaks at 157 TFLOP/s, the fp16 MFMA at 2.5 PFLOP/s, so each
// operand is split into two fp16 values: x scaled by a power of two (a W_out
// row so that its window, below, ends at 2^15, as a state does) is
// hi + lo / 4096 with hi = fp16(x) and lo = fp16(4096 (x - hi)), and
//   w h = hi hi' + (hi lo' + lo hi') / 4096 + (lo lo', up to 2^-22 |w h|: dropped)
// is three fp16 MFMAs accumulated in fp32. Over 64 values of K the cross
// terms are summed apart, scaled once and added to the running sum, so that
// they meet its rounding once. Error against 64 bits (relative 2-norm,
// N(0, 1/d) weights, tanh states) at d = 64 / 256 / 1024: 0.9 / 1.3 / 2.3e-7,
// the fp32 MFMA's two half sums: 1.1 / 2.1 / 4.1e-7.
//
// That holds for sums of many products of values within the pairs' range;
// W_out rows of another kind are found when they are split (k_split_wout):
//  - A row's window is the 29 octaves that hold most of its values. The others
//    (a large negative weight that masks a token while a unit is on, an
//    infinite one, a value next to zero) are far values: zero in the pairs,
//    listed per 32-row slice and added in fp32 to the finished sums.
//  - A tile with more far values than a slice's list holds, or with a row of
//    fewer than 32 + d / 4 non-zero values, where the fp32 MFMA's error is the
//    smaller one (split_min_terms), takes its products on the fp32 MFMA.
// The recurrence counts the states of a row that are zero, and those below 2^-29,
// which the pairs do not hold; a row with one of these, or with fewer than
// 32 + d / 4 others, takes its products on the fp32 MFMA too, after the pairs'
// pass over its tiles if others share them (tanh of an N(0, 1) sum: one row in 7e8 / d).
//
// Bound: at d = 1024, |V| = 32000 a step of up to 64 rows by streaming W_out
// (131 MB at 5.4 TB/s: 24.4 us, was 31.0; plain repeated reads: 18.6), larger ones by the fp16 MFMA at
// the rate large matrix products reach on this card (1.1 PFLOP/s): 193 rows
// 55.4 us (was 126.9), 640 rows 134 us (was 362), 2560 rows 529 us (was
// 1353; K loop 1.07 PFLOP/s, 76 us epilogue). Workgroups of 4 waves, two per
// compute unit, so that one's epilogue and barriers overlap the other's K
// loop; a tile of 128 tokens x 128 rows then streams 43 bytes per clock into
// a compute unit. Reading state fragments 1 to 3 steps ahead of their MFMAs,
// or raising the wave priority around them, changed nothing (136 us at 640).
#include <algorithm>

#include "proj_epilogue.h"
#include "split_f16.h"

namespace sb {
namespace {

constexpr int THREADS = TILE_THREADS;
constexpr int NBM = TILE_BLOCKS;

template <int KB>
union SplitSmem {
  unsigned char stage[2][NBM * SPLIT_CHUNK];      // state chunks, double-buffered
  float xch[4][32 * NBM][part_width(KB)];         // [slice][row][max, sumexp, keys]
};

// K loop of one wave: tot[b] = sum over K of its 32 vocabulary rows x batch
// block b, in chunks of 64. W_out fragments go straight to registers, D
// chunks ahead; the states pass through a double-buffered LDS copy in
// fragment order (16 bytes per lane in lane order, no bank conflicts), one
// chunk ahead in registers and one in LDS.
template <int NB, int D>
__device__ __forceinline__ void split_mainloop(unsigned char (*stage)[NBM * SPLIT_CHUNK], const unsigned char *wl,
                                               const unsigned char *sl, size_t blkstride, int nch, f16v *tot) {
  const int tid = threadIdx.x, lane16 = (tid & 63) * 16;
  u4 a[D][8], sg[NB][2];
  auto loadA = [&](int c, u4 *dst) {
    const unsigned char *p = wl + (size_t)c * SPLIT_CHUNK;
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[i] = *reinterpret_cast<const u4 *>(p + i * FRAG);
  };
  auto loadS = [&](int c) {
    const unsigned char *p = sl + (size_t)c * SPLIT_CHUNK;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 2; ++i) sg[b][i] = *reinterpret_cast<const u4 *>(p + b * blkstride + i * (SPLIT_CHUNK / 2));
  };
  auto storeS = [&](unsigned char *buf) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        *reinterpret_cast<u4 *>(buf + b * SPLIT_CHUNK + i * (SPLIT_CHUNK / 2) + tid * 16) = sg[b][i];
  };
  auto compute = [&](const unsigned char *buf, const u4 *af) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      split_chunk(af, reinterpret_cast<const u4 *>(buf + b * SPLIT_CHUNK + lane16), FRAG / 16, tot[b]);
  };
  // Loads complete in issue order; the fences keep that order fixed, so that
  // a wait for one chunk leaves the later chunks' loads in flight.
  loadS(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < D; ++c) {
    loadA(min(c, nch - 1), a[c]);
    __builtin_amdgcn_sched_barrier(0);
  }
  storeS(stage[0]);
  __builtin_amdgcn_sched_barrier(0);
  loadS(min(1, nch - 1));
  __syncthreads();
  for (int i0 = 0; i0 < nch; i0 += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int i = i0 + j;   // i % D == j
      if (i >= nch) break;
      // Chunk i + 1 into the buffer last read before the previous barrier.
      if (i + 1 < nch) storeS(stage[(i + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      loadS(min(i + 2, nch - 1));
      __builtin_amdgcn_sched_barrier(0);
      compute(stage[i & 1], a[j]);
      __builtin_amdgcn_sched_barrier(0);
      loadA(min(i + D, nch - 1), a[j]);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
    }
  }
}

// The same tile on the fp32 MFMA, from W_out and the states themselves: each K
// half in chunks of 32 values, piece q and element e of a chunk feeding k and
// k + 16, then the halves added, the sums the recompute of a saturated tile
// repeats (beam.hip). The states pass through the same LDS buffers, in
// fragments [4 pieces][64 lanes][4 floats]. Single steps with every tile here,
// d = 1024, |V| = 32000: 193 / 640 rows 200 / 411 us (110 / 200 on pairs; 250 /
// 500 with the projection on the fp32 MFMA throughout, in 8-wave workgroups).
template <int NB>
__device__ __forceinline__ void fp32_mainloop(unsigned char (*stage)[NBM * SPLIT_CHUNK], const float *wl,
                                              const float *sl, const uint32_t *row, int d, f16v *tot) {
  constexpr int KC = 32, BLOCK = 32 * KC * 4;
  const int tid = threadIdx.x, lane16 = (tid & 63) * 16, nch = d / KC;
  f4 a[4], sg[NB];
  f16v first[NB];
  auto loadA = [&](int c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = *reinterpret_cast<const f4 *>(wl + c * KC + 4 * q);
  };
  auto loadS = [&](int c) {
#pragma unroll
    for (int b = 0; b < NB; ++b) sg[b] = *reinterpret_cast<const f4 *>(sl + c * KC + row[b]);
  };
  auto storeS = [&](unsigned char *buf) {
#pragma unroll
    for (int b = 0; b < NB; ++b) *reinterpret_cast<f4 *>(buf + b * BLOCK + tid * 16) = sg[b];
  };
  loadS(0);
  loadA(0);
  storeS(stage[0]);
  loadS(min(1, nch - 1));
  __syncthreads();
  auto half = [&](int c0, int c1, f16v *acc) {
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
      if (c + 1 < nch) storeS(stage[(c + 1) & 1]);
      loadS(min(c + 2, nch - 1));
      const unsigned char *buf = stage[c & 1] + lane16;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const f4 x = *reinterpret_cast<const f4 *>(buf + b * BLOCK + q * FRAG);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][e], x[e], acc[b], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      loadA(min(c + 1, nch - 1));
      __syncthreads();
    }
  };
#pragma unroll
  for (int b = 0; b < NB; ++b) first[b] = f16v{};
  half(0, nch / 2, first);
  half(nch / 2, nch, tot);
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) tot[b][r] = first[b][r] + tot[b][r];
}

template <int KB, int NB, class Row>
__device__ __forceinline__ void split_finish(const DevState &st, SplitSmem<KB> &sm, f16v *tot, int vt, int wv, int R,
                                             Row &&row) {
  if constexpr (KB == 16)
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(tot[b]));   // not one by one in the epilogue, beside its lists
  tile_epilogue<KB, NB>(st, sm.xch, [&](int b) { return tot[b]; }, vt, wv, R, row);
}

// Tile: vocabulary tile vt x NB blocks of 32 rows from row r0.
template <int KB, bool PLAIN, int NB>
__device__ __forceinline__ void split_tile(const DevState &st, SplitSmem<KB> &sm, int vt, int r0, int R) {
  constexpr int D = NB >= 4 ? 2 : NB == 3 ? 3 : 4;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = vt * 4 + wv, nch = st.d / SPLIT_K;
  const size_t blkstride = (size_t)nch * SPLIT_CHUNK;
  f16v tot[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) tot[b] = f16v{};
  split_mainloop<NB, D>(sm.stage, st.wout_t + (size_t)slice * nch * SPLIT_CHUNK + lane * 16,
                        st.hsplit + (size_t)(r0 >> 5) * blkstride + tid * 16, blkstride, nch, tot);
  const SplitScale sc(st.w_scale + 32 * slice + 4 * h);
#pragma unroll
  for (int b = 0; b < NB; ++b) tot[b] = sc.apply(tot[b]);
  if (const int nfar = PLAIN ? 0 : st.w_nfar[slice]) {
    uint32_t row[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) row[b] = (uint32_t)min(r0 + 32 * b + (lane & 31), R - 1) * (uint32_t)st.d;
    add_far<NB>(st.w_far + (size_t)slice * SPLIT_FAR, nfar, h, static_cast<const float *>(st.proj_in), row, tot);
  }
  split_finish<KB, NB>(st, sm, tot, vt, wv, R, [r0](int s, int l) { return r0 + s + l; });
}

// The n rows map[0..n) (n > 32 (NB - 1)) of a row tile on the fp32 MFMA.
template <int KB, int NB>
__device__ __forceinline__ void fp32_tile(const DevState &st, SplitSmem<KB> &sm, int vt, const int *map, int n,
                                          int R) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k0 = 16 * (lane >> 5);
  const float *w = static_cast<const float *>(st.W_out) +
                   (size_t)min((vt * 4 + wv) * 32 + (lane & 31), st.V - 1) * st.d + k0;
  uint32_t row[NB];   // the states are under 4 GiB
#pragma unroll
  for (int b = 0; b < NB; ++b) row[b] = (uint32_t)map[min(32 * b + (lane & 31), n - 1)] * (uint32_t)st.d + k0;
  f16v tot[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) tot[b] = f16v{};
  fp32_mainloop<NB>(sm.stage, w, static_cast<const float *>(st.proj_in) + 4 * wv, row, st.d, tot);
  split_finish<KB, NB>(st, sm, tot, vt, wv, R, [map, n, R](int s, int l) { return s + l < n ? map[s + l] : R; });
}

// Which of a tile's rows (nrows from r0, at most 128) need the fp32 MFMA: all of
// them where the vocabulary tile does. Every wave finds the same.
struct Fp32Rows {
  unsigned long long m[2];   // rows r0 .. + 63 and r0 + 64 .. + 127
  __device__ Fp32Rows(const DevState &st, bool far, int vt, int r0, int nrows) {
    const bool every = split_tile_fp32(st, vt);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const int i = lane + 64 * w;
      m[w] = every || far ? __ballot(i < nrows && (every || split_row_fp32(st, r0 + i))) : 0ull;
    }
  }
  __device__ int count() const { return __popcll(m[0]) + __popcll(m[1]); }
  // The rows in order, to LDS.
  __device__ void list(int *map, int r0) const {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w < 2 && ((m[w & 1] >> lane) & 1ull))
      map[(w ? __popcll(m[0]) : 0) + __popcll(m[w & 1] & ((1ull << lane) - 1ull))] = r0 + 64 * w + lane;
    __syncthreads();
  }
};

// Blocks per row tile for a step of R rows: the count that minimizes the
// load of the fullest compute unit, its tiles times (blocks + 0.35 for a
// tile's start and epilogue); the odd tile of a compute unit runs there
// without a second workgroup to hide its latencies and counts 1.35. Measured
// at d = 1024, |V| = 32000 only (us for 1 / 2 / 3 / 4 blocks): 128 rows 43.0 /
// 36.0 / 45.7 / 41.1, 193 rows 70.8 / 58.8 / 66.5 / 55.4, 320 rows 94.3 /
// 76.6 / 81.0 / 88.3, 384 rows 110.8 / 91.8 / 85.5 / 91.3, 640 rows 183.2 /
// 152.7 / 150.7 / 133.9; the rule takes the fastest in each.
__device__ __forceinline__ int split_tile_blocks(int R, int S, int n_cu) {
  const int B = (R + 31) >> 5;
  int best_bt = NBM;
  float best = 3.0e38f;
  for (int bt = 1; bt <= NBM; ++bt) {
    const int nra = (B + bt - 1) / bt;
    const int k = (S * nra + n_cu - 1) / n_cu;   // tiles of a compute unit
    const float cost = ((float)k + 0.35f * (k & 1)) * ((float)min(bt, B) + 0.35f);
    if (cost <= best) {
      best = cost;
      best_bt = bt;
    }
  }
  return best_bt;
}

// Persistent over the step's tiles, at most two workgroups per compute unit.
// XCD x takes the x-th eighth of the tile list (vocabulary tile major), so
// the row tiles of one vocabulary tile run side by side on one XCD and share
// its L2 copy of the W_out tile; rounds alternate direction, so that a
// workgroup which drew a full row tile draws a partial one in the next.
// A step of plain rows only, of W_out and of states (most are), has a walk of its
// own: a kind looked up per tile, ahead of its K loop, cost 0.3 us per step.
// Other steps take two: the pairs over the tiles that have rows for them, then,
// where a workgroup met others, the fp32 MFMA over those, closed up to blocks of
// 32 in each tile; their records replace the pairs' (a workgroup's own, in both
// walks). One walk of both kinds does not fit the registers.
enum WalkKind { WALK_PLAIN, WALK_PAIRS, WALK_FP32 };
template <int KB, WalkKind KIND>
__device__ __forceinline__ bool split_walk(const DevState &st, SplitSmem<KB> &sm, int *map, bool far, int R) {
  bool others = false;   // rows left to the fp32 MFMA
  const int bt = split_tile_blocks(R, st.S, st.n_cu);
  const int nra = (R + 32 * bt - 1) / (32 * bt);
  const int T = st.S * nra;
  const TileOrder order(st.S, nra, 32 * bt * st.d * 4);
  const int x = blockIdx.x & 7, gx = gridDim.x >> 3, j = blockIdx.x >> 3;
  const int lo = (int)((long long)T * x / 8), nt = (int)((long long)T * (x + 1) / 8) - lo;
  for (int r = 0; r * gx < nt; ++r) {
    const int idx = (r & 1) ? (r + 1) * gx - 1 - j : r * gx + j;
    if (idx >= nt) continue;
    const int tile = lo + idx;
    int vt, rt;
    order.at(tile, vt, rt);
    const int r0 = rt * bt * 32;
    if constexpr (KIND != WALK_FP32) {
      if constexpr (KIND == WALK_PAIRS) {
        const int nrows = min(32 * bt, R - r0), n = Fp32Rows(st, far, vt, r0, nrows).count();
        others |= n > 0;
        if (n == nrows) continue;
      }
      constexpr bool PLAIN = KIND == WALK_PLAIN;
      switch (min(bt, (R - r0 + 31) >> 5)) {
        case 1: split_tile<KB, PLAIN, 1>(st, sm, vt, r0, R); break;
        case 2: split_tile<KB, PLAIN, 2>(st, sm, vt, r0, R); break;
        case 3: split_tile<KB, PLAIN, 3>(st, sm, vt, r0, R); break;
        default: split_tile<KB, PLAIN, 4>(st, sm, vt, r0, R); break;
      }
    } else {
      const Fp32Rows rows(st, far, vt, r0, min(32 * bt, R - r0));
      const int n = rows.count();
      if (n == 0) continue;
      rows.list(map, r0);
      switch ((n + 31) >> 5) {
        case 1: fp32_tile<KB, 1>(st, sm, vt, map, n, R); break;
        case 2: fp32_tile<KB, 2>(st, sm, vt, map, n, R); break;
        case 3: fp32_tile<KB, 3>(st, sm, vt, map, n, R); break;
        default: fp32_tile<KB, 4>(st, sm, vt, map, n, R); break;
      }
    }
  }
  return others;
}

template <int KB>
__global__ __launch_bounds__(THREADS, 2) void k_proj_split(DevState st) {
  const int R = st.ctrl->R, far = st.ctrl->far, w_mixed = st.ctrl->w_mixed;
  if (R <= 0 || w_mixed < 0) return;   // w_mixed is 0 or 1: tested here so that the loads are one wait
  __shared__ SplitSmem<KB> sm;
  __shared__ int map[32 * NBM];
  if (__builtin_expect((w_mixed | far) == 0, 1)) {
    split_walk<KB, WALK_PLAIN>(st, sm, map, false, R);
    return;
  }
  if (split_walk<KB, WALK_PAIRS>(st, sm, map, far != 0, R)) split_walk<KB, WALK_FP32>(st, sm, map, far != 0, R);
}

// W_out, once per decoder (one workgroup per 32 vocabulary rows): the window
// and scale of every row, then its split values in fragment order. A row's
// window are the values whose exponent field is in [top - 28, top]: it ends at
// the largest value where that leaves none below it, else lies where it holds
// most (top is held to [36, 254], so that the factors below are normal
// numbers). With e = top - 126, values are multiplied by 2^(15 - e) and a sum
// of products with 2^15-scaled states by 2^(e - 30). Layout: [S][4 slices]
// [d / 64 chunks][4 steps][hi, lo][64 lanes][8 fp16], lane (h, l) of step s
// holding k = 64 chunk + 16 s + 8 h .. + 7 of vocabulary row
// 128 vt + 32 slice + l (zero past V, and for far values).
__device__ __forceinline__ int exp_field(float x) { return (int)((__float_as_uint(x) >> 23) & 0xFFu); }
__device__ __forceinline__ bool is_far(float x, int top) {
  const int e = exp_field(x);
  return x != 0.0f && (e > top || e <= top - SPLIT_OCTAVES);   // NaN and infinities: e = 255
}

__global__ __launch_bounds__(256) void k_split_wout(DevState st) {
  __shared__ int tops[32];
  __shared__ uint32_t hist[32][128];   // two 16-bit counts per word: values of a row by exponent field
  __shared__ int wave_far[4];
  const int d = st.d, nst = d / 16, tid = threadIdx.x, lane = tid & 63;
  const int vb = blockIdx.x * 32, row = tid >> 3, part = tid & 7;
  const float *W = static_cast<const float *>(st.W_out);
  const float *wr = W + (size_t)min(vb + row, st.V - 1) * d;   // the thread's share: 4 values of every 32
  const bool real = vb + row < st.V;
  uint32_t most_bits = 0u, least = 0xFFFFFFFFu;   // largest magnitude; smallest not zero, less one
  int terms = 0;
  if (real)
    for (int i = part * 4; i < d; i += 32) {
      const u4 w = *reinterpret_cast<const u4 *>(wr + i);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t u = w[q] & 0x7FFFFFFFu;
        most_bits = max(most_bits, u);
        least = min(least, u - 1u);
        terms += u != 0u;
      }
    }
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) {
    most_bits = max(most_bits, (uint32_t)__shfl_xor((int)most_bits, o, 64));
    least = min(least, (uint32_t)__shfl_xor((int)least, o, 64));
    terms += __shfl_xor(terms, o, 64);
  }
  const int largest = (int)(most_bits >> 23), smallest = terms ? (int)((least + 1u) >> 23) : 255;
  int top = min(max(largest, 36), 254);
  const bool wide = largest == 255 || smallest <= top - SPLIT_OCTAVES;
  bool few = terms > 0 && terms < split_min_terms(d);
  int nfar = 0;
  const bool any_wide = __syncthreads_or(wide);
  if (any_wide) {
    for (int i = tid; i < 32 * 128; i += 256) (&hist[0][0])[i] = 0u;
    __syncthreads();
    if (wide)
      for (int i = part * 4; i < d; i += 32) {
        const f4 w = *reinterpret_cast<const f4 *>(wr + i);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (w[q] != 0.0f) atomicAdd(&hist[row][exp_field(w[q]) >> 1], exp_field(w[q]) & 1 ? 65536u : 1u);
      }
    __syncthreads();
    if (wide) {
      auto count = [&](int e) { return e < 0 ? 0 : (int)((hist[row][e >> 1] >> (16 * (e & 1))) & 0xFFFFu); };
      int held = 0;
      for (int e = top; e > top - SPLIT_OCTAVES; --e) held += count(e);
      int most = held;
      for (int t = top - 1; t >= max(36, smallest); --t) {   // of equal ones the lowest: it ends at its largest value
        held += count(t + 1 - SPLIT_OCTAVES) - count(t + 1);
        if (held >= most) {
          most = held;
          top = t;
        }
      }
      few = most > 0 && most < split_min_terms(d);
    }
    // Places of the far values: by row, then by share.
    int n = 0;
    if (wide)
      for (int i = part * 4; i < d; i += 32) {
        const f4 w = *reinterpret_cast<const f4 *>(wr + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) n += is_far(w[q], top);
      }
    int at = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(at, o, 64);
      if (lane >= o) at += y;
    }
    if (lane == 63) wave_far[tid >> 6] = at;
    at -= n;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      at += x < tid >> 6 ? wave_far[x] : 0;
      nfar += wave_far[x];
    }
    if (n > 0 && nfar <= SPLIT_FAR) {
      FarValue *f = st.w_far + (size_t)blockIdx.x * SPLIT_FAR + at;
      for (int i = part * 4; i < d; i += 32) {
        const f4 w = *reinterpret_cast<const f4 *>(wr + i);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (is_far(w[q], top)) *f++ = FarValue{row << 16 | (i + q), w[q]};
      }
    }
  }
  if (part == 0) {
    tops[row] = top;
    st.w_scale[vb + row] = ldexpf(1.0f, top - 126 - 30);
  }
  const bool fp32 = __syncthreads_or(few) || nfar > SPLIT_FAR;
  if (tid == 0) {
    st.w_nfar[blockIdx.x] = fp32 ? -1 : nfar;
    if (fp32 || nfar > 0) st.ctrl->w_mixed = 1;
  }
  const int v = vb + (lane & 31), vtop = tops[lane & 31];
  const float up = ldexpf(1.0f, 15 + 126 - vtop);
  for (int s = tid >> 6; s < nst; s += 4) {
    union {
      _Float16 f[8];
      u4 u;
    } hi, lo;
    hi.u = u4{0u, 0u, 0u, 0u};
    lo.u = hi.u;
    if (v < st.V) {
      const float *src = W + (size_t)v * d + 16 * s + 8 * (lane >> 5);
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = src[i];
      if (any_wide)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = is_far(x[i], vtop) ? 0.0f : x[i];
#pragma unroll
      for (int i = 0; i < 8; ++i) split_f16(x[i] * up, hi.f[i], lo.f[i]);
    }
    unsigned char *dst = st.wout_t + ((size_t)blockIdx.x * nst + s) * (2 * FRAG) + lane * 16;
    *reinterpret_cast<u4 *>(dst) = hi.u;
    *reinterpret_cast<u4 *>(dst + FRAG) = lo.u;
  }
}

}  // namespace

hipError_t launch_split_wout(const DevState &st, hipStream_t s) {
  hipLaunchKernelGGL(k_split_wout, dim3(st.S * 4), dim3(256), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_proj_split(const DevState &st, hipStream_t s) {
  // A multiple of 8, at most two per compute unit, no more than the 32-row
  // tiles of a full step.
  const int G = std::max(8, std::min(st.n_cu / 4 * 8, xcd_grid(st.S * ((st.R_max + 31) / 32))));
  switch (st.tile_keys) {
    case 4: hipLaunchKernelGGL((k_proj_split<4>), dim3(G), dim3(THREADS), 0, s, st); break;
    case 8: hipLaunchKernelGGL((k_proj_split<8>), dim3(G), dim3(THREADS), 0, s, st); break;
    default: hipLaunchKernelGGL((k_proj_split<16>), dim3(G), dim3(THREADS), 0, s, st); break;
  }
  return hipGetLastError();
}

}  // namespace sb
