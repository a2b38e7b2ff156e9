// fp32 vocabulary projection on the fp16 MFMA, fused with the EOS bias, the
// online log-sum-exp and the per-row partial top-k (the bf16 form of the same
// step is in proj.hip):
//   z = W_out h,  z[0] += beta (t - L_x)      [R,d] x [V,d]^T
//
// The fp32 MFMA peaks at 157 TFLOP/s, the fp16 MFMA at 2.5 PFLOP/s, so each
// operand is split into two fp16 values: x scaled by a power of two (a W_out
// row so that its largest value is below 2^15, a state by 2^14) is
// hi + lo / 2048 with hi = fp16(x) and lo = fp16(2048 (x - hi)). x - hi is
// exact in fp32 and has at most 13 significant bits, so hi + lo / 2048 is x
// to at most one unit in the last of its 24 bits (exact for three values in
// four), for every value down to 2^-27 of the row's scale. Then
//   w h = hi hi' + (hi lo' + lo hi') / 2048 + (lo lo' <= 2^-24 |w h|, dropped)
// is three fp16 MFMAs accumulated in fp32. Over 64 values of K the cross
// terms are summed apart, scaled once and added to the running sum, so that
// they meet its rounding once. Error against 64 bits (relative 2-norm,
// N(0, 1/d) weights, tanh states) at d = 64 / 256 / 1024: 0.9 / 1.2 / 2.3e-7,
// the fp32 MFMA's two half sums: 1.1 / 2.1 / 4.1e-7.
//
// Bound: at d = 1024, |V| = 32000 a step of up to 64 rows by streaming W_out
// (131 MB at 5.4 TB/s: 24.4 us, was 31.0), larger ones by the fp16 MFMA at
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

// Tile: vocabulary tile vt x NB blocks of 32 rows from row r0.
template <int KB, int NB>
__device__ __forceinline__ void split_tile(const DevState &st, SplitSmem<KB> &sm, int vt, int r0, int R) {
  constexpr int D = NB >= 4 ? 2 : NB == 3 ? 3 : 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nch = st.d / SPLIT_K;
  const size_t blkstride = (size_t)nch * SPLIT_CHUNK;
  f16v tot[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) tot[b] = f16v{};
  split_mainloop<NB, D>(sm.stage, st.wout_t + ((size_t)(vt * 4 + wv) * nch) * SPLIT_CHUNK + lane * 16,
                        st.hsplit + (size_t)(r0 >> 5) * blkstride + tid * 16, blkstride, nch, tot);
  const SplitScale sc(st.w_scale + vt * TV + 32 * wv + 4 * (lane >> 5));
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    tot[b] = sc.apply(tot[b]);
    asm volatile("" : "+v"(tot[b]));   // not one by one in the epilogue, beside its lists
  }
  tile_epilogue<KB, NB>(st, sm.xch, [&](int b) { return tot[b]; }, vt, wv, r0, R);
}

// Blocks per row tile for a step of R rows: the count that minimizes the
// load of the fullest compute unit, its tiles times (blocks + 0.35 for a
// tile's start and epilogue); the odd tile of a compute unit runs there
// without a second workgroup to hide its latencies and counts 1.35. Measured
// at d = 1024, |V| = 32000 (us for 1 / 2 / 3 / 4 blocks): 128 rows 43.0 /
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
template <int KB>
__global__ __launch_bounds__(THREADS, 2) void k_proj_split(DevState st) {
  const int R = st.ctrl->R;
  if (R <= 0) return;
  __shared__ SplitSmem<KB> sm;
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
    switch (min(bt, (R - r0 + 31) >> 5)) {
      case 1: split_tile<KB, 1>(st, sm, vt, r0, R); break;
      case 2: split_tile<KB, 2>(st, sm, vt, r0, R); break;
      case 3: split_tile<KB, 3>(st, sm, vt, r0, R); break;
      default: split_tile<KB, 4>(st, sm, vt, r0, R); break;
    }
  }
}

// W_out, once per decoder (one workgroup per 32 vocabulary rows): the scale
// of every row, then its split values in fragment order. With every |w| of
// the row below 2^e, values are multiplied by 2^(15 - e) and a sum of
// products with 2^14-scaled states by 2^(e - 29); e is held to [-90, 128], so
// that both factors are normal numbers. Layout: [S][4 slices][d / 64 chunks]
// [4 steps][hi, lo][64 lanes][8 fp16], lane (h, l) of step s holding
// k = 64 chunk + 16 s + 8 h .. + 7 of vocabulary row 128 vt + 32 slice + l
// (zero past V). An infinite value is a low part alone: it then meets only the
// state's high part (which is not zero for |h| above 2^-39), where the high
// part's product with a state's low part of zero would be NaN.
__global__ __launch_bounds__(256) void k_split_wout(DevState st) {
  __shared__ float up[32];
  const int d = st.d, nst = d / 16, tid = threadIdx.x;
  const int vb = blockIdx.x * 32;
  const float *W = static_cast<const float *>(st.W_out);
  {
    const int v = vb + (tid >> 3);
    float mx = 0.0f;
    if (v < st.V)
      for (int i = (tid & 7) * 4; i < d; i += 32) {
        const f4 w = *reinterpret_cast<const f4 *>(W + (size_t)v * d + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) mx = fmaxf(mx, fabsf(w[q]));
      }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    int e = 0;
    if (mx >= INFINITY) e = 128;
    else if (mx > 0.0f) frexpf(mx, &e);
    e = min(max(e, -90), 128);
    if ((tid & 7) == 0) {
      up[tid >> 3] = ldexpf(1.0f, 15 - e);
      st.w_scale[v] = ldexpf(1.0f, e - 29);
    }
  }
  __syncthreads();
  const int ln = tid & 63, v = vb + (ln & 31);
  for (int s = tid >> 6; s < nst; s += 4) {
    union {
      _Float16 f[8];
      u4 u;
    } hi, lo;
    hi.u = u4{0u, 0u, 0u, 0u};
    lo.u = hi.u;
    if (v < st.V) {
      const float *src = W + (size_t)v * d + 16 * s + 8 * (ln >> 5);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = src[i] * up[ln & 31];
        split_f16(x, hi.f[i], lo.f[i]);
        if (fabsf(x) == INFINITY) {
          hi.f[i] = (_Float16)0.0f;
          lo.f[i] = (_Float16)x;
        }
      }
    }
    unsigned char *dst = st.wout_t + ((size_t)blockIdx.x * nst + s) * (2 * FRAG) + ln * 16;
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
