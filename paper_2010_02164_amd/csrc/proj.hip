// bf16 vocabulary projection of the synthetic decoder D (Sec. 2) on gfx950
// MFMA (the fp32 one is in proj_f32.hip), fused with the EOS bias, an online
// log-sum-exp and a per-row partial top-k:
//   z = W_out h,  z[0] += beta (t - L_x)      [R,d] x [V,d]^T
// The R x |V| logits never reach memory: each workgroup writes, per row and
// 128-wide vocabulary tile, (max, sum exp) and its best keys (value, token).
//
// Workgroups of 4 waves, two per compute unit, walk the step's tiles of 128
// vocabulary rows x 1..4 blocks of 32 batch rows on a persistent grid, each
// wave over its own 32 vocabulary rows. The K range is summed in two fixed
// halves, added once at the end; an output's MFMA sequence is the same in
// every tile, so a row's result does not depend on the batch or on the
// tiling.
//
// Bound: streaming W_out up to about 64 rows (65 MB in 15 us at |V| = 32000;
// plain repeated reads: 10.1); beyond, latencies inside a
// wave's K loop (with all loads made trivial it takes 79 % of its time; at
// 5120 rows the MFMAs are 38 % of a tile's cycles, the epilogue 26 %).
// d = 1024, |V| = 32000, us, against workgroups of 8 waves, one per compute
// unit, with the K halves on two wave groups: 21 rows 15.0 (17.3), 389 rows
// 49.5 (56.0), 640 rows 64.5 (77.8), 1600 rows 148 (175), 5120 rows 450 (500).
// Storing a chunk's states before the previous chunk's MFMAs instead of
// after them gave 389 rows 52.0 -> 48.2, 640 rows 67.0 -> 61.4; a third
// chunk of weights in flight 49.4 and 63.2.
//
// The same tile walk, with W_kv in place of W_out and a bf16 store in place
// of the log-sum-exp / top-k epilogue, appends each expansion's KV rows
// (k_kv_append, below).
//
// W_out is streamed straight into registers from a copy laid out in MFMA
// fragment order (one coalesced 1 KB load per wave and fragment), kept D
// chunks ahead; the states pass through a double-buffered LDS tile shared by
// the waves, one chunk ahead in registers and one in LDS.
// Blocks of 32 rows past R are neither loaded nor computed.
#include <algorithm>

#include "proj_epilogue.h"

namespace sb {
namespace {

constexpr int THREADS = TILE_THREADS;
constexpr int NBM = TILE_BLOCKS;
constexpr int CH = 128;          // bytes of a row's K chunk
constexpr int LS = CH + 16;      // padded LDS row stride (bytes)
constexpr int WCH = 4 * FRAG;    // bytes of one wave's weight fragments per chunk

template <int KB>
union ProjSmem {
  unsigned char B[2][32 * NBM][LS];               // state chunks, double-buffered
  float xch[4][32 * NBM][part_width(KB)];         // [slice][row][max, sumexp, keys]
};

// K loop of one wave: acc[half][b] = the sum over a K half of its 32 weight
// rows x batch block b. Chunk c: weight fragments at abase + c * 16 KB (+
// lane * 16 + q * 1 KB), the state tile at bbase + c * 128 bytes (+ boff[u]).
// Weights are loaded D chunks ahead of use into registers; the states one
// chunk ahead into registers and one into LDS, stored before a chunk's MFMAs
// so that nothing but the MFMAs stands before the barrier. Loads are at
// indices clamped to the last chunk, so that none sits in a branch; they
// complete in issue order, and the scheduling fences keep that order fixed.
template <int NB, int D>
__device__ __forceinline__ void proj_mainloop(unsigned char (*stage)[32 * NBM][LS], const unsigned char *abase,
                                              uint32_t alane, const unsigned char *bbase, const uint32_t *boff,
                                              int nk, f16v (*acc)[NB]) {
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int srow = tid >> 3, scol = (tid & 7) * 16;
  u4 a[D][4], sg[NB];
  auto loadA = [&](int c, u4 *dst) {
    const unsigned char *p = abase + (uint32_t)c * (uint32_t)(4 * WCH);
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q] = *reinterpret_cast<const u4 *>(p + alane + q * FRAG);
  };
  auto loadB = [&](int c) {
    const unsigned char *p = bbase + (uint32_t)c * CH;
#pragma unroll
    for (int u = 0; u < NB; ++u) sg[u] = *reinterpret_cast<const u4 *>(p + boff[u]);
  };
  auto storeB = [&](unsigned char (*T)[LS]) {
#pragma unroll
    for (int u = 0; u < NB; ++u) *reinterpret_cast<u4 *>(&T[srow + 32 * u][scol]) = sg[u];
  };
  auto compute = [&](unsigned char (*T)[LS], const u4 *af, f16v *c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // K permutation: lane half h at piece q feeds k = chunk + 32h + 8q + e,
      // identically for both operands.
      u4 braw[NB];
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) braw[bb] = *reinterpret_cast<const u4 *>(&T[32 * bb + l32][64 * h + 16 * q]);
#pragma unroll
      for (int bb = 0; bb < NB; ++bb)
        c[bb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, af[q]),
                                                        __builtin_bit_cast(bf8, braw[bb]), c[bb], 0, 0, 0);
    }
  };
  loadB(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < D; ++c) {
    loadA(min(c, nk - 1), a[c]);
    __builtin_amdgcn_sched_barrier(0);
  }
  storeB(stage[0]);
  __builtin_amdgcn_sched_barrier(0);
  loadB(min(1, nk - 1));
  __syncthreads();
  const int nh = nk >> 1;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int c0 = half * nh, c1 = c0 + nh;
    if (half)   // chunk c0 + j into a[j]
      for (int r = nh % D; r > 0; --r) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const u4 t = a[0][q];
#pragma unroll
          for (int x = 0; x + 1 < D; ++x) a[x][q] = a[x + 1][q];
          a[D - 1][q] = t;
        }
      }
    for (int i0 = c0; i0 < c1; i0 += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int i = i0 + j;
        if (i >= c1) break;
        // Chunk i + 1 into the buffer last read before the previous barrier.
        if (i + 1 < nk) storeB(stage[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        loadB(min(i + 2, nk - 1));
        __builtin_amdgcn_sched_barrier(0);
        compute(stage[i & 1], a[j], acc[half]);
        __builtin_amdgcn_sched_barrier(0);
        loadA(min(i + D, nk - 1), a[j]);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
      }
    }
  }
}

// KV append epilogue of one 32-row block of a wave's 32 outputs (the layout
// of block_lists): row j's bf16(sum) values go to the KV rows of the
// expanded candidate, at (beam, level t-1, rank), outputs o0 + 8*(reg/4) +
// 4h + reg%4.
__device__ __forceinline__ uint16_t bf16_rne_f(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ void kv_store_block(const DevState &st, const f16v &z, int o0, int h, int j, int R) {
  if (j >= R) return;
  const int NO = st.kv_layers * 2 * st.d;
  const int slot = st.r_slot[j], beam = slot / st.k, rank = slot - beam * st.k;
  uint16_t *out = st.kvs + (((size_t)beam * st.max_len_cap + (st.r_t[j] - 1)) * st.k + rank) * NO + o0 + 4 * h;
#pragma unroll
  for (int gq = 0; gq < 4; ++gq) {
    u2 pk;
    pk[0] = (uint32_t)bf16_rne_f(z[4 * gq + 0]) | ((uint32_t)bf16_rne_f(z[4 * gq + 1]) << 16);
    pk[1] = (uint32_t)bf16_rne_f(z[4 * gq + 2]) | ((uint32_t)bf16_rne_f(z[4 * gq + 3]) << 16);
    *reinterpret_cast<u2 *>(out + 8 * gq) = pk;
  }
}

// Weights and rows a tile walk reads: W_out and the projection input for
// the vocabulary projection; W_kv and the new states for the KV append.
struct GemmOperands {
  const unsigned char *w;   // fragment-ordered weights, 128 outputs per tile
  const void *in;           // [R][d] rows
};

// Tile of NB blocks of 32 rows from row r0 and weight tile vt.
template <int KB, bool KV, int NB>
__device__ __forceinline__ void proj_tile(const DevState &st, const GemmOperands &op, ProjSmem<KB> &sm, int vt, int r0,
                                          int R) {
  constexpr int D = NB >= 4 ? 2 : NB == 3 ? 3 : 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rowbytes = st.d * 2, nk = rowbytes / CH;   // even: d is a multiple of 128
  // State staging: thread -> rows tid/8 + 32u of the tile (clamped to R-1),
  // 16-byte column tid%8 of the chunk.
  uint32_t boff[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u)
    boff[u] = (uint32_t)min(r0 + (tid >> 3) + 32 * u, R - 1) * (uint32_t)rowbytes + (tid & 7) * 16;
  f16v acc[2][NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[0][b] = acc[1][b] = f16v{};
  // Weight fragments of this wave: chunk c at ((vt*nk + c)*4 + wv) * 4 KB.
  proj_mainloop<NB, D>(sm.B, op.w + ((size_t)vt * nk * 4 + wv) * WCH, (uint32_t)lane * 16u,
                       static_cast<const unsigned char *>(op.in), boff, nk, acc);
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int reg = 0; reg < 16; ++reg) acc[0][b][reg] += acc[1][b][reg];
  // With 16 keys the sums are formed here: left to the compiler they move into
  // the epilogue, block by block, and both halves stay in registers beside its
  // key lists (256 registers and 18 spilled, now 237 and none).
  if constexpr (KB == 16)
#pragma unroll
    for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(acc[0][b]));
  if constexpr (KV) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      kv_store_block(st, acc[0][b], vt * TV + 32 * wv, lane >> 5, r0 + 32 * b + (lane & 31), R);
  } else {
    tile_epilogue<KB, NB>(st, sm.xch, [&](int b) { return acc[0][b]; }, vt, wv, R,
                          [r0](int s, int l) { return r0 + s + l; });
  }
}

// Blocks per row tile for a step of R rows: the rule of the fp32 projection
// (split_tile_blocks) with 0.7 of a block for a tile's start and epilogue,
// whose weight is larger next to a third of the MFMAs. Measured at d = 1024,
// |V| = 32000 only (us for 1 / 2 / 3 / 4 blocks): 64 rows 16.7 / 18.4 / 18.7 /
// 18.8, 128 rows 27.0 / 21.5 / 25.6 / 25.1, 193 rows 43.6 / 34.6 / 39.2 /
// 30.6, 320 rows 54.6 / 42.9 / 43.3 / 47.0, 640 rows 100.5 / 73.7 / 73.0 /
// 64.7, 5120 rows 842 / 626 / 553 / 495.
__device__ __forceinline__ int row_tile_blocks(int R, int S, int n_cu) {
  const int B = (R + 31) >> 5;
  int best_bt = NBM;
  float best = 3.0e38f;
  for (int bt = 1; bt <= NBM; ++bt) {
    const int nra = (B + bt - 1) / bt;
    const int k = (S * nra + n_cu - 1) / n_cu;   // tiles of a compute unit
    const float cost = ((float)k + 0.35f * (k & 1)) * ((float)min(bt, B) + 0.7f);
    if (cost <= best) {
      best = cost;
      best_bt = bt;
    }
  }
  return best_bt;
}

// Persistent launch: at most two workgroups per compute unit, each walking
// its share of the active tiles (weight tile major, row tile minor).
// Workgroup ids are dealt round robin to the 8 XCDs; XCD x takes the x-th
// eighth of the tile list, so the row tiles of one weight tile run side by
// side on one XCD and share its L2 copy of the weights. Rounds alternate
// direction over the XCD's workgroups, so that a workgroup which drew a full
// row tile in one round draws a partial one in the next. Only tiles holding
// rows of this step are visited, and no workgroup is launched just to exit
// (idle ones would occupy compute units that the dispatcher then withholds
// from working ones).
template <int KB, bool KV>
__device__ __forceinline__ void tile_walk(const DevState &st, const GemmOperands &op, int nvt) {
  const int R = st.ctrl->R;
  if (R <= 0) return;
  __shared__ ProjSmem<KB> sm;
  const int bt = row_tile_blocks(R, nvt, st.n_cu);
  const int nra = (R + 32 * bt - 1) / (32 * bt);
  const int T = nvt * nra;
  const TileOrder order(nvt, nra, 32 * bt * st.d * 2);
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
      case 1: proj_tile<KB, KV, 1>(st, op, sm, vt, r0, R); break;
      case 2: proj_tile<KB, KV, 2>(st, op, sm, vt, r0, R); break;
      case 3: proj_tile<KB, KV, 3>(st, op, sm, vt, r0, R); break;
      default: proj_tile<KB, KV, 4>(st, op, sm, vt, r0, R); break;
    }
  }
}

template <int KB>
__global__ __launch_bounds__(THREADS, 2) void k_proj(DevState st) {
  tile_walk<KB, false>(st, GemmOperands{st.wout_t, st.proj_in}, st.S);
}

// KV rows of every expansion of the step: bf16(h . W_kv[l][j]) for the
// L*2*d outputs, the [R,d] x [d, L*2*d] product on the projection's tiles
// and K order (K halves summed apart and added once, so a row's KV values do
// not depend on the rows sharing the step), stored at the candidate's
// (beam, level, rank) place (App. A.2's incremental decoder state).
__global__ __launch_bounds__(THREADS, 2) void k_kv_append(DevState st) {
  tile_walk<4, true>(st, GemmOperands{st.wkv_t, st.hbuf}, st.kv_layers * 2 * st.d / TV);
}

// W_out [V][d] -> MFMA fragment order [S][nk][4 slices][4 pieces][64 lanes][16 B]:
// lane (h, l) of slice s at piece q holds bytes kt*128 + 64h + 16q .. +15 of
// vocabulary row 128*vt + 32s + l (zero past V).
__global__ void k_relayout_wout(const unsigned char *__restrict__ src, unsigned char *__restrict__ dst, int V,
                                int rowbytes, int S) {
  const int nk = rowbytes / CH;
  const size_t pieces = (size_t)S * nk * 4 * 4 * 64;
  for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < pieces; p += (size_t)gridDim.x * blockDim.x) {
    const int ln = (int)(p & 63);
    const int q = (int)((p >> 6) & 3);
    const int s = (int)((p >> 8) & 3);
    const size_t vk = p >> 10;                  // vt * nk + kt
    const int kt = (int)(vk % nk);
    const int vt = (int)(vk / nk);
    const int v = vt * TV + 32 * s + (ln & 31);
    u4 val = {0u, 0u, 0u, 0u};
    if (v < V)
      val = *reinterpret_cast<const u4 *>(src + (size_t)v * rowbytes + (size_t)kt * CH + 64 * (ln >> 5) + 16 * q);
    *reinterpret_cast<u4 *>(dst + p * 16) = val;
  }
}

// W_kv [L][2][d_in][d_out] -> the same fragment order, output feature
// v = plane * d + o (plane = 2l + j) in place of the vocabulary row: lane
// (h, l) of slice s at piece q holds the 8 bf16 values W_kv[plane][k0 + e][o],
// k0 = kt*64 + 32h + 8q, e < 8, of output v = 128*vt + 32s + l.
__global__ void k_relayout_wkv(const uint16_t *__restrict__ W, unsigned char *__restrict__ dst, int d, int NO) {
  const int nk = d * 2 / CH;
  const size_t pieces = (size_t)(NO / TV) * nk * 4 * 4 * 64;
  for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < pieces; p += (size_t)gridDim.x * blockDim.x) {
    const int ln = (int)(p & 63);
    const int q = (int)((p >> 6) & 3);
    const int s = (int)((p >> 8) & 3);
    const size_t vk = p >> 10;
    const int kt = (int)(vk % nk);
    const int vt = (int)(vk / nk);
    const int v = vt * TV + 32 * s + (ln & 31);
    const int plane = v / d, o = v - plane * d;
    const int k0 = kt * (CH / 2) + 32 * (ln >> 5) + 8 * q;
    const uint16_t *src = W + ((size_t)plane * d + k0) * d + o;
    uint16_t e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = src[(size_t)i * d];
    u4 val = {(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16),
              (uint32_t)e[4] | ((uint32_t)e[5] << 16), (uint32_t)e[6] | ((uint32_t)e[7] << 16)};
    *reinterpret_cast<u4 *>(dst + p * 16) = val;
  }
}

}  // namespace

hipError_t launch_relayout_wout(const DevState &st, hipStream_t s) {
  if (st.dtype == 0) return launch_split_wout(st, s);
  const int rowbytes = st.d * 2;
  hipLaunchKernelGGL(k_relayout_wout, dim3(2048), dim3(256), 0, s, static_cast<const unsigned char *>(st.W_out),
                     st.wout_t, st.V, rowbytes, st.S);
  return hipGetLastError();
}

hipError_t launch_proj(const DevState &st, hipStream_t s) {
  if (st.dtype == 0) return launch_proj_split(st, s);
  // Multiple of 8, at most two per compute unit, no more than the 32-row
  // tiles of a full step (a small vocabulary then still spreads a large step
  // over the device).
  const int G = std::max(8, std::min(st.n_cu / 4 * 8, xcd_grid(st.S * ((st.R_max + 31) / 32))));
  switch (st.tile_keys) {
    case 4: hipLaunchKernelGGL((k_proj<4>), dim3(G), dim3(THREADS), 0, s, st); break;
    case 8: hipLaunchKernelGGL((k_proj<8>), dim3(G), dim3(THREADS), 0, s, st); break;
    default: hipLaunchKernelGGL((k_proj<16>), dim3(G), dim3(THREADS), 0, s, st); break;
  }
  return hipGetLastError();
}

hipError_t launch_kv_append(const DevState &st, hipStream_t s) {
  // Sized like the projection's grid, over the L*2*d/128 output tiles.
  const int nvt = st.kv_layers * 2 * st.d / TV;
  const int G = std::max(8, std::min(st.n_cu / 4 * 8, xcd_grid(nvt * ((st.R_max + 31) / 32))));
  hipLaunchKernelGGL(k_kv_append, dim3(G), dim3(THREADS), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_relayout_wkv(const DevState &st, const uint16_t *W_kv, hipStream_t s) {
  hipLaunchKernelGGL(k_relayout_wkv, dim3(2048), dim3(256), 0, s, W_kv, st.wkv_t, st.d, st.kv_layers * 2 * st.d);
  return hipGetLastError();
}

}  // namespace sb
