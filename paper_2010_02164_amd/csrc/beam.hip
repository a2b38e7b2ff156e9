// Row merge, per-beam top-k with pruning and finalization, and the
// backtrack of finished hypotheses.
//
//   K_beam     : per selected beam, merge the projection's per-tile partials
//                of each active parent's row into its log-sum-exp and best k
//                tokens, with log-probabilities lp = z - lse (Sec. 2
//                log-likelihoods); rank the k|V| expansions (only each
//                parent's best k can reach the top k) plus one no-op per
//                terminated candidate, keep the top k (Sec. 2), apply the
//                heuristics H (Sec. 4: relative threshold delta against the
//                best candidate, possibly terminated (App. A.3); at most M
//                kept expansions per parent), mark EOS / max-length
//                terminations, and finish the beam when nothing active
//                survives (App. A.1: terminated candidates stay on the beam
//                and are output once nothing active ranks above them).
//                Continuing beams get their new candidates' states.
//   K_backtrack: rebuild each finished hypothesis's tokens from the
//                backpointer history, one thread per hypothesis.
#include "mfma_common.h"
#include "sb_internal.h"
#include "split_f16.h"
#include "topk.h"
#include "wave.h"

namespace sb {
namespace {

// Maximum of a 64-bit key, in every lane.
template <int S>
__device__ __forceinline__ cand_key max_stage(cand_key x) {
  cand_key a, b;
  stage64<S>(x, a, b);
  return a > b ? a : b;
}
// Over the G lanes of a row (8 or 64).
template <int G>
__device__ __forceinline__ cand_key group_max_key(cand_key x) {
  x = max_stage<0>(x);
  x = max_stage<1>(x);
  x = max_stage<2>(x);
  if constexpr (G == 64) {
    x = max_stage<3>(x);
    x = max_stage<4>(x);
    x = max_stage<5>(x);
  }
  return x;
}

// Log-sum-exp combine of (max, sum exp) pairs over the G lanes of a row;
// every lane ends with the same result. The merge is not symmetric in its operands once
// the compiler fuses a product into the sum, so both lanes of a pair take
// them in the same order: the lower lane's first (the swap stages 4 and 5
// already hand both lanes the pair in that order).
template <int S>
__device__ __forceinline__ void lse_stage(float &m, float &s) {
  uint32_t ma, mb, sa, sb;
  stage32<S>(__float_as_uint(m), ma, mb);
  stage32<S>(__float_as_uint(s), sa, sb);
  if constexpr (S <= 3) {
    const int lane = (int)(threadIdx.x & 63);
    const bool lower = S == 0 ? !(lane & 1) : S == 1 ? !(lane & 2) : S == 2 ? (lane & 7) < 4 : (lane & 15) < 8;
    if (!lower) {
      const uint32_t tm = ma, ts = sa;
      ma = mb;
      sa = sb;
      mb = tm;
      sb = ts;
    }
  }
  float M = __uint_as_float(ma), Sm = __uint_as_float(sa);
  lse_merge(M, Sm, __uint_as_float(mb), __uint_as_float(sb));
  m = M;
  s = Sm;
}
template <int G>
__device__ __forceinline__ void group_lse(float &m, float &s) {
  lse_stage<0>(m, s);
  lse_stage<1>(m, s);
  lse_stage<2>(m, s);
  if constexpr (G == 64) {
    lse_stage<3>(m, s);
    lse_stage<4>(m, s);
    lse_stage<5>(m, s);
  }
}

// The logits of a 32-row slice s of vocabulary tile vt for one row, recomputed
// by the projection's own MFMA sequence so that they equal its logits bit for
// bit (the MFMA's internal rounding is not modelled, it is replayed). Every
// column of the MFMA gets the row's state, so all 32 columns hold the same
// logits. The loops are unrolled no further than the registers of the rest of
// the row merge reach: few tiles come here.
constexpr int W_FRAG = 1024;   // bytes of a wave-wide fragment of W_out

// fp32: the split products chunk by chunk, then the row scales.
__device__ __forceinline__ f16v recompute_slice_f32(const DevState &st, int row, int vt, int s, int lane) {
  const int nch = st.d / SPLIT_K;
  const u4 *x = reinterpret_cast<const u4 *>(st.hsplit + split_state_off(st.d, row, 8 * (lane >> 5)));
  const u4 *a = reinterpret_cast<const u4 *>(st.wout_t + (size_t)(vt * 4 + s) * nch * SPLIT_CHUNK) + lane;
  f16v tot = {};
#pragma unroll 1
  for (int c = 0; c < nch; ++c) {
    f16v cross = {};
#pragma unroll 2
    for (int i = 0; i < 4; ++i, a += 2 * W_FRAG / 16, x += 2 * W_FRAG / 16) split_step(a[0], a[64], x[0], x[64], tot, cross);
    split_flush(cross, tot);
  }
  const int slice = vt * 4 + s, nfar = st.w_nfar[slice];
  f16v z = SplitScale(st.w_scale + 32 * slice + 4 * (lane >> 5)).apply(tot);
  if (nfar > 0) {
    const uint32_t at = (uint32_t)row * (uint32_t)st.d;
    add_far<1>(st.w_far + (size_t)slice * SPLIT_FAR, nfar, lane >> 5, static_cast<const float *>(st.proj_in), &at, &z);
  }
  return z;
}

// Logit z[v] of one row where the projection took it on the fp32 MFMA,
// which adds its two products to the sum one after the other, lane half 0's
// first: K halves in chunks of 32 values, per chunk the products of k and
// k + 16, then the halves added.
__device__ __forceinline__ float recompute_logit_fp32(const DevState &st, int row, int v) {
  const int d = st.d;
  const float *w = static_cast<const float *>(st.W_out) + (size_t)v * d;
  const float *x = static_cast<const float *>(st.proj_in) + (size_t)row * d;
  float first = 0.0f, acc = 0.0f;
#pragma unroll 1
  for (int c = 0; c < d; c += 32) {
    if (c == d / 2) {
      first = acc;
      acc = 0.0f;
    }
#pragma unroll 4
    for (int i = 0; i < 16; ++i) {
      acc = fmaf(w[c + i], x[c + i], acc);
      acc = fmaf(w[c + i + 16], x[c + i + 16], acc);
    }
  }
  return first + acc;
}

// bf16: each K half accumulated chunk by chunk and piece by piece, then the
// halves added once.
__device__ __forceinline__ f16v recompute_slice_bf16(const DevState &st, int row, int vt, int s, int lane) {
  constexpr int CH = 128;
  const int nk = st.d * 2 / CH, nh = nk >> 1;
  const unsigned char *x = static_cast<const unsigned char *>(st.proj_in) + (size_t)row * st.d * 2 + 64 * (lane >> 5);
  const unsigned char *a = st.wout_t + ((size_t)vt * nk * 4 + s) * 4 * W_FRAG + lane * 16;
  f16v first = {}, acc = {};
#pragma unroll 1
  for (int c = 0; c < nk; ++c, a += 16 * W_FRAG, x += CH) {
    if (c == nh) {
      first = acc;
      acc = f16v{};
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u4 av = *reinterpret_cast<const u4 *>(a + q * W_FRAG);
      const u4 bv = *reinterpret_cast<const u4 *>(x + 16 * q);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, av), __builtin_bit_cast(bf8, bv), acc, 0, 0,
                                                    0);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) first[r] += acc[r];
  return first;
}

// The keys of the tile's 128 logits, to LDS.
__device__ __forceinline__ void recompute_tile(const DevState &st, int row, int vt, int lane, cand_key *keys) {
  const int h = lane >> 5, l32 = lane & 31;
  const float bias = st.beta * (float)(st.r_t[row] - st.r_Lx[row]);
  if (st.dtype == 0 && (split_tile_fp32(st, vt) || split_row_fp32(st, row))) {
#pragma unroll 1
    for (int i = lane; i < 128; i += 64) {
      const int v = vt * 128 + i;
      float x = v < st.V ? recompute_logit_fp32(st, row, v) : 0.0f;
      if (v == 0) x += bias;
      keys[i] = v < st.V ? make_key(x, v) : 0ull;
    }
    return;
  }
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    f16v z;
    if (st.dtype == 1) z = recompute_slice_bf16(st, row, vt, s, lane);
    else z = recompute_slice_f32(st, row, vt, s, lane);
    // Lane (h, l) with l < 16: register l, vocabulary row 8 (l / 4) + 4h + l % 4 of the slice.
    float x = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (r == l32) x = z[r];
    const int i = 32 * s + 8 * (l32 >> 2) + 4 * h + (l32 & 3), v = vt * 128 + i;
    if (v == 0) x += bias;
    if (l32 < 16) keys[i] = v < st.V ? make_key(x, v) : 0ull;
  }
}

// The k best of the row's kept keys, from the records themselves: the largest
// key below the last one drawn, k times. Lane r < k receives the key of rank r;
// returns the k-th.
__device__ __forceinline__ cand_key draw_records(const float *base, int S, int lane, int k, cand_key &mine) {
  constexpr int PW = part_width(TILE_KEYS_SHORT);
  cand_key last = ~0ull;
#pragma unroll 1
  for (int r = 0; r < k; ++r) {
    cand_key best = 0ull;
#pragma unroll 1
    for (int t = lane; t < S; t += 64) {
      TopK<TILE_KEYS_SHORT> o;
      topk_load(o, base + (size_t)t * PW + 2);
#pragma unroll
      for (int j = 0; j < TILE_KEYS_SHORT; ++j) best = o.k[j] < last && o.k[j] > best ? o.k[j] : best;
    }
    last = group_max_key<64>(best);
    if (lane == r) mine = last;
  }
  return last;
}

// Merge the per-tile partials of one row by G lanes (a wave, or 8 lanes when
// there are at most 8 tiles; `lane` counts within them). Each lane folds the
// tiles lane, lane+G, ... into (max, sum exp) and a sorted best-KB list
// (loads issued a batch at a time before they are folded). The row's
// log-sum-exp is combined over the lanes and taken from lane 0; the row's k
// best keys are drawn in k rounds of a maximum over the lists' heads,
// the lane holding the winner dropping it (keys are distinct: they carry
// the token). Lane r < k receives the key of rank r.
//
// A tile record keeps its TK best keys (TK <= KB). With full lists, TK = KB >= k,
// the k keys drawn are the row's best. With short ones, if a tile's last kept
// key ranks above the k-th key drawn, the tile may hold further keys of the
// best k (rare: TK of the row's best k - 1 in one 128-token tile; at most
// (k - 1) / TK tiles, as all their kept keys rank above it): such tiles are
// recomputed from W_out one by one, and each time the k best drawn from the
// tile's logits and the keys drawn before. Any other tile's unkept keys rank below its last kept key, so
// at most at the k-th key drawn, and more candidates can only raise the k-th.
// A lane's list is 8 keys for every k > 4 there (a lane rarely holds more than
// 8 of a row's best 16); where a lane's 8th key ranks above the k-th drawn, the
// k kept keys are first drawn again from the records.
template <int KB, int TK, int G>
__device__ __forceinline__ double merge_row(const DevState &st, int row, int lane, int k, cand_key *sat_keys,
                                            cand_key &mine) {
  constexpr int PW = part_width(TK);
  constexpr int LB = TK == TILE_KEYS_SHORT && KB > 8 ? 8 : KB;   // keys of a lane's list
  // Partials in flight per lane (full-length lists come with fewer than 64
  // tiles, one per lane).
  constexpr int NBT = TK == TILE_KEYS_SHORT && G == 64 ? 4 : 1;
  const float *base = st.part + (size_t)row * st.S * PW;
  float m = -INFINITY, s = 0.0f;
  TopK<LB> tk;
  topk_init(tk);
  cand_key last_max = 0ull;   // largest last kept key over the lane's tiles
#pragma unroll 1
  for (int t0 = lane; t0 < st.S; t0 += G * NBT) {
    float rec[NBT][PW];
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
      const int t = min(t0 + G * u, st.S - 1);
      const uint4 *p = reinterpret_cast<const uint4 *>(base + (size_t)t * PW);
#pragma unroll
      for (int x = 0; x < PW / 4; ++x) {
        const uint4 v = p[x];
        rec[u][4 * x] = __uint_as_float(v.x);
        rec[u][4 * x + 1] = __uint_as_float(v.y);
        rec[u][4 * x + 2] = __uint_as_float(v.z);
        rec[u][4 * x + 3] = __uint_as_float(v.w);
      }
    }
    if constexpr (TK == TILE_KEYS_SHORT && NBT == 4) {
      // Four sorted 4-key runs (empty past the last tile) merged by
      // bitonic networks into the batch's best KB, then into the list.
      TopK<4> run[4];
#pragma unroll
      for (int u = 0; u < NBT; ++u) {
        const bool ok = t0 + G * u < st.S;
        topk_load(run[u], rec[u] + 2);
#pragma unroll
        for (int j = 0; j < 4; ++j) run[u].k[j] = ok ? run[u].k[j] : 0ull;
        if (ok) lse_merge(m, s, rec[u][0], rec[u][1]);
        last_max = run[u].k[3] > last_max ? run[u].k[3] : last_max;
      }
      TopK<LB> batch;
      if constexpr (LB == 4) {
        topk_merge(run[0], run[1]);
        topk_merge(run[2], run[3]);
        topk_merge(run[0], run[2]);
        batch = run[0];
      } else {
        cand_key a8[8], b8[8];
        merge_sorted<4>(run[0].k, run[1].k, a8);
        merge_sorted<4>(run[2].k, run[3].k, b8);
        TopK<8> x, y;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          x.k[j] = a8[j];
          y.k[j] = b8[j];
        }
        topk_merge(x, y);
        batch = x;
      }
      if (t0 == lane) tk = batch;
      else topk_merge(tk, batch);
    } else {
#pragma unroll
      for (int u = 0; u < NBT; ++u) {
        if (t0 + G * u < st.S) {
          TopK<TK> t4;
          topk_load(t4, rec[u] + 2);
          TopK<LB> o;
          topk_init(o);
#pragma unroll
          for (int j = 0; j < TK; ++j) o.k[j] = t4.k[j];
          lse_merge(m, s, rec[u][0], rec[u][1]);
          last_max = t4.k[TK - 1] > last_max ? t4.k[TK - 1] : last_max;
          topk_merge(tk, o);
        }
      }
    }
  }
  group_lse<G>(m, s);
  const cand_key lane_last = LB < KB ? tk.k[LB - 1] : 0ull;
  cand_key kth = 0ull;
  mine = 0ull;
#pragma unroll 1
  for (int r = 0; r < k; ++r) {
    const cand_key best = group_max_key<G>(tk.k[0]);
    if (lane == r) mine = best;
    kth = best;
    if (tk.k[0] == best) {
#pragma unroll
      for (int j = 0; j + 1 < LB; ++j) tk.k[j] = tk.k[j + 1];
      tk.k[LB - 1] = 0ull;
    }
  }
  // The row's log-sum-exp as lane 0 has it, for every lane.
  const double lse = __shfl((double)m + log((double)s), 0, G);
  if constexpr (TK >= KB) return lse;
  else {
    static_assert(G == 64 && TK == TILE_KEYS_SHORT, "short lists come with 64 or more tiles");
    // Expected, so that the rare code stands behind the kernel's own: between the
    // rows' merges it cost 0.4 of 12.2 us (|V| = 32000, 128 beams of 5).
    if (__builtin_expect(__ballot(last_max > kth || lane_last > kth) == 0ull, 1)) return lse;
    if (__ballot(lane_last > kth)) kth = draw_records(base, st.S, lane, k, mine);
    if (lane >= k) mine = 0ull;
#pragma unroll 1
    for (int t0 = 0; t0 < st.S; t0 += 64) {
      const int t = t0 + lane;
      TopK<TK> o;
      topk_load(o, base + (size_t)min(t, st.S - 1) * PW + 2);
      unsigned long long mask = __ballot(t < st.S && o.k[TK - 1] > kth);
      if (lane == 0 && mask)
        atomicAdd(reinterpret_cast<unsigned long long *>(&st.ctrl->tile_recomputes),
                  (unsigned long long)__popcll(mask));
#pragma unroll 1
      for (; mask; mask &= mask - 1) {
        const int vt = t0 + __ffsll((long long)mask) - 1;
        recompute_tile(st, row, vt, lane, sat_keys);
        if (key_idx(mine) >> 7 == vt) mine = 0ull;   // among the recomputed
        // The wave's own writes, read by its other lanes.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const cand_key x = sat_keys[lane], y = sat_keys[lane + 64];
        cand_key drawn = 0ull, last = ~0ull;
#pragma unroll 1
        for (int r = 0; r < k; ++r) {
          cand_key best = mine < last ? mine : 0ull;
          best = x < last && x > best ? x : best;
          best = y < last && y > best ? y : best;
          last = group_max_key<64>(best);
          if (lane == r) drawn = last;
        }
        mine = drawn;
      }
    }
    return lse;
  }
}

// Row merge as its own kernel (wave per row), for the single-expansion
// debug entry point: writes lse and the k best log-probabilities/tokens.
template <int KB, int TK>
__global__ __launch_bounds__(256) void k_rowmerge(DevState st) {
  const int R = st.ctrl->R;
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= R) return;
  cand_key mine;
  const int k = st.k;
  __shared__ cand_key sat_keys[TK < KB ? 4 : 1][TK < KB ? 128 : 1];
  const double lse = merge_row<KB, TK, 64>(st, row, lane, k, sat_keys[TK < KB ? threadIdx.x >> 6 : 0], mine);
  if (lane == 0) st.r_lse[row] = lse;
  if (lane < k) {
    st.top_lp[(size_t)row * k + lane] = (double)key_val(mine) - lse;
    st.top_tok[(size_t)row * k + lane] = key_idx(mine);
  }
}

// Ranking of an expansion: higher score first, then the smaller secondary
// key (parent rank << 24 | token + 1; a no-op has token -1).
__device__ __forceinline__ bool ranks_above(double sa, int ka, double sb, int kb) {
  return sa > sb || (sa == sb && ka < kb);
}

// Threads of a beam workgroup, at least one per candidate of the ranking (k *
// (k + 1) of them):
//  - up to 8 vocabulary tiles and k <= 7: one wave, 8 lanes per parent row, so
//    that a beam takes one wave slot and its steps no barrier (|V| = 256, 2048
//    records, k = 5: 24.0 us with 4 waves, 10.9 with one; |V| = 1000, 8 records, k = 4: 8.7 and
//    6.8);
//  - up to 8 tiles, k <= 15: 4 waves, a wave per parent row;
//  - else 8 waves, a wave per parent row.
constexpr int BEAM_THREADS = 512;
constexpr int BEAM_THREADS_SMALL = 256;
constexpr int BEAM_THREADS_WAVE = 64;
constexpr int NO_KEY = 0x7FFFFFFF;

// A candidate expansion of the per-beam ranking (16 bytes, one LDS read).
struct Cand {
  double score;
  int key, pad;
};

template <int KB, int TK, int NT>
__global__ __launch_bounds__(NT) void k_beam(DevState st) {
  constexpr int G = NT == BEAM_THREADS_WAVE ? 8 : 64;                       // lanes per parent row
  constexpr int T1 = NT > 64 ? 64 : 0, T2 = NT > 128 ? 128 : 0;             // threads with work of their own
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int k = st.k;
  const int base = b * k;
  const bool fairseq = st.rule == 1;
  const int KC = k + (fairseq ? 1 : 0);   // children drawn per parent
  // Everything the beam needs from its records is loaded in one round,
  // before the selection flag is tested.
  const int row0 = st.b_row0[b];
  const uint32_t active = st.b_mask[b] & 0xFFFFu;
  int my_status = SLOT_EMPTY;
  double my_score = 0.0;
  if (tid < k) {
    my_status = st.s_status[base + tid];
    my_score = st.s_score[base + tid];
  }
  int my_q = 0, my_t = 0, my_ml = 0, my_nout = 0;
  if (tid == T1) {
    my_q = st.b_input[b];
    my_t = st.b_steps[b] + 1;     // 1-based index of the emitted token
    my_ml = st.b_ml[b];
    my_nout = st.b_nout[b];
  }
  // The KV ancestry buffer holding this beam's current ranks (read before
  // thread 0 flips the parity at the end of the step).
  const int apar = st.kv_layers > 0 ? st.b_par[b] : 0;
  if (row0 < 0) return;   // not expanded (every beam when nothing is live)
  __shared__ int sl_status[KMAX_SUPPORTED], sl_row[KMAX_SUPPORTED];
  __shared__ double sl_score[KMAX_SUPPORTED];
  __shared__ int q_in_sh, t_sh, max_len_sh, nout_sh;
  // Best KC log-probabilities and tokens of each active parent's row.
  __shared__ double ch_lp[KMAX_SUPPORTED * KMAX_SUPPORTED];
  __shared__ int ch_tok[KMAX_SUPPORTED * KMAX_SUPPORTED];
  // The new beam, in rank order, and (Fairseq rule) this step's outputs.
  __shared__ double nscore[KMAX_SUPPORTED], oscore[KMAX_SUPPORTED];
  __shared__ int npar[KMAX_SUPPORTED], ntok[KMAX_SUPPORTED], nstat[KMAX_SUPPORTED];
  __shared__ int opar[KMAX_SUPPORTED], otok[KMAX_SUPPORTED], ostat[KMAX_SUPPORTED];
  __shared__ int nw_sh, nact_sh, no_sh;
  // Recomputed keys of a row merge's rare case, per wave.
  __shared__ cand_key sat_keys[TK < KB ? NT / 64 : 1][TK < KB ? 128 : 1];
  // Candidates (at most k KC list entries + k no-ops) and the ranks kept.
  __shared__ Cand cand[KMAX_SUPPORTED * (KMAX_SUPPORTED + 1)];
  __shared__ double r_score[2 * KMAX_SUPPORTED];
  __shared__ int r_key[2 * KMAX_SUPPORTED];
  if (tid < k) {
    sl_status[tid] = my_status;
    sl_row[tid] = row0 + __popc(active & ((1u << tid) - 1u));   // of an active candidate
    sl_score[tid] = my_score;
  }
  if (tid == T1) {
    q_in_sh = my_q;
    t_sh = my_t;
    max_len_sh = my_ml;
    nout_sh = my_nout;
  }
  __syncthreads();
  const int q_in = q_in_sh, t = t_sh, max_len = max_len_sh, nout0 = nout_sh;

  // Row merge of every active parent: wave w takes parents w, w + NT / 64, ...,
  // or all of them 8 lanes each.
  for (int par = tid / G; par < k; par += NT / G) {
    if (sl_status[par] != SLOT_ACTIVE) continue;
    const int gl = lane % G;
    cand_key mine;
    const double lse = merge_row<KB, TK, G>(st, sl_row[par], gl, KC, sat_keys[TK < KB ? wave : 0], mine);
    if (gl < KC) {
      ch_lp[par * KC + gl] = (double)key_val(mine) - lse;
      ch_tok[par * KC + gl] = key_idx(mine);
    }
  }
  __syncthreads();

  // Ranking of all expansions (key: score, parent rank, token; Sec. 2):
  // thread c < C holds candidate c (parent c / KC's child c % KC, or, paper
  // rule, the no-op of terminated parent c - k KC); a candidate's rank is
  // the count of candidates that rank above it, all keys being distinct.
  // Ranks below RM (k, or 2k under the Fairseq rule) are kept.
  const int NCL = k * KC;
  const int C = NCL + (fairseq ? 0 : k);
  const int RM = fairseq ? 2 * k : k;
  double cs = -INFINITY;
  int ck = NO_KEY;
  bool cv = false;
  if (tid < NCL) {
    const int p = tid / KC, j = tid - p * KC;
    if (sl_status[p] == SLOT_ACTIVE) {
      const int tok = ch_tok[p * KC + j];
      if (tok >= 0 && tok < st.V) {
        cs = sl_score[p] + ch_lp[p * KC + j];
        ck = (p << 24) | (tok + 1);
        cv = true;
      }
    }
  } else if (tid < C) {
    const int p = tid - NCL;
    if (sl_status[p] == SLOT_EOS || sl_status[p] == SLOT_MAXLEN) {
      cs = sl_score[p];
      ck = p << 24;
      cv = true;
    }
  }
  // Records up to a multiple of 8; invalid ones (score -inf) rank below
  // every valid candidate.
  const int C8 = (C + 7) & ~7;
  if (tid < C8) cand[tid] = Cand{cs, ck, 0};
  const int nvalid = __syncthreads_count(cv);
  if constexpr (NT == BEAM_THREADS) {
    // CP threads per candidate (as many as there are, up to 16) compare it with
    // every CP-th of the others and add up.
    const int CP = NT >= 16 * C8 ? 16 : NT >= 8 * C8 ? 8 : NT >= 4 * C8 ? 4 : NT >= 2 * C8 ? 2 : 1;
    if (tid < CP * C8) {
      const int me = tid / CP, part = tid - me * CP;
      const Cand mine = cand[me];
      int rank = 0;
      for (int c0 = part; c0 < C8; c0 += 8 * CP) {
        Cand o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) o[u] = cand[min(c0 + u * CP, C8 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += c0 + u * CP < C8 && ranks_above(o[u].score, o[u].key, mine.score, mine.key) ? 1 : 0;
      }
      if (CP > 1) rank += (int)dpp_partner<0>((uint32_t)rank);
      if (CP > 2) rank += (int)dpp_partner<1>((uint32_t)rank);
      if (CP > 4) rank += (int)dpp_partner<2>((uint32_t)rank);
      if (CP > 8) rank += (int)dpp_partner<3>((uint32_t)rank);
      if (part == 0 && mine.key != NO_KEY && rank < RM) {
        r_score[rank] = mine.score;
        r_key[rank] = mine.key;
      }
    }
  } else {
    if (cv) {
      int rank = 0;
      for (int c0 = 0; c0 < C8; c0 += 8) {
        Cand o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) o[u] = cand[c0 + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += ranks_above(o[u].score, o[u].key, cs, ck) ? 1 : 0;
      }
      if (rank < RM) {
        r_score[rank] = cs;
        r_key[rank] = ck;
      }
    }
  }
  __syncthreads();

  if (wave == 0) {
    // Lane r < nfull holds the expansion of rank r.
    const int nfull = min(RM, nvalid);
    double rs = -INFINITY;
    int rk = NO_KEY;
    if (lane < nfull) {
      rs = r_score[lane];
      rk = r_key[lane];
    }
    if (!fairseq) {
      // Heuristics H (Sec. 4) on B' in rank order: drop x if
      // score(x) < best - delta, best = B'[0] (possibly terminated,
      // App. A.3); drop an expansion whose parent already has M kept
      // expansions (no-ops exempt). A parent's kept expansions before rank r
      // are its first M delta-survivors, so the M test needs only their count.
      const double ref = __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(__double_as_longlong(rs) >> 32), 0) << 32) |
                                              (uint32_t)__builtin_amdgcn_readlane((int)__double_as_longlong(rs), 0));
      const int rpar = rk >> 24, rtok = (rk & 0xFFFFFF) - 1;
      const bool keepd = lane < nfull && !(rs < ref - st.delta);
      int before = 0;
#pragma unroll 1
      for (int o = 0; o < nfull; ++o) {
        const int okk = __builtin_amdgcn_readlane(rk, o);
        const int okeep = __builtin_amdgcn_readlane((int)keepd, o);
        before += (o < lane && okeep && (okk >> 24) == rpar && (okk & 0xFFFFFF) != 0);
      }
      const bool kept = keepd && (rtok < 0 || before < st.M);
      int status = SLOT_EMPTY;
      if (kept) {
        if (rtok < 0) status = sl_status[rpar];                   // no-op keeps EOS / MAXLEN
        else status = rtok == 0 ? SLOT_EOS : (t == max_len ? SLOT_MAXLEN : SLOT_ACTIVE);
      }
      const unsigned long long km = __ballot(kept);
      const unsigned long long am = __ballot(kept && status == SLOT_ACTIVE);
      if (kept) {
        const int nr = __popcll(km & ((1ull << lane) - 1ull));
        nscore[nr] = rs;
        npar[nr] = rpar;
        ntok[nr] = rtok;
        nstat[nr] = status;
      }
      if (lane == 0) {
        nw_sh = __popcll(km);
        nact_sh = __popcll(am);
        no_sh = 0;
      }
    } else {
      // Fairseq rule (App. A.1): a terminated expansion among the best k is
      // output at once (until k outputs); the new beam is the first k
      // active expansions in rank order. Both lie within the first 2k ranks.
      const int rpar = rk >> 24, rtok = (rk & 0xFFFFFF) - 1;
      const bool valid = lane < nfull;
      const bool term = valid && (rtok == 0 || t == max_len);
      const unsigned long long below = (1ull << lane) - 1ull;
      const unsigned long long tm = __ballot(term && lane < k);
      const int f = __popcll(tm & below);
      const bool out = term && lane < k && nout0 + f < k;
      const unsigned long long act = __ballot(valid && !term);
      const int nr = __popcll(act & below);
      const bool inbeam = valid && !term && nr < k;
      if (out) {
        oscore[f] = rs;
        opar[f] = rpar;
        otok[f] = rtok;
        ostat[f] = rtok == 0 ? SLOT_EOS : SLOT_MAXLEN;
      }
      if (inbeam) {
        nscore[nr] = rs;
        npar[nr] = rpar;
        ntok[nr] = rtok;
        nstat[nr] = SLOT_ACTIVE;
      }
      if (lane == 0) {
        const int nw = min(k, __popcll(act));
        const int no = min(__popcll(tm), k - nout0);
        nw_sh = nw;
        no_sh = no;
        // The input finishes with k outputs, or when nothing active is left.
        nact_sh = (nout0 + no >= k) ? 0 : nw;
      }
    }
  }
  __syncthreads();
  const int w = nw_sh, no = no_sh;
  const bool ends = nact_sh == 0;
  const int fin = ends ? (int)st.ctrl->timesteps : 0;

  // History: backpointers of level t, indexed by the input's queue position:
  // the new beam at positions 0..w-1, this step's outputs at k + f.
  uint32_t *bprow = st.bp + ((size_t)q_in * st.max_len_cap + (t - 1)) * st.bpw;
  if (tid < w && !(fairseq && ends)) {
    const uint32_t tokbits = ntok[tid] < 0 ? BP_NOOP : (uint32_t)ntok[tid];
    bprow[tid] = ((uint32_t)npar[tid] << 24) | tokbits;
  }
  if (fairseq && tid >= T1 && tid < T1 + no) {
    const int f = tid - T1;
    bprow[k + f] = ((uint32_t)opar[f] << 24) | (uint32_t)otok[f];
    OutHyp h;
    h.score = oscore[f];
    h.length = 0;
    h.status = ostat[f];
    h.finalize_step = fin;
    h.level = t;
    h.pos = k + f;
    h.pad = 0;
    st.o_hyp[(size_t)q_in * k + nout0 + f] = h;
  }

  if (ends) {
    int total;
    if (!fairseq) {
      // Y[i] = the survivors in rank order; tokens are rebuilt later.
      total = w;
      if (tid < w) {
        OutHyp h;
        h.score = nscore[tid];
        h.length = 0;
        h.status = nstat[tid];
        h.finalize_step = fin;
        h.level = t;
        h.pos = tid;
        h.pad = 0;
        st.o_hyp[(size_t)q_in * k + tid] = h;
      }
    } else {
      // Y[i] = the outputs in the order they were finalized; those of
      // earlier steps get the finishing timestep too.
      total = nout0 + no;
      if (tid >= T2 && tid < T2 + nout0) st.o_hyp[(size_t)q_in * k + (tid - T2)].finalize_step = fin;
    }
    if (tid < k) {
      st.s_status[base + tid] = SLOT_EMPTY;
    }
    if (tid == 0) {
      st.o_count[q_in] = total;
      st.b_input[b] = -1;
      atomicAdd(reinterpret_cast<unsigned long long *>(&st.ctrl->hyps), (unsigned long long)total);
      atomicAdd(reinterpret_cast<unsigned long long *>(&st.ctrl->finished), 1ull);
    }
    return;
  }

  // Continue: write the new beam into ranks 0..w-1 (no-ops keep their
  // state; active children take their parent's new state h).
  if (tid < k) {
    if (tid < w) {
      st.s_status[base + tid] = nstat[tid];
      st.s_score[base + tid] = nscore[tid];
      if (ntok[tid] >= 0) st.s_tok[base + tid] = ntok[tid];
    } else {
      st.s_status[base + tid] = SLOT_EMPTY;
    }
  }
  if (wave == 0) {
    const int status = lane < w ? nstat[lane] : SLOT_EMPTY;
    const unsigned long long am = __ballot(status == SLOT_ACTIVE), tm = __ballot(status > SLOT_ACTIVE);
    if (lane == 0) st.b_mask[b] = (uint32_t)am | (uint32_t)tm << 16;
  }
  if (tid == 0) {
    st.b_steps[b] = t;
    st.b_par[b] ^= 1;
    st.b_nout[b] = nout0 + no;
  }
  // State copy: s_h[rank] <- hbuf[row(parent)] for every active survivor, with
  // the digit planes and list of the exact bf16 recurrence.
  if constexpr (NT == BEAM_THREADS) {
    // A thread takes one 16-byte chunk of several survivors (spread over
    // groups of threads when a state has fewer chunks than the workgroup
    // threads) and loads them all, without branches, before it stores the
    // first: 128 beams, |V| = 32000, bf16, k = 10: 22.8 -> 21.6 us per
    // timestep. Beams of one wave lose by it (k = 4: 7.1 -> 7.8 us).
    const int hch = st.d * (st.dtype == 1 ? 2 : 4) / 16;
    const int dch = st.rec_i8 ? (int)(rec_dig_row_bytes(st.d) / 16) : 0, ach = st.rec_i8 ? (int)(sizeof(RowAux) / 16) : 0;
    const int tot = hch + dch + ach;
    const int groups = max(1, NT / tot), grp = groups > 1 ? tid / tot : 0;
    constexpr int U = 8;
    if (grp < groups) {
      for (int c = tid - grp * tot; c < tot; c += groups > 1 ? tot : NT) {
        const uint4 *src;
        uint4 *dst;
        int ch;   // chunks per row of this array
        if (c < hch) {
          src = static_cast<const uint4 *>(st.hbuf) + c;
          dst = static_cast<uint4 *>(st.s_h) + c;
          ch = hch;
        } else if (c < hch + dch) {
          src = reinterpret_cast<const uint4 *>(st.hd) + (c - hch);
          dst = reinterpret_cast<uint4 *>(st.s_hd) + (c - hch);
          ch = dch;
        } else {
          src = reinterpret_cast<const uint4 *>(st.haux) + (c - hch - dch);
          dst = reinterpret_cast<uint4 *>(st.s_haux) + (c - hch - dch);
          ch = ach;
        }
        for (int r0 = grp; r0 < w; r0 += U * groups) {
          uint4 v[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int r = min(r0 + u * groups, w - 1);
            v[u] = nstat[r] == SLOT_ACTIVE ? src[(size_t)sl_row[npar[r]] * ch] : uint4{0u, 0u, 0u, 0u};
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int r = r0 + u * groups;
            if (r < w && nstat[r] == SLOT_ACTIVE) dst[(size_t)(base + r) * ch] = v[u];
          }
        }
      }
    }
  } else {
    const int rowbytes = st.d * (st.dtype == 1 ? 2 : 4);
    const int chunks = rowbytes / 16;
    const uint4 *__restrict__ hb = static_cast<const uint4 *>(st.hbuf);
    uint4 *__restrict__ sh = static_cast<uint4 *>(st.s_h);
    const int total = w * chunks;
    for (int x = tid; x < total; x += NT) {
      const int r = x / chunks, c = x - r * chunks;
      if (nstat[r] == SLOT_ACTIVE) sh[(size_t)(base + r) * chunks + c] = hb[(size_t)sl_row[npar[r]] * chunks + c];
    }
    // The state's digit planes and list, for the exact bf16 recurrence.
    if (st.rec_i8) {
      const int dch = (int)(rec_dig_row_bytes(st.d) / 16), ach = (int)(sizeof(RowAux) / 16), tch = dch + ach;
      const uint4 *__restrict__ hd = reinterpret_cast<const uint4 *>(st.hd);
      uint4 *__restrict__ shd = reinterpret_cast<uint4 *>(st.s_hd);
      const uint4 *__restrict__ ha = reinterpret_cast<const uint4 *>(st.haux);
      uint4 *__restrict__ sha = reinterpret_cast<uint4 *>(st.s_haux);
      for (int x = tid; x < w * tch; x += NT) {
        const int r = x / tch, c = x - r * tch;
        if (nstat[r] != SLOT_ACTIVE) continue;
        const size_t src = sl_row[npar[r]];
        if (c < dch) shd[(size_t)(base + r) * dch + c] = hd[src * dch + c];
        else sha[(size_t)(base + r) * ach + (c - dch)] = ha[src * ach + (c - dch)];
      }
    }
  }
  // KV state: an active child's ancestors are its parent's (levels 0 .. t-2)
  // and the parent itself (level t-1), copied into the other buffer as
  // 4-byte words; the word holding level t-1 is built by one thread.
  if (st.kv_layers > 0) {
    const int A4 = st.anc_stride / 4;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(st.anc) + ((size_t)apar * st.n * k + base) * A4;
    uint32_t *dst = reinterpret_cast<uint32_t *>(st.anc) + ((size_t)(apar ^ 1) * st.n * k + base) * A4;
    const int nw = (t - 1) / 4 + 1, last = (t - 1) / 4, sh8 = ((t - 1) & 3) * 8;
    for (int x = tid; x < w * nw; x += NT) {
      const int r = x / nw, wi = x - r * nw;
      if (nstat[r] != SLOT_ACTIVE) continue;
      uint32_t v = src[(size_t)npar[r] * A4 + wi];
      if (wi == last) v = (v & ~(0xFFu << sh8)) | ((uint32_t)npar[r] << sh8);
      dst[(size_t)r * A4 + wi] = v;
    }
  }
}

// One thread per (input, rank): walk the backpointers from the final level
// down to 1, skipping no-op levels, and write the tokens in order.
__global__ __launch_bounds__(256) void k_backtrack(DevState st, int q0, int q1) {
  const int k = st.k;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long q = q0 + gid / k;
  const int rank = (int)(gid % k);
  if (q >= q1) return;
  if (rank >= st.o_count[q]) return;
  OutHyp *h = st.o_hyp + (size_t)q * k + rank;
  const int bpw = st.bpw;
  const uint32_t *bp = st.bp + (size_t)q * st.max_len_cap * bpw;
  const int top = min(h->level, st.max_len_cap);
  const int pos0 = min(max(h->pos, 0), bpw - 1);
  int pos = pos0, len = 0;
  for (int lev = top; lev >= 1; --lev) {
    const uint32_t e = bp[(size_t)(lev - 1) * bpw + pos];
    len += (e & 0xFFFFFFu) != BP_NOOP;
    pos = min((int)(e >> 24), k - 1);
  }
  int32_t *out = st.o_tok + ((size_t)q * k + rank) * st.max_len_cap;
  pos = pos0;
  int idx = len;
  for (int lev = top; lev >= 1; --lev) {
    const uint32_t e = bp[(size_t)(lev - 1) * bpw + pos];
    const uint32_t tok = e & 0xFFFFFFu;
    if (tok != BP_NOOP) out[--idx] = (int32_t)tok;
    pos = min((int)(e >> 24), k - 1);
  }
  h->length = len;
}

// Collect: copy the tokens of the hypotheses of inputs [q0, q1) from their
// padded rows to their places in the packed buffer (offsets set by the
// host; -1 marks a rank the input does not have). Four hypotheses per
// workgroup, one wave each, lanes striding over the tokens.
__global__ __launch_bounds__(256) void k_pack(DevState st, int q0, int q1) {
  const long long hyp = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (hyp >= (long long)(q1 - q0) * st.k) return;
  const long long off = st.o_off[hyp];
  if (off < 0) return;
  const size_t slot = (size_t)q0 * st.k + hyp;
  const int len = min(st.o_hyp[slot].length, st.max_len_cap);
  const int32_t *src = st.o_tok + slot * st.max_len_cap;
  for (int j = lane; j < len; j += 64) st.o_pack[off + j] = src[j];
}

}  // namespace

hipError_t launch_rowmerge(const DevState &st, hipStream_t s) {
  const int G = (st.R_max + 3) / 4;
  const bool sh = st.tile_keys == TILE_KEYS_SHORT;
  switch (st.kbucket) {
    case 4: hipLaunchKernelGGL((k_rowmerge<4, 4>), dim3(G), dim3(256), 0, s, st); break;
    case 8:
      if (sh) hipLaunchKernelGGL((k_rowmerge<8, 4>), dim3(G), dim3(256), 0, s, st);
      else hipLaunchKernelGGL((k_rowmerge<8, 8>), dim3(G), dim3(256), 0, s, st);
      break;
    default:
      if (sh) hipLaunchKernelGGL((k_rowmerge<16, 4>), dim3(G), dim3(256), 0, s, st);
      else hipLaunchKernelGGL((k_rowmerge<16, 16>), dim3(G), dim3(256), 0, s, st);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_beam(const DevState &st, hipStream_t s) {
  const bool sh = st.tile_keys == TILE_KEYS_SHORT;
  const bool small = st.S <= 8 && st.k <= 15, wave = st.S <= 8 && st.k <= 7;
#define SB_BEAM_NT(KB, TK, NT) hipLaunchKernelGGL((k_beam<KB, TK, NT>), dim3(st.n), dim3(NT), 0, s, st)
#define SB_BEAM(KB, TK)                                                            \
  do {                                                                             \
    if constexpr (KB <= 8 && TK == KB) {                                           \
      if (wave) {                                                                  \
        SB_BEAM_NT(KB, TK, BEAM_THREADS_WAVE);                                     \
        break;                                                                     \
      }                                                                            \
    }                                                                              \
    if constexpr (TK == KB) {                                                      \
      if (small) {                                                                 \
        SB_BEAM_NT(KB, TK, BEAM_THREADS_SMALL);                                    \
        break;                                                                     \
      }                                                                            \
    }                                                                              \
    SB_BEAM_NT(KB, TK, BEAM_THREADS);                                              \
  } while (0)
  switch (st.kbucket) {
    case 4: SB_BEAM(4, 4); break;
    case 8:
      if (sh) SB_BEAM(8, 4);
      else SB_BEAM(8, 8);
      break;
    default:
      if (sh) SB_BEAM(16, 4);
      else SB_BEAM(16, 16);
      break;
  }
#undef SB_BEAM
#undef SB_BEAM_NT
  return hipGetLastError();
}

hipError_t launch_pack(const DevState &st, int q0, int q1, hipStream_t s) {
  if (q1 <= q0) return hipSuccess;
  const long long hyps = (long long)(q1 - q0) * st.k;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)((hyps + 3) / 4)), dim3(256), 0, s, st, q0, q1);
  return hipGetLastError();
}

hipError_t launch_backtrack(const DevState &st, int q0, int q1, hipStream_t s) {
  if (q1 <= q0) return hipSuccess;
  const long long total = (long long)(q1 - q0) * st.k;
  hipLaunchKernelGGL(k_backtrack, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, st, q0, q1);
  return hipGetLastError();
}

}  // namespace sb
