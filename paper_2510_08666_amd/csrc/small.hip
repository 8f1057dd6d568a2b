// The non-GEMM kernels of the step: token bookkeeping, embedding, expert-output combine (both also leave the
// row's 1/rms for the next consumer), ballot-based token->expert permutation, LM-head partial merge, threshold commit,
// and the KV import / export used by tests.
#include "gemm.hpp"
#include "kernels.hpp"
#include "routing.hpp"

namespace dinfer {

static thread_local const int32_t* t_live_word = nullptr;
void set_live_word(const int32_t* d_live) { t_live_word = d_live; }
const int32_t* live_word() { return t_live_word; }
static bool g_single_slice = false;
void set_single_slice(bool on) { g_single_slice = on; }
bool single_slice() { return g_single_slice; }

// ---------------------------------------------------------------- rotary table
// cos / sin of pos * theta^(-2j/hd), computed in double on the device and stored as float.
__global__ void rope_table_kernel(float* __restrict__ cos_tab, float* __restrict__ sin_tab, int max_pos, int head_dim,
                                  float theta) {
  const int half = head_dim / 2;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)max_pos * half) return;
  const int pos = (int)(i / half), j = (int)(i % half);
  const double ang = (double)pos * pow((double)theta, -2.0 * j / head_dim);
  cos_tab[i] = (float)cos(ang);
  sin_tab[i] = (float)sin(ang);
}
void launch_rope_table(float* cos_tab, float* sin_tab, int max_pos, int head_dim, float theta, hipStream_t st) {
  const int64_t n = (int64_t)max_pos * (head_dim / 2);
  rope_table_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(cos_tab, sin_tab, max_pos, head_dim, theta);
}

// ---------------------------------------------------------------- token bookkeeping
// `limit` = positions a sequence may use (rotary table and page-table row); a prefix length that would
// leave it is pulled back so that no later kernel indexes outside its buffers.
// Runs in one workgroup (the extra one of the embedding launch), token by token: sequence by sequence, each behind the
// loads of its offset and base, the launch took as long as its sequences (hidden 2048, 60 of 32 tokens 23.5 us, 16 of them
// 7.5; now 10.0 and 5.6).
__device__ inline void token_meta(const SeqSpan& span, const int32_t* __restrict__ d_base, int limit,
                                  int32_t* __restrict__ tok_seq, int32_t* __restrict__ tok_pos,
                                  int32_t* __restrict__ seq_nkeys, int32_t* __restrict__ qtile) {
  __shared__ int32_t s_off[MAX_SEQS + 1], s_base[MAX_SEQS], s_tile[MAX_SEQS];
  static_assert(MAX_SEQS <= WAVE, "one lane per sequence");
  const int n_seq = span.n_seq;
  if (threadIdx.x < WAVE) {
    const int s = min((int)threadIdx.x, n_seq - 1), o = span.off[s], len = span.off[s + 1] - o;
    const int base = d_base ? max(0, min(d_base[s], limit - len)) : 0, tiles = (len + TILE - 1) / TILE;
    int incl = (int)threadIdx.x < n_seq ? tiles : 0;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
      const int up = __shfl_up(incl, d, WAVE);
      if ((int)threadIdx.x >= d) incl += up;
    }
    if ((int)threadIdx.x < n_seq) {
      s_off[s] = o;
      s_base[s] = base;
      s_tile[s] = incl - tiles;
      seq_nkeys[s] = base + len;
      if (s == n_seq - 1) s_off[n_seq] = o + len;
    }
  }
  __syncthreads();
  const int T = s_off[n_seq];
  for (int i = threadIdx.x; i < T; i += blockDim.x) {
    int s = 0;                                  // the last sequence that begins at or before token i
#pragma unroll
    for (int step = MAX_SEQS / 2; step > 0; step >>= 1)
      if (s + step < n_seq && s_off[s + step] <= i) s += step;
    const int at = i - s_off[s];
    tok_seq[i] = s;
    tok_pos[i] = s_base[s] + at;
    if (at % TILE == 0) {
      int32_t* q = qtile + (s_tile[s] + at / TILE) * 3;
      q[0] = s;
      q[1] = i;
      q[2] = min(TILE, s_off[s + 1] - i);
    }
  }
}

// ---------------------------------------------------------------- RMSNorm helpers
constexpr int NORM_THREADS = 256;

__device__ inline float block_sum_256(float v, float* sh) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[wave] = v;
  __syncthreads();
  const float r = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return r;
}

// x[t] = emb[token[t]];  ssq[t] = sum(x[t]^2);  xn[t] = planes of x[t] * gain.  Workgroup T, one past the tokens,
// writes the token bookkeeping of the forward instead (nothing here reads it): one launch less per forward.
// Bound by its traffic (a row read, the float32 row and its planes written): a thread takes four consecutive columns
// at a time (hidden is a multiple of 64), since element by element the 2-byte plane stores fill the store path
// (4287 rows of 2048: 39 us).
template <typename E>
__global__ __launch_bounds__(NORM_THREADS) void embed_kernel(const int32_t* __restrict__ tokens, const E* __restrict__ emb,
                                                             int H, int V, float* __restrict__ x,
                                                             float* __restrict__ ssq, const float* __restrict__ gain,
                                                             E* __restrict__ xn, int T, SmoothIn sm, SeqSpan span,
                                                             const int32_t* __restrict__ d_base, int limit,
                                                             int32_t* __restrict__ tok_seq, int32_t* __restrict__ tok_pos,
                                                             int32_t* __restrict__ seq_nkeys, int32_t* __restrict__ qtile,
                                                             const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  __shared__ float sh[4];
  const int t = blockIdx.x;
  if (t == T) {
    token_meta(span, d_base, limit, tok_seq, tok_pos, seq_nkeys, qtile);
    return;
  }
  const E* row = emb + (int64_t)min(max(tokens[t], 0), V - 1) * H;
  // iteration smoothing: a still-masked position adds alpha times what the previous iteration retained for it
  const bool smooth = sm.delta && ((sm.mask[t / sm.block_len] >> (t % sm.block_len)) & 1ull);
  float ss = 0.f;
#pragma unroll 2
  for (int c = 4 * threadIdx.x; c < H; c += 4 * NORM_THREADS) {
    f32x4 v = load_elems4<E>(row + c);
    const f32x4 g = *reinterpret_cast<const f32x4*>(gain + c);
    f32x4 n;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (smooth) v[i] += sm.alpha * sm.delta[(int64_t)t * H + c + i];
      n[i] = v[i] * g[i];
      ss += v[i] * v[i];
    }
    *reinterpret_cast<f32x4*>(x + (int64_t)t * H + c) = v;
    store_actk4<E>(xn, T, t, c, n);
  }
  ss = block_sum_256(ss, sh);
  if (threadIdx.x == 0) ssq[t] = ss;
}
void launch_embed(bool bf16, const int32_t* tokens, const void* emb, int T, int H, int V, float* x,
                  float* ssq, const float* gain, void* xn, const SmoothIn* smooth, const SeqSpan& span,
                  const int32_t* d_base, int limit, int32_t* tok_seq, int32_t* tok_pos, int32_t* seq_nkeys,
                  int32_t* qtile, hipStream_t st) {
  const SmoothIn sm = smooth ? *smooth : SmoothIn{nullptr, 0.f, nullptr, 1};
  if (bf16)
    embed_kernel<bf16_t><<<T + 1, NORM_THREADS, 0, st>>>(tokens, (const bf16_t*)emb, H, V, x, ssq, gain, (bf16_t*)xn, T, sm,
                                                         span, d_base, limit, tok_seq, tok_pos, seq_nkeys, qtile, live_word());
  else
    embed_kernel<float><<<T + 1, NORM_THREADS, 0, st>>>(tokens, (const float*)emb, H, V, x, ssq, gain, (float*)xn, T, sm,
                                                        span, d_base, limit, tok_seq, tok_pos, seq_nkeys, qtile, live_word());
}

// ---------------------------------------------------------------- iteration smoothing: probabilities
// p[t][v] = exp(z[t][v] - max_t) / sum_t as a k-major activation matrix [T][Kpad] (zero past the vocabulary):
// the B operand of the expected-embedding contraction.  Bound by its 2 x 4 * T * V bytes of traffic: neighbouring
// threads take the quads of one token and k-step, then the next token, so that a wave stores one contiguous piece; it
// reads 128 bytes (two k-steps) of every row.
template <typename E>
__global__ __launch_bounds__(256) void prob_planes_kernel(const float* __restrict__ logits, const float* __restrict__ stats,
                                                           int T, int V, int Kpad, E* __restrict__ probs,
                                                           const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  constexpr int KS = ET<E>::KS, Q = KS / 4, U = 32 / KS;   // U k-steps = 128 bytes of logits
  const int64_t n = (int64_t)(Kpad / (KS * U)) * T * Q;
  const bool aligned = V % 4 == 0;                          // rows of logits start on 16-byte boundaries
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int quad = (int)(i % Q), t = (int)(i / Q % T);
    const int v0 = (int)(i / (Q * T)) * (KS * U) + quad * 4;
    const float m = stats[2 * t], inv = 1.f / stats[2 * t + 1];
    const float* row = logits + (int64_t)t * V;
    f32x4 z[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * KS;
      if (aligned && v + 4 <= V) {
        z[u] = *reinterpret_cast<const f32x4*>(row + v);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) z[u][e] = v + e < V ? row[v + e] : -INFINITY;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      f32x4 p;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = __expf(z[u][e] - m) * inv;
      store_actk4<E>(probs, T, t, v0 + u * KS, p);
    }
  }
}
void launch_prob_planes(bool bf16, const float* logits, const float* stats, int T, int V, int Kpad, void* probs,
                        hipStream_t st) {
  const int64_t threads = (int64_t)(Kpad / 32) * T * (bf16 ? 4 : 2);
  const unsigned grid = (unsigned)(threads / 256 + 1 < 8192 ? threads / 256 + 1 : 8192);
  if (bf16) prob_planes_kernel<bf16_t><<<grid, 256, 0, st>>>(logits, stats, T, V, Kpad, (bf16_t*)probs, live_word());
  else prob_planes_kernel<float><<<grid, 256, 0, st>>>(logits, stats, T, V, Kpad, (float*)probs, live_word());
}

// x[t] += sum_j w[t][j] * O[t*k+j]  (j ascending: a fixed summation order);  ssq[t] = sum of squares and the
// normalised-input planes of the new row.  (Forwards of more than 32 tokens; smaller ones fold this into the down
// projection.)
// A thread takes four columns, so that all loads of a row are under way at once (with 256 threads that took the 1024-column
// chunks one after the other 8.4 us at 64 tokens and 10.7 at 512, now 5.4 and 9.0).  The sum of squares keeps the order of those
// chunks: the threads past 256 hand their columns down.
template <typename E>
__global__ __launch_bounds__(MAX_HIDDEN / 4) void combine_kernel(float* __restrict__ x, const float* __restrict__ O,
                                                                 const float* __restrict__ topk_w, int top_k,
                                                                 int H, float* __restrict__ ssq,
                                                                 const float* __restrict__ gain, E* __restrict__ xn,
                                                                 E* __restrict__ xn_hi, int T, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  __shared__ float sh[4];
  __shared__ f32x4 s_acc[MAX_HIDDEN / 4 - NORM_THREADS];
  const int t = blockIdx.x, col = 4 * threadIdx.x;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (col < H) {
    const float* orow = O + (int64_t)t * top_k * H + col;
    const f32x4 xr = *reinterpret_cast<const f32x4*>(x + (int64_t)t * H + col);
    const f32x4 g = *reinterpret_cast<const f32x4*>(gain + col);
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j)
      if (j < top_k) {
        const float w = topk_w[t * top_k + j];
        const f32x4 o = *reinterpret_cast<const f32x4*>(orow + (int64_t)j * H);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += w * o[i];
      }
    f32x4 n;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[i] += xr[i];
      n[i] = acc[i] * g[i];
    }
    *reinterpret_cast<f32x4*>(x + (int64_t)t * H + col) = acc;
    store_actk4<E>(xn, T, t, col, n);
    if constexpr (Planes<E>::N > 1)
      if (xn_hi) store_elems4<E>(xn_hi + ((int64_t)(col / ET<E>::KS) * T + t) * ET<E>::KS + col % ET<E>::KS, n);
    if (threadIdx.x >= NORM_THREADS) s_acc[threadIdx.x - NORM_THREADS] = acc;
  }
  __syncthreads();
  float ss = 0.f;
  if (threadIdx.x < NORM_THREADS) {
#pragma unroll
    for (int i = 0; i < 4; ++i) ss += acc[i] * acc[i];
    for (int c = NORM_THREADS + threadIdx.x; 4 * c < H; c += NORM_THREADS) {
      const f32x4 a = s_acc[c - NORM_THREADS];
#pragma unroll
      for (int i = 0; i < 4; ++i) ss += a[i] * a[i];
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  }
  __syncthreads();
  if (threadIdx.x == 0) ssq[t] = sh[0] + sh[1] + sh[2] + sh[3];
}
void launch_combine(bool bf16, float* x, const float* O, const float* topk_w, int top_k,
                    int T, int H, float* ssq, const float* gain, void* xn, hipStream_t st, void* xn_hi) {
  const int threads = H / 4 <= NORM_THREADS ? NORM_THREADS : (H / 4 + WAVE - 1) / WAVE * WAVE;
  if (bf16)
    combine_kernel<bf16_t><<<T, threads, 0, st>>>(x, O, topk_w, top_k, H, ssq, gain, (bf16_t*)xn, (bf16_t*)xn_hi, T, live_word());
  else
    combine_kernel<float><<<T, threads, 0, st>>>(x, O, topk_w, top_k, H, ssq, gain, (float*)xn, nullptr, T, live_word());
}

// Half a row's k-step (eight elements, 16 bytes) per thread; a test hook's kernel.
__global__ __launch_bounds__(256) void high_plane_kernel(const bf16_t* __restrict__ xn, int64_t n, bf16_t* __restrict__ xn_hi) {
  constexpr int KS = ET<bf16_t>::KS, NP = Planes<bf16_t>::N;
  static_assert(KS == 16, "two threads per k-step of a row");
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) *reinterpret_cast<bf16x8*>(xn_hi + i * 8) = *reinterpret_cast<const bf16x8*>(xn + (i >> 1) * (NP * KS) + (i & 1) * 8);
}
void launch_high_plane(const void* xn, int T, int H, void* xn_hi, hipStream_t st) {
  const int64_t n = (int64_t)T * (H / 8);
  high_plane_kernel<<<(int)((n + 255) / 256), 256, 0, st>>>((const bf16_t*)xn, n, (bf16_t*)xn_hi);
}

// ---------------------------------------------------------------- token -> expert permutation
// More than 64 tokens (below, the expert kernels sort the pairs for themselves: routing.hpp).  Stable counting
// sort of the (token, slot) pairs by expert.  The router's workgroups have left the histogram of their tokens,
// hist[n_hist][MAX_EXPERTS], `hists` of them for 32 tokens; workgroup g of this launch, which takes 32 tokens, adds up those before its own and all of them, which
// gives the place of its first pair of every expert, and places its group's pairs: a wave takes 64 consecutive pairs
// (a chunk) and forms the ballots "which lanes go to expert e" for all experts at once by OR-ing lane bits into its own
// 64 LDS words; the population of ballot e is the chunk's count for e, the bits below a lane in its expert's ballot
// the pair's rank inside the chunk.  Workgroup 0 also writes the tables.  A few dependent round trips, whatever the
// number of pairs (a single workgroup over all pairs: 41 us for 34296 of them, 9 for 4096, 6 for 1280).
constexpr int PERMUTE_WAVES = 4;
static_assert(TILE * MAX_TOPK <= PERMUTE_WAVES * WAVE, "a group's pairs are at most one chunk per wave");
__global__ __launch_bounds__(PERMUTE_WAVES * WAVE) void permute_kernel(const int32_t* __restrict__ expert_of_pair, int n_pairs, int pairs_per_group,
                                                        const int32_t* __restrict__ hist, int n_hist, int hists, int n_exp,
                                                        int32_t* __restrict__ cnt, int32_t* __restrict__ off,
                                                        int32_t* __restrict__ perm,
                                                        int32_t* __restrict__ work, int group_tiles, int round,
                                                        const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  __shared__ unsigned long long s_ballot[PERMUTE_WAVES * MAX_EXPERTS];
  __shared__ int32_t s_before[PERMUTE_WAVES * MAX_EXPERTS], s_total[PERMUTE_WAVES * MAX_EXPERTS], s_first[MAX_EXPERTS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, group = blockIdx.x;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int in_group = wave * WAVE + lane, p = group * pairs_per_group + in_group;
  const int e = in_group < pairs_per_group && p < n_pairs ? expert_of_pair[p] : -1;
  {
    int before = 0, total = 0;                              // lane = expert
#pragma unroll 8
    for (int g = wave; g < n_hist; g += PERMUTE_WAVES) {
      const int n = hist[g * MAX_EXPERTS + lane];
      total += n;
      before += g < group * hists ? n : 0;
    }
    s_before[wave * MAX_EXPERTS + lane] = before;
    s_total[wave * MAX_EXPERTS + lane] = total;
    s_ballot[wave * MAX_EXPERTS + lane] = 0ull;
  }
  __syncthreads();
  if (e >= 0) atomicOr(&s_ballot[wave * MAX_EXPERTS + e], 1ull << lane);
  if (wave == 0) {
    int tot = 0, mine = 0;
#pragma unroll
    for (int w = 0; w < PERMUTE_WAVES; ++w) {
      tot += s_total[w * MAX_EXPERTS + lane];
      mine += s_before[w * MAX_EXPERTS + lane];
    }
    if (lane >= n_exp) tot = 0;
    int incl = tot;                                         // inclusive scan over the lanes (experts)
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int up = __shfl_up(incl, o, WAVE);
      if (lane >= o) incl += up;
    }
    s_first[lane] = incl - tot + mine;
    if (group == 0) {
      if (lane < n_exp) {
        cnt[lane] = tot;
        off[lane] = incl - tot;
        if (lane == n_exp - 1) off[n_exp] = incl;
      }
      const uint64_t has_rows = __ballot(tot > 0);
      if (lane == 0) {
        off[STAT_ACTIVE_SUM] += __popcll(has_rows);
        off[STAT_PERMUTATIONS] += 1;
      }
      // Work list of the many-token expert GEMMs: one item per (expert, group of up to group_tiles 32-row tiles), the
      // groups with the most tiles first, so that the long ones start first.
      const int rows_per = group_tiles * TILE, full = tot / rows_per, rem = tot % rows_per, rem_tiles = (rem + TILE - 1) / TILE;
      int4* items = reinterpret_cast<int4*>(work + WORK_ITEMS);
      const int start = incl - tot;
      int at = 0, light = 0, heavy = 0;                     // items so far; of them with one or two tiles, with the most
      for (int k = group_tiles; k >= 1; --k) {
        const int mine_k = (k == group_tiles ? full : 0) + (rem_tiles == k ? 1 : 0);
        int incl_k = mine_k;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
          const int up = __shfl_up(incl_k, o, WAVE);
          if (lane >= o) incl_k += up;
        }
        const int first = at + incl_k - mine_k, n_k = __shfl(incl_k, WAVE - 1, WAVE);
        if (k == group_tiles)
          for (int g = 0; g < full; ++g) items[first + g] = make_int4(lane, start + g * rows_per, rows_per, 0);
        if (rem_tiles == k) items[first + mine_k - 1] = make_int4(lane, start + full * rows_per, rem, 0);
        at += n_k;
        if (k <= 2) light += n_k;
        if (k == group_tiles) heavy = n_k;
      }
      if (lane == 0) {
        work[WORK_BIG] = at - expert_piece_items(at, light, round);
        work[WORK_ALL] = at;
        work[WORK_HEAVY] = heavy;
        work[WORK_LIGHT] = light;
      }
    }
  }
  __syncthreads();
  if (e >= 0) {
    int r = s_first[e] + __popcll(s_ballot[wave * MAX_EXPERTS + e] & below);
    for (int w = 0; w < wave; ++w) r += __popcll(s_ballot[w * MAX_EXPERTS + e]);
    perm[r] = p;
  }
}
// The bound that the interface states for a context (dinfer_workspace_bytes); counts and positions are 32-bit and the grid of
// the expert GEMMs grows with a 128th of the pairs, so the kernels themselves do not need it.
constexpr int PERMUTE_MAX_PAIRS = 65535;
int permute_max_pairs() { return PERMUTE_MAX_PAIRS; }
void launch_permute(const int32_t* topk_idx, int n_pairs, int top_k, const int32_t* hist, int hist_tokens, int E, int32_t* cnt,
                    int32_t* off, int32_t* perm, int32_t* work, int group_tiles, int round, hipStream_t st) {
  const int per_group = TILE * top_k;
  permute_kernel<<<(n_pairs + per_group - 1) / per_group, PERMUTE_WAVES * WAVE, 0, st>>>(
      topk_idx, n_pairs, per_group, hist, (n_pairs / top_k + hist_tokens - 1) / hist_tokens, TILE / hist_tokens, E, cnt, off, perm, work, group_tiles, round, live_word());
}

// The tables of permute_kernel for at most 64 tokens, where no kernel of a forward needs them; a test hook's kernel, one wave.  It
// puts them together from what the expert kernels read off the routing: PairIds with N pairs in a lane, expert by expert, and up to 32
// tokens also TokenExperts, from which a second permutation is made; an entry in which the two differ is -1.
template <int N>
__global__ __launch_bounds__(WAVE) void pair_tables_kernel(const int32_t* __restrict__ topk_idx, int T, int top_k, int n_exp, int32_t* __restrict__ cnt,
                                                           int32_t* __restrict__ off, int32_t* __restrict__ perm) {
  constexpr int PAIRS = N * WAVE;
  __shared__ int32_t s_pair[WAVE], s_cnt[MAX_EXPERTS], s_perm[PAIRS], s_other[PAIRS];
  const int lane = threadIdx.x, n_pairs = T * top_k;
  for (int p = lane; p < PAIRS; p += WAVE) s_perm[p] = s_other[p] = -1;
  s_cnt[lane] = 0;
  PairIds<N> ids;
  ids.load(topk_idx, n_pairs);
  const uint64_t experts = ids.experts();
  bool same = true;
  for (int i = 0; i < __popcll(experts); ++i) {
    __syncthreads();
    const int4 it = ids.rows_of(nth_bit(experts, i), s_pair);
    __syncthreads();
    if (lane < it.z && it.y + lane < n_pairs) s_perm[it.y + lane] = s_pair[lane];
    if (lane == 0 && it.x < n_exp) {
      s_cnt[it.x] = it.z;
      off[it.x] = it.y;
    }
  }
  if constexpr (N * WAVE == TILE * MAX_TOPK) {
    TokenExperts tokens;
    tokens.load(topk_idx, T, top_k);
    same = tokens.experts() == experts;
    for (int e = 0; e < n_exp; ++e) {
      const int row = tokens.row_of(e);
      for (int j = 0; j < top_k; ++j)
        if (lane < TILE && row >= 0 && row < n_pairs && topk_idx[lane * top_k + j] == e) s_other[row] = lane * top_k + j;
    }
  }
  __syncthreads();
  if constexpr (N * WAVE != TILE * MAX_TOPK)
    for (int p = lane; p < PAIRS; p += WAVE) s_other[p] = s_perm[p];
  for (int p = lane; p < n_pairs; p += WAVE) perm[p] = same && s_perm[p] == s_other[p] ? s_perm[p] : -1;
  int at = 0;
  for (int i = 0; i < lane; ++i) at += s_cnt[i];
  if (lane < n_exp) {
    cnt[lane] = s_cnt[lane];
    if (!(experts >> lane & 1)) off[lane] = at;               // without rows: nothing says where
    if (lane == n_exp - 1) off[n_exp] = at + s_cnt[lane];
  }
}
void launch_pair_tables(const int32_t* topk_idx, int T, int top_k, int E, int32_t* cnt, int32_t* off, int32_t* perm, hipStream_t st) {
  if (T <= TILE) pair_tables_kernel<TILE * MAX_TOPK / WAVE><<<1, WAVE, 0, st>>>(topk_idx, T, top_k, E, cnt, off, perm);
  else pair_tables_kernel<2 * TILE * MAX_TOPK / WAVE><<<1, WAVE, 0, st>>>(topk_idx, T, top_k, E, cnt, off, perm);
}

// ---------------------------------------------------------------- LM-head partial merge
// One workgroup per token row over the LmStat partials of the LM head's workgroups (lm_combine), fixed tree ->
// deterministic.  The partials of a row lie next to each other: part[token][n_parts].
__global__ __launch_bounds__(256) void lm_merge_kernel(const f32x4* __restrict__ part, int n_parts,
                                                        float* __restrict__ conf, int32_t* __restrict__ argmax,
                                                        float* __restrict__ stats, const uint64_t* __restrict__ mask,
                                                        int block_len, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  __shared__ LmStat sh[4];
  const int t = blockIdx.x;
  if (mask && !((mask[t / block_len] >> (t % block_len)) & 1ull)) return;   // a decided position: nothing was computed
  LmStat a{-INFINITY, 0.f, 0x7fffffff};
  // the loads of up to U rounds (64 registers) are issued together, those past the end of the row not at all: round by round,
  // each behind a memory round trip, 2456 partials took 7.2 us at 160 tokens, now 5.6
  constexpr int U = 16;
  for (int w0 = threadIdx.x; w0 < n_parts; w0 += U * 256) {
    f32x4 p[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (w0 + u * 256 < n_parts) p[u] = part[(int64_t)t * n_parts + w0 + u * 256];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (w0 + u * 256 < n_parts) a = lm_combine(a, LmStat{p[u][0], p[u][1], __float_as_int(p[u][2])});
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    LmStat b{__shfl_xor(a.m, o, WAVE), __shfl_xor(a.s, o, WAVE), __shfl_xor(a.id, o, WAVE)};
    a = lm_combine(a, b);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    a = lm_combine(lm_combine(sh[0], sh[1]), lm_combine(sh[2], sh[3]));
    conf[t] = 1.f / a.s;
    argmax[t] = a.id;
    if (stats) {            // the row's largest logit and sum exp(z - max): what a later correction of the softmax needs
      stats[2 * t] = a.m;
      stats[2 * t + 1] = a.s;
    }
  }
}
void launch_lm_merge(const float* part, int n_parts, int T, float* conf, int32_t* argmax, float* stats,
                     hipStream_t st, const uint64_t* mask, int block_len) {
  lm_merge_kernel<<<T, 256, 0, st>>>((const f32x4*)part, n_parts, conf, argmax, stats, mask, block_len, live_word());
}

// Row list of the LM head when only undecided positions are wanted: lane s counts the set bits of sequence s,
// a scan over the lanes gives its offset, and it lists its positions in ascending order.
__global__ __launch_bounds__(64) void lm_rows_kernel(const uint64_t* __restrict__ mask, int n_seq, int block_len,
                                                      int32_t* __restrict__ rows, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  const int lane = threadIdx.x;
  const uint64_t keep = block_len >= 64 ? ~0ull : ((1ull << block_len) - 1);
  uint64_t m = lane < n_seq ? mask[lane] & keep : 0ull;
  const int n = __popcll(m);
  int incl = n;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const int up = __shfl_up(incl, o, WAVE);
    if (lane >= o) incl += up;
  }
  int at = 1 + incl - n;
  while (m) {
    const int pos = __ffsll((unsigned long long)m) - 1;
    rows[at++] = lane * block_len + pos;
    m &= m - 1;
  }
  if (lane == WAVE - 1) rows[0] = incl;
}
void launch_lm_rows(const uint64_t* mask, int n_seq, int block_len, int32_t* rows, hipStream_t st) {
  lm_rows_kernel<<<1, WAVE, 0, st>>>(mask, n_seq, block_len, rows, live_word());
}

// ---------------------------------------------------------------- decoder: credit decoding
// Credits are sparse: a (position, token) pair can only ever hold credit if the token was the position's top-1
// candidate at some step, so a position keeps a short list of (token id, credit).  Fusing alpha*log(1 + credit) into
// the logits then changes only the listed logits of the row, and the enhanced softmax follows from the row's plain
// (max, sum exp) by exchanging those few terms -- for which the listed logits are recomputed here as dot products
// of the row's normalised-input planes with the listed rows of the packed LM head.  One workgroup per position.
template <typename E>
__global__ __launch_bounds__(256) void credit_kernel(const E* __restrict__ W, const E* __restrict__ xn,
                                                      RowNorm norm, int T, int H, int V, float scale,
                                                      const float* __restrict__ stats, const uint64_t* __restrict__ mask,
                                                      int block_len, float alpha, float beta, float gamma,
                                                      int32_t* __restrict__ cred_ids, float* __restrict__ cred_val,
                                                      int32_t* __restrict__ cred_n, float* __restrict__ conf,
                                                      int32_t* __restrict__ argmax) {
  typedef typename ET<E>::vec vec;
  constexpr int G = ET<E>::G, KS = ET<E>::KS, NP = Planes<E>::N;
  __shared__ int32_t s_ids[CREDIT_CAP];
  __shared__ float s_val[CREDIT_CAP], s_z[CREDIT_CAP];
  __shared__ int32_t s_n;
  const int row = blockIdx.x, seq = row / block_len, pos = row % block_len;
  if (!((mask[seq] >> pos) & 1ull)) return;            // decided positions keep their plain values
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float M = stats[2 * row], S = stats[2 * row + 1];
  const int v_top = argmax[row];
  const float p_top = conf[row];
  if (wave == 0) {
    // equation 1: discount every credit, reward the current top-1 candidate with p^gamma
    int n = cred_n[row];
    n = min(max(n, 0), CREDIT_CAP);
    int id = lane < n ? cred_ids[(int64_t)row * CREDIT_CAP + lane] : -1;
    float val = lane < n ? cred_val[(int64_t)row * CREDIT_CAP + lane] * beta : INFINITY;
    const float reward = powf(p_top, gamma);
    const uint64_t hit = __ballot(lane < n && id == v_top);
    int slot;
    if (hit) {
      slot = __ffsll((unsigned long long)hit) - 1;
      if (lane == slot) val += reward;
    } else {
      if (n < CREDIT_CAP) {
        slot = n++;
      } else {                                          // list full: the smallest credit makes room
        const float smallest = -wave_max(-val);
        slot = __ffsll((unsigned long long)__ballot(val == smallest)) - 1;
      }
      if (lane == slot) {
        id = v_top;
        val = reward;
      }
    }
    if (lane < n) {
      cred_ids[(int64_t)row * CREDIT_CAP + lane] = id;
      cred_val[(int64_t)row * CREDIT_CAP + lane] = val;
      s_ids[lane] = id;
      s_val[lane] = val;
    }
    if (lane == 0) {
      cred_n[row] = n;
      s_n = n;
    }
  }
  __syncthreads();
  const int n = s_n;
  const int ksteps = H / KS;
  const float zs = row_rinv(norm.ssq, norm.n_ssq, T, row, H, norm.eps) * scale;
  // an id outside the vocabulary (a row of NaN has no candidate and leaves one in the list) is no row of the LM head
  auto listed = [&](int k) { return (unsigned)s_ids[k] < (unsigned)V; };
  for (int k = wave; k < n; k += 4) {
    if (!listed(k)) continue;
    const int v = s_ids[k];
    float z;
    if (v == v_top) {
      z = M;                                           // exactly the value the plain sum was built around
    } else {
      const int task = v / (2 * TILE), which = (v / TILE) & 1, r = v % TILE;
      float acc = 0.f;
      for (int j = lane; j < H / G; j += WAVE) {       // one 16-byte chunk of the row per lane and round
        const int k0 = j * G, ks = k0 / KS, h = (k0 % KS) / G;
        const vec wv = load16<E>(W + ((((int64_t)task * ksteps + ks) * 2 + which) * WAVE + h * TILE + r) * G);
        const E* xp = xn + act_index<E>(T, row, k0);
        const vec hi = load16<E>(xp);
#pragma unroll
        for (int e = 0; e < G; ++e) {
          float x = to_f32(hi[e]);
          if (NP == 2) x += to_f32(xp[KS + e]);
          acc += to_f32(wv[e]) * x;
        }
      }
      z = wave_sum(acc) * zs;
    }
    if (lane == 0) s_z[k] = z;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    // equation 2 on the listed logits; every other term of the softmax is unchanged
    float Mt = M;
    for (int k = 0; k < n; ++k)
      if (listed(k)) Mt = fmaxf(Mt, s_z[k] + alpha * log1pf(s_val[k]));
    float St = S * __expf(M - Mt);
    int best = 0x7fffffff;
    for (int k = 0; k < n; ++k) {
      if (!listed(k)) continue;
      const float zt = s_z[k] + alpha * log1pf(s_val[k]);
      St += __expf(zt - Mt) - __expf(s_z[k] - Mt);
      if (zt == Mt && s_ids[k] < best) best = s_ids[k];
    }
    conf[row] = 1.f / St;
    argmax[row] = best;
  }
}
void launch_credit(bool bf16, const void* w_lm, const void* xn, RowNorm norm, int T, int H, int V, float scale,
                   const float* stats, const uint64_t* mask, int block_len, float alpha, float beta, float gamma,
                   int32_t* cred_ids, float* cred_val, int32_t* cred_n, float* conf, int32_t* argmax, hipStream_t st) {
  if (bf16)
    credit_kernel<bf16_t><<<T, 256, 0, st>>>((const bf16_t*)w_lm, (const bf16_t*)xn, norm, T, H, V, scale, stats, mask,
                                             block_len, alpha, beta, gamma, cred_ids, cred_val, cred_n, conf, argmax);
  else
    credit_kernel<float><<<T, 256, 0, st>>>((const float*)w_lm, (const float*)xn, norm, T, H, V, scale, stats, mask,
                                            block_len, alpha, beta, gamma, cred_ids, cred_val, cred_n, conf, argmax);
}

// ---------------------------------------------------------------- decoder: threshold commit
// One wavefront per sequence, lane = block position.  The set of lanes to commit is a 64-bit ballot.
// conf / argmax hold one row per forward token: position i of sequence s is row s*row_stride + row_off + i (the
// rows before row_off are the neighbours a vicinity-refresh forward carries along).  When conf_out / argmax_out
// are given, the block's values are also stored compactly as [sequence][block_len].
__global__ __launch_bounds__(64) void commit_kernel(const float* __restrict__ conf, const int32_t* __restrict__ argmax,
                                                     int block_len, int row_stride, int row_off,
                                                     int32_t* __restrict__ tokens, uint64_t* __restrict__ mask,
                                                     CommitRule rule, int32_t* __restrict__ n_committed,
                                                     float* __restrict__ conf_out, int32_t* __restrict__ argmax_out,
                                                     int32_t* __restrict__ next_live, int32_t* __restrict__ steps,
                                                     const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  __shared__ float conf_of[64];
  const float threshold = rule.threshold;
  const int fixed_k = rule.fixed_k;
  const int s = blockIdx.x, lane = threadIdx.x;
  const uint64_t old = mask[s] & (block_len >= 64 ? ~0ull : ((1ull << block_len) - 1));
  const bool masked = lane < block_len && ((old >> lane) & 1ull);
  const int row = s * row_stride + row_off + lane;
  const float c = lane < block_len ? conf[row] : -1.f;
  const int am = lane < block_len ? argmax[row] : 0;
  if (conf_out && lane < block_len) {
    conf_out[s * block_len + lane] = c;
    argmax_out[s * block_len + lane] = am;
  }
  uint64_t sel = 0;
  if (fixed_k > 0) {
    float val = masked ? c : -1.f;
    for (int r = 0; r < fixed_k; ++r) {
      const float best = wave_max(val);
      if (best < 0.f) break;                       // nothing left
      const uint64_t hit = __ballot(val == best);
      const int winner = __ffsll((unsigned long long)hit) - 1;
      sel |= 1ull << winner;
      if (lane == winner) val = -1.f;
    }
  } else {
    sel = __ballot(masked && c >= threshold);
    if (rule.hier) {
      // Runs of consecutive masked positions: lane's run is first .. last.  A run without a commit so far offers
      // its positions at or above the lower boundary; the one closest to the run's centre wins (then the more
      // confident, then the lower position).
      conf_of[lane] = c;
      __syncthreads();
      const uint64_t gaps = ~old;                                        // decided positions and everything past the block
      const uint64_t below = gaps & ((1ull << lane) - 1);
      const uint64_t above = lane < 63 ? gaps & (~0ull << (lane + 1)) : 0ull;
      const int first = below ? 64 - __clzll((long long)below) : 0;
      const int last = above ? __ffsll((unsigned long long)above) - 2 : 63;
      const uint64_t run = (last >= 63 ? ~0ull : ((2ull << last) - 1)) & ~((1ull << first) - 1);
      const bool open = masked && (sel & run) == 0;
      const uint64_t offers = __ballot(open && c >= rule.tau_low);
      bool wins = open && c >= rule.tau_low;
      if (wins) {
        const int mine = abs(2 * lane - (first + last));
        uint64_t rivals = offers & run & ~(1ull << lane);
        while (rivals) {
          const int j = __ffsll((unsigned long long)rivals) - 1;
          rivals &= rivals - 1;
          const int theirs = abs(2 * j - (first + last));
          const float cj = conf_of[j];
          if (theirs < mine || (theirs == mine && (cj > c || (cj == c && j < lane)))) wins = false;
        }
      }
      sel |= __ballot(wins);
    }
    if (sel == 0 && old != 0) {
      const float val = masked ? c : -1.f;
      const float best = wave_max(val);
      const uint64_t hit = __ballot(masked && val == best);
      if (hit) sel = 1ull << (__ffsll((unsigned long long)hit) - 1);
    }
  }
  if ((sel >> lane) & 1ull) tokens[s * block_len + lane] = am;
  if (lane == 0) {
    mask[s] = old & ~sel;
    n_committed[s] = __popcll(sel);
    // a loop of steps enqueued ahead of the host: the next step is needed if any sequence still has a masked
    // position (an OR over the sequences: integer, so the order of arrival does not matter), and this one counted
    if (next_live && (old & ~sel)) atomicOr(next_live, 1);
    if (steps && s == 0) atomicAdd(steps, 1);
  }
}
void launch_commit(const float* conf, const int32_t* argmax, int n_seq, int block_len, int row_stride, int row_off,
                   int32_t* tokens, uint64_t* mask, CommitRule rule, int32_t* n_committed, float* conf_out,
                   int32_t* argmax_out, hipStream_t st, int32_t* next_live, int32_t* steps) {
  commit_kernel<<<n_seq, 64, 0, st>>>(conf, argmax, block_len, row_stride, row_off, tokens, mask, rule, n_committed,
                                      conf_out, argmax_out, next_live, steps, live_word());
}

// Start of a loop of steps enqueued ahead of the host: flags[0] = does any sequence have a masked position;
// flags[1 .. n_flags) = 0 (each step's decoder raises the flag of the step after it); steps[0] = 0.
__global__ void loop_begin_kernel(const uint64_t* __restrict__ mask, int n_seq, int32_t* __restrict__ flags, int n_flags,
                                  int32_t* __restrict__ steps) {
  for (int i = 1 + threadIdx.x; i < n_flags; i += blockDim.x) flags[i] = 0;
  if (threadIdx.x == 0) {
    uint64_t any = 0;
    for (int s = 0; s < n_seq; ++s) any |= mask[s];
    flags[0] = any != 0;
    steps[0] = 0;
  }
}
void launch_loop_begin(const uint64_t* mask, int n_seq, int32_t* flags, int n_flags, int32_t* steps, hipStream_t st) {
  loop_begin_kernel<<<1, 256, 0, st>>>(mask, n_seq, flags, n_flags, steps);
}

// ---------------------------------------------------------------- generation loop over blocks
__global__ __launch_bounds__(64) void block_begin_kernel(int block_len, int mask_id, int eos_id,
                                                          int32_t* __restrict__ finished, bool first,
                                                          int32_t* __restrict__ block_tokens, uint64_t* __restrict__ mask) {
  const int s = blockIdx.x, lane = threadIdx.x;
  const bool fin = !first && finished[s] != 0;
  if (first && lane == 0) finished[s] = 0;
  if (lane < block_len) block_tokens[s * block_len + lane] = fin ? eos_id : mask_id;
  if (lane == 0) mask[s] = fin ? 0ull : (block_len >= 64 ? ~0ull : ((1ull << block_len) - 1));
}
void launch_block_begin(int n_seq, int block_len, int mask_id, int eos_id, int32_t* finished, bool first,
                        int32_t* block_tokens, uint64_t* mask, hipStream_t st) {
  block_begin_kernel<<<n_seq, 64, 0, st>>>(block_len, mask_id, eos_id, finished, first, block_tokens, mask);
}
// One wave walks the sequences, so that the count of finished sequences needs no atomics.
__global__ __launch_bounds__(64) void block_end_kernel(int n_seq, int block_len, int n_blocks, int block_index, int eos_id,
                                                        const int32_t* __restrict__ block_tokens, int32_t* __restrict__ out,
                                                        int32_t* __restrict__ finished, int32_t* __restrict__ n_finished) {
  const int lane = threadIdx.x;
  int count = 0;
  for (int s = 0; s < n_seq; ++s) {
    const int tok = lane < block_len ? block_tokens[s * block_len + lane] : -1;
    if (lane < block_len) out[((int64_t)s * n_blocks + block_index) * block_len + lane] = tok;
    const bool fin = finished[s] != 0 || (eos_id >= 0 && __ballot(lane < block_len && tok == eos_id) != 0);
    if (fin) {
      ++count;
      if (lane == 0) finished[s] = 1;
    }
  }
  if (lane == 0) n_finished[0] = count;
}
void launch_block_end(int n_seq, int block_len, int n_blocks, int block_index, int eos_id, const int32_t* block_tokens,
                      int32_t* out, int32_t* finished, int32_t* n_finished, hipStream_t st) {
  block_end_kernel<<<1, 64, 0, st>>>(n_seq, block_len, n_blocks, block_index, eos_id, block_tokens, out, finished,
                                     n_finished);
}
__global__ void fill_blocks_kernel(int block_len, int n_blocks, int first_block, int eos_id, int32_t* __restrict__ out) {
  const int s = blockIdx.x;
  for (int i = first_block * block_len + threadIdx.x; i < n_blocks * block_len; i += blockDim.x)
    out[(int64_t)s * n_blocks * block_len + i] = eos_id;
}
void launch_fill_blocks(int n_seq, int block_len, int n_blocks, int first_block, int eos_id, int32_t* out,
                        hipStream_t st) {
  if (first_block >= n_blocks) return;
  fill_blocks_kernel<<<n_seq, 256, 0, st>>>(block_len, n_blocks, first_block, eos_id, out);
}

// Token run of a vicinity-refresh forward: per sequence the look_back neighbour ids, then the block's ids; the run
// starts look_back positions before the block (never before position 0).
__global__ void vicinity_pack_kernel(int block_len, int look_back, const int32_t* __restrict__ block_tokens,
                                     const int32_t* __restrict__ vicinity_tokens, const int32_t* __restrict__ prefix_len,
                                     int32_t* __restrict__ run_tokens, int32_t* __restrict__ run_base) {
  const int s = blockIdx.x, n = look_back + block_len;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    run_tokens[s * n + i] = i < look_back ? vicinity_tokens[s * look_back + i] : block_tokens[s * block_len + i - look_back];
  if (threadIdx.x == 0) run_base[s] = max(0, prefix_len[s] - look_back);
}
void launch_vicinity_pack(int n_seq, int block_len, int look_back, const int32_t* block_tokens,
                          const int32_t* vicinity_tokens, const int32_t* prefix_len, int32_t* run_tokens,
                          int32_t* run_base, hipStream_t st) {
  vicinity_pack_kernel<<<n_seq, 128, 0, st>>>(block_len, look_back, block_tokens, vicinity_tokens, prefix_len, run_tokens,
                                              run_base);
}

__global__ void add_i32_kernel(int32_t* a, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] += v;
}
void launch_add_i32(int32_t* a, int n, int v, hipStream_t st) {
  add_i32_kernel<<<(n + 63) / 64, 64, 0, st>>>(a, n, v);
}

// ---------------------------------------------------------------- streaming-read probe (benchmarks)
// Reads `bytes` once with the access pattern of the weight streams (each wave walks contiguous 256 KiB chunks,
// 16 KiB-loads in flight) and keeps nothing: its duration is the practical HBM read ceiling of the chip.
__global__ __launch_bounds__(256) void stream_read_kernel(const f32x4* __restrict__ p, size_t n_chunks, float* sink) {
  constexpr size_t CHUNK = (256 << 10) / 16;
  const size_t wave = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (size_t c = wave; c < n_chunks; c += (size_t)gridDim.x * 4) {
    const f32x4* q = p + c * CHUNK + lane;
    for (size_t i = 0; i < CHUNK; i += 64 * 16) {
      f32x4 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = __builtin_nontemporal_load(q + i + u * 64);   // as the weight streams do: measured 7.1 against 6.3 TB/s
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v[u];
    }
  }
  if (acc[0] + acc[1] + acc[2] + acc[3] == 1.2345e38f) sink[0] = 1.f;   // never true for finite sums of this data
}
void launch_stream_read(const void* buf, size_t bytes, float* sink, hipStream_t st) {
  const size_t n_chunks = bytes / (256 << 10);
  if (n_chunks == 0) return;
  const unsigned wgs = (unsigned)(n_chunks < 4096 ? (n_chunks + 3) / 4 : 1024);
  stream_read_kernel<<<wgs, 256, 0, st>>>((const f32x4*)buf, n_chunks, sink);
}

// ---------------------------------------------------------------- KV import / export (tests)
template <typename E>
__global__ void kv_copy_kernel(bool to_pool, E* __restrict__ kv_layer, KvGeom geom, const int32_t* __restrict__ page_row,
                               int first_pos, int n_pos, float* __restrict__ k, float* __restrict__ v) {
  const int D = geom.n_heads * geom.head_dim;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n_pos * D) return;
  const int r = (int)(i / D), f = (int)(i % D);
  const int pos = first_pos + r;
  const int page = safe_page(geom, page_row[pos / PAGE]), slot = pos % PAGE;
  const int64_t ki = kv_k_index(geom, page, f / geom.head_dim, slot, f % geom.head_dim);
  const int64_t vi = kv_v_index(geom, page, f / geom.head_dim, slot, f % geom.head_dim);
  if (to_pool) {
    kv_layer[ki] = from_f32<E>(k[i]);
    kv_layer[vi] = from_f32<E>(v[i]);
  } else {
    k[i] = to_f32(kv_layer[ki]);
    v[i] = to_f32(kv_layer[vi]);
  }
}
void launch_kv_copy(bool bf16, bool to_pool, void* kv_layer, KvGeom geom, const int32_t* page_row, int first_pos,
                    int n_pos, float* k, float* v, hipStream_t st) {
  const int64_t n = (int64_t)n_pos * geom.n_heads * geom.head_dim;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (bf16) kv_copy_kernel<bf16_t><<<blocks, 256, 0, st>>>(to_pool, (bf16_t*)kv_layer, geom, page_row, first_pos, n_pos, k, v);
  else kv_copy_kernel<float><<<blocks, 256, 0, st>>>(to_pool, (float*)kv_layer, geom, page_row, first_pos, n_pos, k, v);
}

}  // namespace dinfer
