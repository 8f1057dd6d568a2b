// The weight-streaming contractions with the most bytes: routed-expert grouped GEMMs and the LM head, in the
// shared-operand form of wide_stream.hpp for every token count.  A workgroup takes a few tasks (64 output features
// each) and 1, 2 or 4 tiles of 32 token rows; each wave streams the whole K range of one task and keeps its
// accumulators in registers (no split of K, no fold), and the activation fragments go through LDS once per
// workgroup.  With hundreds of token rows a wave that fetched its own activation operands would pull several
// times more bytes through the L2 than it streams weights from HBM; with few rows it still keeps the compute
// unit's address path busy with 64 separate rows per load.  Work that would leave most of the chip idle (a few items
// beyond a full round, small models) goes out in pieces instead: one task per workgroup, K cut over its waves.
#include "kernels.hpp"
#include "routing.hpp"
#include "wide_stream.hpp"

namespace dinfer {

constexpr int WT = 4;      // token tiles per workgroup above 64 tokens
// Waves (= tasks) per workgroup and weight chunks in flight per wave.  Eight waves put two on every SIMD, so one
// computes while the other waits for LDS or memory, and the activation fragments are shared by eight tasks.
// (Measured at 512 tokens: four waves with two, four or six weight chunks in flight are slower for the expert
// GEMMs, 131 to 134 against 120 microseconds; four waves in the LM head, 450 against 352.)
static_assert(EXPERT_WT == WT && EXPERT_TILE == TILE, "expert_plan.hpp counts in these units");
// (tasks per workgroup of the LM head: lm_plan.hpp)
static_assert(LM_SMALL_T == TILE && LM_MID_T == 2 * TILE, "the forms of the LM head take one, two and four token tiles");
constexpr int XCDS = 8;      // accelerator dies, each with its own L2; workgroup i of a launch runs on die i % 8

// ------------------------------------------------------------------------------------------------
// Routed experts.  An item is a run of an expert's sorted rows, {expert, first sorted row, rows, 0}: up to 64 tokens all
// rows of an expert (the i-th expert with rows: PairIds in routing.hpp), beyond groups of up to 64 or 128 rows, heaviest
// first (the work list of the permutation kernel).  pair(): the (token, slot) pair of sorted row r.
//   GEMM 1: task = 32 gate features + the same 32 up features;  y = silu(gate) * up  -> Y[sorted row][I]
//   GEMM 2: task = 64 adjacent output features of the down projection                -> O[token*top_k + slot][H]
// ------------------------------------------------------------------------------------------------
template <typename E> struct GateUp {
  static constexpr bool COUNTS = true;     // keeps the running totals of experts with rows
  const E* W;
  const E* xn;
  const float* rinv;
  E* Y;
  const int32_t* perm;   // more than 64 tokens
  int T, H, I, top_k;
  const float* topk_w;   // the routing weight, when the down projection sums the experts itself; else null
  __device__ int ksteps() const { return H / ET<E>::KS; }
  __device__ int n_tasks() const { return I / TILE; }
  __device__ const E* act() const { return xn; }
  __device__ int64_t act_rows() const { return T; }
  template <class P> __device__ int act_row(int, P&& pair) const { return pair() / top_k; }
  // what the lane needs to know about sorted row r
  struct Row {
    int act;         // its row among the activations
    float r, wgt;
  };
  __device__ Row row(int, int pair) const {
    const int tok = pair / top_k;
    return Row{tok, rinv[tok], topk_w ? topk_w[pair] : 1.f};
  }
  __device__ static float silu(float x) { return x / (1.f + __expf(-x)); }
  // accumulator registers 4g .. 4g+3 of both tiles of `task`: four consecutive features of sorted row r
  __device__ void store(const Row& w, int r, int task, int g, int half, const f32x4& a, const f32x4& b) const {
    f32x4 y;
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = silu(a[i] * w.r) * (b[i] * w.r) * w.wgt;
    store_actk4<E>(Y, (int64_t)T * top_k, r, task * TILE + acc_row(4 * g, half), y);
  }
};
template <typename E> struct Down {
  static constexpr bool COUNTS = false;
  const E* W;
  const E* Y;
  float* O;
  const int32_t* perm;
  int n_pairs, H, I;
  __device__ int ksteps() const { return I / ET<E>::KS; }
  __device__ int n_tasks() const { return H / (2 * TILE); }
  __device__ const E* act() const { return Y; }
  __device__ int64_t act_rows() const { return n_pairs; }
  template <class P> __device__ int act_row(int r, P&&) const { return r; }
  struct Row {
    int act, pair;
  };
  __device__ Row row(int r, int pair) const { return Row{r, pair}; }
  __device__ void store(const Row& w, int, int task, int g, int half, const f32x4& a, const f32x4& b) const {
    float* o = O + (int64_t)w.pair * H + (2 * task) * TILE + acc_row(4 * g, half);
    *reinterpret_cast<f32x4*>(o) = a;
    *reinterpret_cast<f32x4*>(o + TILE) = b;
  }
};

// One item and WW tasks (task group tg) by a workgroup: every wave streams its task's whole K range.  pair_of(i): the pair of
// the item's row i.
template <typename E, int WT, int WW, int KID, class Op, class PairOf>
__device__ inline void expert_tasks(const Op& op, const int4& it, int tg, char* lds, PairOf&& pair_of) {
  typedef typename ET<E>::vec vec;
  constexpr int KS = ET<E>::KS, NP = Planes<E>::N;
  TRACE_MARK(KID, 3);
  const int e = it.x, base = it.y, n_rows = it.z;
  const int nt = min(WT, (n_rows + TILE - 1) / TILE);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int n_tasks = op.n_tasks(), task = min(tg * WW + wave, n_tasks - 1), ksteps = op.ksteps();
  // The rows hang on the permutation: that chain is resolved while the first weights are in flight.  What the epilogue
  // needs of them waits in registers; where the accumulators of four tiles leave too few, it is asked for again there.
  constexpr bool AGAIN = WT >= 4;
  typename Op::Row rows[WT];
  auto row_of = [&](int t) {
    const int i = min(t * TILE + col, n_rows - 1);
    return op.row(base + i, pair_of(i));
  };
  auto staged = [&](int r) {
    const int i = min((wave % WT) * TILE + r, n_rows - 1);
    return op.act_row(base + i, [&] { return pair_of(i); });
  };
  if constexpr (!AGAIN) {
#pragma unroll
    for (int t = 0; t < WT; ++t) rows[t] = row_of(t);
  }
  f32x16 acc0[WT], acc1[WT];
  zero_acc<WT>(acc0);
  zero_acc<WT>(acc1);
  wide_stream<E, WT, WW, KID>(op.W + ((int64_t)e * n_tasks + task) * task_stride_elems<E>(ksteps), ksteps, op.act(), staged, op.act_rows() * (NP * KS), reinterpret_cast<vec*>(lds), nt, acc0, acc1, wave);
  if (tg * WW + wave >= n_tasks) return;
  if constexpr (AGAIN) {
#pragma unroll
    for (int t = 0; t < WT; ++t) rows[t] = row_of(t);
  }
#pragma unroll
  for (int t = 0; t < WT; ++t) {
    if (t < nt && t * TILE + col < n_rows) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 a, b;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[i] = acc0[t][4 * g + i];
          b[i] = acc1[t][4 * g + i];
        }
        op.store(rows[t], base + t * TILE + col, task, g, half, a, b);
      }
    }
  }
  TRACE_MARK(KID, 7);
}

// One item of up to TT tiles and ONE task by a workgroup of KW waves, which cut the task's K range and meet in LDS.
template <typename E, int TT, int KW, class Op, class PairOf>
__device__ inline void expert_piece(const Op& op, const int4& it, int task, char* lds, PairOf&& pair_of) {
  constexpr int PER = 4, EW = 16 / PER;
  static_assert(KW >= EW, "the first EW waves run the epilogue");
  const int e = it.x, base = it.y, n_rows = it.z;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int ksteps = op.ksteps(), per = (ksteps + KW - 1) / KW, ks0 = min(ksteps, wave * per), ks1 = min(ksteps, ks0 + per);
  typename Op::Row rows[TT];
  PlaneLoader<E, TT> ld;
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const int i = min(t * TILE + col, n_rows - 1);
    rows[t] = op.row(base + i, pair_of(i));
    ld.set(t, op.act(), op.act_rows(), rows[t].act, half);
  }
  f32x16 acc0[TT], acc1[TT];
  zero_acc<TT>(acc0);
  zero_acc<TT>(acc1);
  stream_task<E, TT, (TT == 1 ? 8 : 4)>(op.W + ((int64_t)e * op.n_tasks() + task) * task_stride_elems<E>(ksteps), ks0, ks1, ld, acc0, acc1);
  float* red = reinterpret_cast<float*>(lds);
  spill_partials<TT, 2 * TT * 16>(red, wave, lane, acc0, acc1);
  __syncthreads();
  if (wave >= EW) return;
  float a0[TT][PER], a1[TT][PER];
  fold_partials<TT, KW, PER>(red, lane, wave * PER, a0, a1);
#pragma unroll
  for (int t = 0; t < TT; ++t)
    if (t * TILE + col < n_rows)
      op.store(rows[t], base + t * TILE + col, task, wave, half, f32x4{a0[t][0], a0[t][1], a0[t][2], a0[t][3]},
               f32x4{a1[t][0], a1[t][1], a1[t][2], a1[t][3]});
}

// Up to 64 tokens: the workgroup's item, the i-th expert with rows, from the routing; false where there is none.
template <int TT> __device__ inline bool routed_item(const int32_t* __restrict__ topk_idx, int n_pairs, int i, int32_t* s_pair, int32_t* totals, int4& it) {
  PairIds<TT * TILE * MAX_TOPK / WAVE> ids;
  ids.load(topk_idx, n_pairs);
  const uint64_t experts = ids.experts();
  const int n = __popcll(experts);
  if (totals && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    totals[0] += n;
    totals[1] += 1;
  }
  if (i >= n) return false;                         // uniform over the block
  it = ids.rows_of(nth_bit(experts, i), s_pair);
  __syncthreads();
  return true;
}

// Grid (task groups, experts): one workgroup each, those beyond the experts with rows at the end.
template <typename E, int WT, int WW, int KID, class Op>
__global__ __launch_bounds__(WW * WAVE) __attribute__((amdgpu_waves_per_eu(2))) void expert_kernel(Op op, const int32_t* __restrict__ topk_idx, int n_pairs,
                                                                                                 int32_t* __restrict__ totals,
                                                                                                 const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  __shared__ __align__(16) int32_t s_pair[WAVE];
  int4 it;
  if (!routed_item<WT>(topk_idx, n_pairs, blockIdx.y, s_pair, totals, it)) return;
  expert_tasks<E, WT, WW, KID, Op>(op, it, blockIdx.x, lds_raw, [&](int i) { return s_pair[i]; });
}

// Grid (tasks, experts): every task in pieces (up to 64 tokens, few tasks: see launch_expert_op).
template <typename E, int TT, class Op>
__global__ __launch_bounds__(EXPERT_WW * WAVE) __attribute__((amdgpu_waves_per_eu(2))) void expert_pieces_kernel(Op op, const int32_t* __restrict__ topk_idx, int n_pairs,
                                                                                                              int32_t* __restrict__ totals,
                                                                                                              const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  extern __shared__ __align__(16) char lds_raw[];
  __shared__ __align__(16) int32_t s_pair[WAVE];
  int4 it;
  if (!routed_item<TT>(topk_idx, n_pairs, blockIdx.y, s_pair, totals, it)) return;
  expert_piece<E, TT, EXPERT_WW, Op>(op, it, blockIdx.x, lds_raw, [&](int i) { return s_pair[i]; });
}

// More than 64 tokens.  Grid (task groups, rows): the first rows are items in whole task groups (WW tasks, one per
// wave), the workgroups of the further ones take the remaining, light items task by task, the last ones find nothing and
// return.  All workgroups of whole items are resident at once (eight waves fill a compute unit), so that items beyond a
// full round of the chip begin another one: at 512 tokens two experts with a few rows more than 128 did so for eight
// workgroups, and the launch's 256 others ended between 70 and 100 us, those at 137 (gate/up 142 us a launch, 109 with
// the pieces, which the units that finish early pick up; down 87 and 71).
template <typename E, int WT, int WW, int KID, class Op>
__global__ __launch_bounds__(WW * WAVE) __attribute__((amdgpu_waves_per_eu(2))) void expert_many_kernel(Op op, const int32_t* __restrict__ work,
                                                                                                            const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  const int4* items = reinterpret_cast<const int4*>(work + WORK_ITEMS);
  const int n_big = work[WORK_BIG];
  auto pairs_at = [&](int base) { return [&op, base](int i) { return op.perm[base + i]; }; };
  int piece;
  if constexpr (wide_expert_shared(KID)) {
    // an item's task groups on one die, one after the other, and behind them its expert's other items (expert_plan.hpp)
    const int wg = blockIdx.y * gridDim.x + blockIdx.x, whole = expert_unit_wgs(n_big, gridDim.x);
    if (wg < whole) {
      const ExpertUnit u = expert_unit(wg, work[WORK_HEAVY], work[WORK_ALL] - work[WORK_LIGHT], n_big, gridDim.x);
      if (u.item >= 0) {
        const int4 it = items[u.item];
        expert_tasks<E, WT, WW, KID, Op>(op, it, u.group, lds_raw, pairs_at(it.y));
      }
      return;
    }
    piece = wg - whole;
  } else {
    if ((int)blockIdx.y < n_big) {
      const int4 it = items[blockIdx.y];
      expert_tasks<E, WT, WW, KID, Op>(op, it, blockIdx.x, lds_raw, pairs_at(it.y));
      return;
    }
    piece = ((int)blockIdx.y - n_big) * gridDim.x + blockIdx.x;
  }
  const int n_tasks = op.n_tasks();
  if (piece >= (work[WORK_ALL] - n_big) * n_tasks) return;   // uniform over the block
  const int4 it = items[n_big + piece / n_tasks];
  if (it.z <= TILE) expert_piece<E, 1, WW, Op>(op, it, piece % n_tasks, lds_raw, pairs_at(it.y));
  else expert_piece<E, 2, WW, Op>(op, it, piece % n_tasks, lds_raw, pairs_at(it.y));
}

// Up to 32 / 64 tokens: one / two token tiles and SMALL_WW tasks per workgroup
// (trace ids 16 .. 19); more: four tiles, eight tasks, the work list of the permutation kernel (ids 10, 11).
// (Measured, gate/up + down in microseconds: two tasks 69.8 + 37.6 at 32 tokens and 86.6 + 49.2 at 64; four tasks
// 68.9 + 38.9 and 88.1 + 50.7; the earlier per-wave-operand kernels, whose four waves split K, 72.9 + 38.6 and
// 100.5 + 55.2.  Four or six weight chunks in flight per wave instead of two: 71.9 + 39.4 at 32 tokens, 90.8 + 53.0
// at 64.)
constexpr int SMALL_WW = 2;
// The gate/up projection of up to 32 tokens takes one task per workgroup: with 49 to 56 experts touched, 16
// two-task workgroups per expert are 3.1 to 3.5 per compute unit, so some units carry four (2 MB) and the launch
// lasts as long as those; 32 one-task workgroups per expert put 1.75 MB on the fullest unit (78 -> 70 us for such
// layers, 69.1 -> 65.7 us on average at batch 1, though every workgroup now stages the activation rows for itself).
constexpr int GU1_WW = 1;
// More than 64 tokens: expert_plan.hpp (trace ids 20, 21 for the form of few rows per expert, 10, 11 for the other).
// LDS of expert_many_kernel: staged fragments, or two tiles of WW waves' partial sums
template <int WW> constexpr size_t many_lds() { return (size_t)WW * 2 * 2 * 16 * WAVE * 4; }

// KID: trace ids of the forms for up to 32, up to 64, few rows per expert, many rows per expert, several items per expert
// (Up to 32 tokens the down projection takes its first form, ids 18 and the pieces of one tile, only under the single-slice
// test switch: expert_down_fused_kernel has it otherwise.)
template <typename E, int WW1, int K1, int K2, int K3, int K4, int K5, class Op>
static void launch_expert_op(const Op& op, const ExpertArgs& a, int n_tasks, hipStream_t st) {
  const int n_pairs = a.T * a.top_k;
  auto grid = [&](int ww, int items) { return dim3((n_tasks + ww - 1) / ww, items); };
  if (a.T <= 2 * TILE) {
    int32_t* totals = Op::COUNTS ? a.off + STAT_ACTIVE_SUM : nullptr;
    // Few tasks over all experts (one per compute unit or less): a workgroup of eight waves each, since a wave alone with
    // a task is bound by its chain of loads and matrix instructions (8 experts of 512, hidden 256, float32: gate/up 14.6
    // -> 9.6 us at 32 tokens, 23 -> 13 at 64, down at 64 tokens 37 -> 17.5).
    if (a.E * n_tasks <= EXPERT_CUS && a.T <= TILE)
      expert_pieces_kernel<E, 1, Op><<<dim3(n_tasks, a.E), EXPERT_WW * WAVE, many_lds<EXPERT_WW>() / 2, st>>>(op, a.topk_idx, n_pairs, totals, live_word());
    else if (a.E * n_tasks <= EXPERT_CUS)
      expert_pieces_kernel<E, 2, Op><<<dim3(n_tasks, a.E), EXPERT_WW * WAVE, many_lds<EXPERT_WW>(), st>>>(op, a.topk_idx, n_pairs, totals, live_word());
    else if (a.T <= TILE)
      expert_kernel<E, 1, WW1, K1, Op><<<grid(WW1, a.E), WW1 * WAVE, wide_lds<E, K1, 1>(), st>>>(op, a.topk_idx, n_pairs, totals, live_word());
    else
      expert_kernel<E, 2, SMALL_WW, K2, Op><<<grid(SMALL_WW, a.E), SMALL_WW * WAVE, wide_lds<E, K2, 2>(), st>>>(op, a.topk_idx, n_pairs, totals, live_word());
  } else {
    auto many = [&](auto kernel, int wt, int ww, size_t lds, int more = 0) {   // more: rows of the grid for the whole multiple of dies
      const dim3 whole = grid(ww, expert_work_items(a.E, n_pairs, wt) + more);
      const int pieces = expert_most_piece_items(a.E, n_pairs, a.H, a.I) * n_tasks;
      kernel<<<dim3(whole.x, whole.y + (pieces + whole.x - 1) / whole.x), ww * WAVE, lds, st>>>(op, a.work, live_word());
    };
    if (expert_group_tiles(a.E, n_pairs) == MID_WT) many(expert_many_kernel<E, MID_WT, MID_WW, K3, Op>, MID_WT, MID_WW, many_lds<MID_WW>());
    else if (expert_shared(sizeof(E) == 2, a.E, n_pairs, grid(EXPERT_WW, 1).x)) many(expert_many_kernel<E, WT, EXPERT_WW, K5, Op>, WT, EXPERT_WW, many_lds<EXPERT_WW>(), XCDS - 1);
    else many(expert_many_kernel<E, WT, EXPERT_WW, K4, Op>, WT, EXPERT_WW, many_lds<EXPERT_WW>());
  }
}
template <typename E> static GateUp<E> gate_up_op(const ExpertArgs& a) {
  return GateUp<E>{(const E*)a.w_gate_up, (const E*)a.xn, a.rinv, (E*)a.y, a.perm, a.T, a.H, a.I, a.top_k, a.topk_w};
}
template <typename E> static void launch_gate_up_wide_t(const ExpertArgs& a, hipStream_t st) {
  launch_expert_op<E, GU1_WW, 16, 17, 20, 10, 25>(gate_up_op<E>(a), a, a.I / TILE, st);
}
template <typename E> static void launch_down_wide_t(const ExpertArgs& a, hipStream_t st) {
  const Down<E> op{(const E*)a.w_down, (const E*)a.y, a.o, a.perm, a.T * a.top_k, a.H, a.I};
  launch_expert_op<E, SMALL_WW, 18, 19, 21, 11, 26>(op, a, a.H / (2 * TILE), st);
}
void launch_expert_gate_up_wide(bool bf16, const ExpertArgs& a, hipStream_t st) {
  if (bf16) launch_gate_up_wide_t<bf16_t>(a, st);
  else launch_gate_up_wide_t<float>(a, st);
}
void launch_expert_down_wide(bool bf16, const ExpertArgs& a, hipStream_t st) {
  if (bf16) launch_down_wide_t<bf16_t>(a, st);
  else launch_down_wide_t<float>(a, st);
}

// ------------------------------------------------------------------------------------------------
// LM head fused with the confidence reduction, many-token form.  A workgroup takes one task group (8 tasks = 512
// vocabulary ids) and one group of 128 tokens; a wave turns its accumulators (64 vocabulary ids x 128 tokens) into
// one (max, sum-exp, lowest arg max) partial per token: part[token][task group, wave].  Logits are never
// stored (unless the debug pointer is set).
// The token groups of one task group stream the same weights.  Workgroups go to the dies in turn, so the launch is
// one-dimensional and workgroup i = die (i % 8), turn (i / 8): consecutive turns of ONE die take the token groups
// of one task group, which then run side by side behind the same L2 (measured at 512 tokens: 0.88 GB fetched from
// HBM per launch for 0.64 GB of weights, where four separate passes would fetch 2.6 GB).
// ------------------------------------------------------------------------------------------------
template <typename E, int WT, int KID, int WW>
__global__ __launch_bounds__(WW * WAVE) __attribute__((amdgpu_waves_per_eu(WT == 1 && WW == LM_SMALL_WW ? 3 : 2))) void lm_head_wide_kernel(const E* __restrict__ W, const E* __restrict__ xn,
                                                                  RowNorm norm, int T, int H, int V,
                                                                  float scale, float* __restrict__ part,
                                                                  float* __restrict__ logits_out,
                                                                  const int32_t* __restrict__ rows, LmPlan plan,
                                                                  const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  vec* sb = reinterpret_cast<vec*>(lds_raw);
  constexpr int KS = ET<E>::KS, NP = Planes<E>::N;
  const int wave_of_lane = threadIdx.x >> 6, wave = __builtin_amdgcn_readfirstlane(wave_of_lane), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  // With a row list the workgroup's 128 "tokens" are entries of the list, and the token groups are counted from
  // the list's length: the grid is sized for all T rows, and the workgroups left over at its end return at once.
  const int n_rows = rows ? min(rows[0], T) : T;
  if (n_rows == 0) return;              // uniform over the workgroup
  // The token groups take equal numbers of tiles: they stream the same weights side by side, and a group of one tile
  // beside one of four runs ahead of it and fetches them from memory again (160 tokens: 248 us as 4 + 1, 209 as 3 + 2).
  const int tiles = (n_rows + TILE - 1) / TILE, groups = (tiles + WT - 1) / WT, per_group = (tiles + groups - 1) / groups;
  const int turn = blockIdx.x / XCDS;
  const int tgroup = (turn / groups) * XCDS + blockIdx.x % XCDS;
  const int n_tasks = plan.tasks;
  // Partials of a row lie next to each other for the merge kernel (a stride of 8 KB apart it took 27 us for 512 tokens).
  // Up to 64 tokens a workgroup leaves one per row, more tokens: its waves one each (folding them there costs the
  // launch 8 us at 512 tokens, more than the merge saves).
  constexpr bool FOLD = KID != 9;
  const int n_groups = plan.whole, first_piece = plan.first_piece, n_parts = plan.parts;
  if (tgroup >= n_groups + n_tasks - first_piece) return;   // uniform over the workgroup
  LmStat* s_stat = reinterpret_cast<LmStat*>(lds_raw);   // [WW][WT * TILE], once the fragments are done with
  static_assert(WW * WT * TILE * sizeof(LmStat) <= wide_lds<E, KID, WT>(), "the statistics fit the staging area");
  const bool quads = V % 4 == 0 && ((uintptr_t)logits_out & 15) == 0;   // rows of logits start on 16-byte boundaries
  auto row_of = [&](int i) { return rows ? min(max(rows[1 + min(i, n_rows - 1)], 0), T - 1) : min(i, T - 1); };
  constexpr bool ONLY_PIECES = FOLD && WW == LM_PIECE_WW;
  if constexpr (FOLD && WW >= LM_MID_WW) {
    if (ONLY_PIECES || tgroup >= n_groups) {
      // One task, its K range cut over the waves (one token group: n_rows <= WT * TILE): a wave ends up with PER
      // accumulator registers of both weight tiles.
      constexpr int PER = 16 / WW;
      const int wave = wave_of_lane;   // a scalar K range costs the per-wave stream 5 % (float32, 84 tasks of K = 3328: 44.3 -> 47.6 us)
      const int task = first_piece + tgroup - n_groups, ksteps = H / KS, per = (ksteps + WW - 1) / WW;
      const int ks0 = min(ksteps, wave * per), ks1 = min(ksteps, ks0 + per);
      PlaneLoader<E, WT> ld;
      float zs[WT];
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        const int tok = row_of(t * TILE + col);
        ld.set(t, xn, T, tok, half);
        zs[t] = row_rinv(norm.ssq, norm.n_ssq, T, tok, H, norm.eps) * scale;
      }
      f32x16 acc0[WT], acc1[WT];
      zero_acc<WT>(acc0);
      zero_acc<WT>(acc1);
      stream_task<E, WT, (WT == 1 ? 8 : 4)>(W + (int64_t)task * task_stride_elems<E>(ksteps), ks0, ks1, ld, acc0, acc1);
      float* red = reinterpret_cast<float*>(lds_raw);
      spill_partials<WT, 2 * WT * 16>(red, wave, lane, acc0, acc1);
      __syncthreads();
      float a0[WT][PER], a1[WT][PER];
      fold_partials<WT, WW, PER>(red, lane, wave * PER, a0, a1);
      __syncthreads();   // the partial sums have been read: s_stat takes their place
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        LmStat st{-INFINITY, 0.f, 0x7fffffff};
        float z[2 * PER];
#pragma unroll
        for (int i = 0; i < 2 * PER; ++i) {
          const int id = (2 * task + i / PER) * TILE + acc_row(wave * PER + i % PER, half);
          z[i] = id < V ? (i < PER ? a0[t][i % PER] : a1[t][i % PER]) * zs[t] : -INFINITY;
          if (z[i] > st.m) {
            st.m = z[i];
            st.id = id;
          }
          if (logits_out && t * TILE + col < n_rows && id < V) logits_out[(int64_t)row_of(t * TILE + col) * V + id] = z[i];
        }
        if (st.m > -INFINITY) {
#pragma unroll
          for (int i = 0; i < 2 * PER; ++i) st.s += __expf(z[i] - st.m);
        }
        st = lm_combine(st, LmStat{__shfl_xor(st.m, 32, WAVE), __shfl_xor(st.s, 32, WAVE), __shfl_xor(st.id, 32, WAVE)});
        if (half == 0) s_stat[wave * WT * TILE + t * TILE + col] = st;
      }
      __syncthreads();
      for (int i = threadIdx.x; i < min(n_rows, WT * TILE); i += WW * WAVE) {
        LmStat a = s_stat[i];
#pragma unroll
        for (int w = 1; w < WW; ++w) a = lm_combine(a, s_stat[w * WT * TILE + i]);
        *reinterpret_cast<f32x4*>(part + ((int64_t)row_of(i) * n_parts + tgroup) * 4) = f32x4{a.m, a.s, __int_as_float(a.id), 0.f};
      }
      return;
    }
  }
  if constexpr (!ONLY_PIECES) {
  const int tok0 = (turn % groups) * per_group * TILE;
  const int nt = min(per_group, tiles - (turn % groups) * per_group);
  if (nt <= 0) return;                  // uniform: fewer tiles than groups * per_group
  TRACE_MARK(KID, 3);
  const int slot = tgroup * WW + wave, task = min(slot, n_tasks - 1);
  const int ksteps = H / KS;
  int tok_of[WT];
  float zs[WT];
#pragma unroll
  for (int t = 0; t < WT; ++t) {
    tok_of[t] = row_of(tok0 + t * TILE + col);
    zs[t] = row_rinv(norm.ssq, norm.n_ssq, T, tok_of[t], H, norm.eps) * scale;
  }
  f32x16 acc0[WT], acc1[WT];
  zero_acc<WT>(acc0);
  zero_acc<WT>(acc1);
  wide_stream<E, WT, WW, KID>(W + (int64_t)task * task_stride_elems<E>(ksteps), ksteps, xn,
                                      [&](int r) { return row_of(tok0 + (wave % WT) * TILE + r); }, (int64_t)T * (WidePlanes<E, KID>::N * KS), sb, nt, acc0, acc1, wave);
#pragma unroll
  for (int t = 0; t < WT; ++t) {
    const bool listed = tok0 + t * TILE + col < n_rows;
    const int tok = listed ? tok_of[t] : T;     // T: no row
    float m = -INFINITY, sum = 0.f;
    int best = 0x7fffffff;
    if (t < nt && slot < n_tasks) {
      // 128 logits per lane at four tiles: the maximum first, then the lowest id that has it (from the last one down), so that
      // a logit costs a compare and a select less than with both at once, and only the vocabulary's last task tests ids
      // against its end (512 tokens: 12 of a workgroup's 79 us were spent here).
      const int id0 = 2 * task * TILE + 4 * half;
      auto id_of = [](int i) { return (i >> 4) * TILE + acc_row(i & 15, 0); };   // + id0: ascends with i
      float z[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) z[i] = (i < 16 ? acc0[t][i & 15] : acc1[t][i & 15]) * zs[t];
      if ((2 * task + 2) * TILE > V) {   // uniform
#pragma unroll
        for (int i = 0; i < 32; ++i)
          if (id0 + id_of(i) >= V) z[i] = -INFINITY;
      }
#pragma unroll
      for (int i = 0; i < 32; ++i) m = fmaxf(m, z[i]);   // passes over NaN
      int at = 0;
#pragma unroll
      for (int i = 31; i >= 0; --i) at = z[i] == m ? id_of(i) : at;
      if (m > -INFINITY) best = id0 + at;
      if (logits_out && !quads && tok < T) {
#pragma unroll
        for (int i = 0; i < 32; ++i)
          if (id0 + id_of(i) < V) logits_out[(int64_t)tok * V + id0 + id_of(i)] = z[i];
      }
      if (logits_out && quads && tok < T) {
        // every lane stores into a row of its own, so the address unit takes the 64 lanes one by one: four
        // consecutive ids per store (32 tokens: LM head with stored logits 137 us, element by element)
#pragma unroll
        for (int i = 0; i < 32; i += 4) {
          const int id = (2 * task + (i >> 4)) * TILE + acc_row(i & 15, half);
          if (id < V) *reinterpret_cast<f32x4*>(logits_out + (int64_t)tok * V + id) = f32x4{z[i], z[i + 1], z[i + 2], z[i + 3]};
        }
      }
      if (m > -INFINITY) {
#pragma unroll
        for (int i = 0; i < 32; ++i) sum += __expf(z[i] - m);
      }
    }
    // fold the two half-waves (same token, other rows); up to 64 tokens also the workgroup's waves (other ids), through LDS
    const LmStat w = lm_combine(LmStat{m, sum, best}, LmStat{__shfl_xor(m, 32, WAVE), __shfl_xor(sum, 32, WAVE), __shfl_xor(best, 32, WAVE)});
    if constexpr (FOLD) {
      if (t == 0) __syncthreads();   // the staged fragments have been read by every wave
      if (half == 0) s_stat[wave * WT * TILE + t * TILE + col] = w;
    } else if (half == 0 && t < nt && tok < T) {
      *reinterpret_cast<f32x4*>(part + ((int64_t)tok * n_parts + slot) * 4) = f32x4{w.m, w.s, __int_as_float(w.id), 0.f};
    }
  }
  if constexpr (FOLD) {
    __syncthreads();
    for (int i = threadIdx.x; i < nt * TILE; i += WW * WAVE) {
      LmStat a = s_stat[i];
#pragma unroll
      for (int w = 1; w < WW; ++w) a = lm_combine(a, s_stat[w * WT * TILE + i]);
      if (tok0 + i < n_rows)
        *reinterpret_cast<f32x4*>(part + ((int64_t)row_of(tok0 + i) * n_parts + tgroup) * 4) = f32x4{a.m, a.s, __int_as_float(a.id), 0.f};
    }
  }
  TRACE_MARK(KID, 7);
  }
}

// ------------------------------------------------------------------------------------------------
// LM head, form of five and six token tiles (where: lm_half): half a task (32 vocabulary ids, one weight tile) per wave, four tasks
// per workgroup, the high plane as in the form above, statistics of a task's two halves put together at the end (with a fold of two
// partials instead, 1 to 2 us less and confidences 4e-8 off the form above).  Bound by what a compute unit
// takes in (1 MB of weights and as much as 0.75 MB of rows per workgroup) and the last, partial round of workgroups (2.4 rounds of them at
// 157184 ids).  Twelve k-steps of weights in flight per wave: 16, 24 or 32 were slower at 160 tokens (140.8 us, 144.5, 150, 211: loads return
// in order, so that the rows on their way to LDS wait behind them), 8 as fast (141.1); rows requested two chunks ahead 160 against 155.
// ------------------------------------------------------------------------------------------------
constexpr int LMH_WW = 8, LMH_WT = 6, LMH_TASKS = LMH_WW / 2;      // waves, token tiles and tasks of a workgroup
constexpr int LMH_KC = 4, LMH_PRE = 3, LMH_NB = 3;                 // as WideShape's KC, PRE, NB
template <typename E> constexpr size_t lm_half_lds() { return (size_t)LMH_NB * LMH_KC * LMH_WT * WidePieces<E, 9>::TILE_VECS * 16; }

// acc[t] += the wave's tile times token tile t, NT tiles, over ksteps k-steps (a multiple of LMH_KC).  w: the tile's k-step 0;
// row_of(tile, r): activation row; SN tiles are staged, an even number of at least NT: wave w stages half of them for k-step w / 2 of
// every chunk.
template <typename E, int NT, int SN, class RowOf>
__device__ inline void lm_half_stream(const E* __restrict__ w, int ksteps, const E* __restrict__ act, RowOf&& row_of, int64_t bkstride,
                                      typename ET<E>::vec* sb, f32x16 (&acc)[NT], int wave) {
  typedef typename ET<E>::vec vec;
  typedef WidePieces<E, 9> Pc;
  static_assert(Pc::N == 2 && Pc::ROWS == TILE && LMH_KC * 2 == LMH_WW && SN % 2 == 0 && SN >= NT, "a load is a k-step of a whole tile");
  constexpr int KC = LMH_KC, PRE = LMH_PRE, NB = LMH_NB, PP = SN / 2;
  constexpr int STEP = 2 * WAVE * 16, ROW_BYTES = 32, BUF = KC * SN * Pc::TILE_VECS;
  const int lane = threadIdx.x & 63, n_chunks = ksteps / KC, last = n_chunks - 1;
  const uint32_t wlane = lane * 16;
  auto wload = [&](int c, int ks) { return load16_stream<E>((const E*)((const char*)w + (int64_t)(min(c, last) * KC + ks) * STEP + wlane)); };
  vec wa[PRE][KC], bset[PP];
  const int pks = wave >> 1, ptile = (wave & 1) * PP;
  uint32_t src[PP];
#pragma unroll
  for (int j = 0; j < PP; ++j) src[j] = (uint32_t)row_of(ptile + j, lane >> 1) * ROW_BYTES + (lane & 1) * 16;
#pragma unroll
  for (int i = 0; i < PRE; ++i)
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) wa[i][ks] = wload(i, ks);
  const int dst = (pks * SN + ptile) * Pc::TILE_VECS + Pc::slot(lane >> 1, lane & 1);
  auto fetch = [&](int c, vec (&b)[PP]) {
    const char* base = (const char*)(act + (int64_t)(min(c, last) * KC + pks) * bkstride);
#pragma unroll
    for (int j = 0; j < PP; ++j) b[j] = load16<E>((const E*)(base + src[j]));
  };
  auto put = [&](int buf, const vec (&b)[PP]) {
#pragma unroll
    for (int j = 0; j < PP; ++j) sb[buf + dst + j * Pc::TILE_VECS] = b[j];
  };
  {
    vec b0[NB - 1][PP];
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) fetch(i, b0[i]);
    fetch(NB - 1, bset);
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) put(i * BUF, b0[i]);
  }
  const int rd = Pc::slot(lane & 31, lane >> 5);
  constexpr int F = KC * NT, FD = 4;
  vec ring[FD];
  auto frag = [&](int buf, int f) { return sb[buf + ((f / NT) * SN + f % NT) * Pc::TILE_VECS + rd]; };
  int cur = 0;
  __syncthreads();
  static_for<FD>([&](auto J) { ring[decltype(J)::value] = frag(0, decltype(J)::value); });
  auto chunk = [&](auto I, int c) {
    constexpr int i = decltype(I)::value;
    __syncthreads();
    const int nxt = cur + BUF < NB * BUF ? cur + BUF : 0;
    put(nxt + BUF < NB * BUF ? nxt + BUF : 0, bset);
    fetch(c + NB, bset);
    static_for<F>([&](auto Fi) {
      constexpr int f = decltype(Fi)::value, ks = f / NT, t = f % NT;
      const vec b = ring[f % FD];
      if constexpr (f + FD < F) ring[f % FD] = frag(cur, f + FD);
      else ring[f % FD] = frag(nxt, f + FD - F);
      __builtin_amdgcn_sched_barrier(0);
      mfma32(acc[t], wa[i][ks], b);
    });
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) wa[i][ks] = wload(c + PRE, ks);
    cur = nxt;
  };
  int c0 = 0;       // whole rounds without a test between the chunks, the first one in front of the loop: see wide_stream_nt
  if (n_chunks >= PRE) {
    static_for<PRE>([&](auto I) { chunk(I, decltype(I)::value); });
    for (c0 = PRE; c0 + PRE <= n_chunks; c0 += PRE) static_for<PRE>([&](auto I) { chunk(I, c0 + decltype(I)::value); });
  }
  static_for<PRE - 1>([&](auto I) {
    if (c0 + decltype(I)::value < n_chunks) chunk(I, c0 + decltype(I)::value);   // uniform over the workgroup
  });
}

template <typename E>
__global__ __launch_bounds__(LMH_WW * WAVE) __attribute__((amdgpu_waves_per_eu(2))) void lm_head_half_kernel(const E* __restrict__ W, const E* __restrict__ xn,
                                                                  RowNorm norm, int T, int H, int V, float scale, float* __restrict__ part,
                                                                  float* __restrict__ logits_out, const int32_t* __restrict__ rows, int n_tasks,
                                                                  int n_parts, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  __shared__ __align__(16) float s_scale[LMH_WT * TILE];
  __shared__ __align__(16) int32_t s_row[LMH_WT * TILE];
  constexpr int KS = ET<E>::KS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int n_rows = rows ? min(rows[0], T) : T;
  if (n_rows == 0) return;              // uniform over the workgroup
  const int tiles = (n_rows + TILE - 1) / TILE, groups = (tiles + LMH_WT - 1) / LMH_WT, per_group = (tiles + groups - 1) / groups;
  const int turn = blockIdx.x / XCDS, tgroup = (turn / groups) * XCDS + blockIdx.x % XCDS, tile0 = (turn % groups) * per_group;
  if (tgroup * LMH_TASKS >= n_parts) return;
  const int nt = min(per_group, tiles - tile0);
  if (nt <= 0) return;                  // uniform: fewer tiles than groups * per_group
  const int slot = tgroup * LMH_TASKS + (wave >> 1), task = min(slot, n_tasks - 1), ksteps = H / KS, tok0 = tile0 * TILE;
  auto row_of = [&](int i) { return rows ? min(max(rows[1 + min(i, n_rows - 1)], 0), T - 1) : min(i, T - 1); };
  if (threadIdx.x < LMH_WT * TILE) {    // read behind the stream's barriers
    const int row = row_of(tok0 + threadIdx.x);
    s_row[threadIdx.x] = row;
    s_scale[threadIdx.x] = row_rinv(norm.ssq, norm.n_ssq, T, row, H, norm.eps) * scale;
  }
  const bool quads = V % 4 == 0 && ((uintptr_t)logits_out & 15) == 0;   // rows of logits start on 16-byte boundaries
  // Statistics of a task's two halves, once the fragments are done with, in the order of a lane that has both (lm_head_wide_kernel): the
  // maximum of either half to the other's wave, exponentials against that of both, and the sum runs on from the first half's into the second's.
  float* s_max = reinterpret_cast<float*>(lds_raw);                    // [wave][tile][lane]
  float* s_sum = s_max + LMH_WW * LMH_WT * WAVE;                       // [task][tile][lane]
  int32_t* s_id = reinterpret_cast<int32_t*>(s_sum + LMH_TASKS * LMH_WT * WAVE);
  static_assert((LMH_WW + 2 * LMH_TASKS) * LMH_WT * WAVE * 4 <= lm_half_lds<E>(), "they fit the staging area");
  auto run = [&](auto N, auto S) {
    constexpr int NT = decltype(N)::value, SN = decltype(S)::value;
    f32x16 acc[NT];
    zero_acc<NT>(acc);
    lm_half_stream<E, NT, SN>(W + (int64_t)task * task_stride_elems<E>(ksteps) + (wave & 1) * (WAVE * ET<E>::G), ksteps, xn,
                              [&](int t, int r) { return row_of(tok0 + t * TILE + r); }, (int64_t)T * KS, reinterpret_cast<vec*>(lds_raw), acc, wave);
    __syncthreads();                    // the staged fragments have been read by every wave
    const int id0 = (2 * task + (wave & 1)) * TILE + 4 * half, pair = (wave >> 1) * LMH_WT;
    float m[NT];
    int best[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float zs = s_scale[t * TILE + col];
      f32x16& z = acc[t];
      m[t] = -INFINITY;
      best[t] = 0x7fffffff;
      if (slot < n_tasks) {             // the maximum first, then the lowest id that has it: see lm_head_wide_kernel
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] *= zs;
        if ((2 * task + (wave & 1) + 1) * TILE > V) {   // uniform
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (id0 + acc_row(i, 0) >= V) z[i] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) m[t] = fmaxf(m[t], z[i]);   // passes over NaN
        int at = 0;
#pragma unroll
        for (int i = 15; i >= 0; --i) at = z[i] == m[t] ? acc_row(i, 0) : at;
        if (m[t] > -INFINITY) best[t] = id0 + at;
        if (logits_out && tok0 + t * TILE + col < n_rows) {
          float* out = logits_out + (int64_t)s_row[t * TILE + col] * V + id0;
          if (quads) {
#pragma unroll
            for (int i = 0; i < 16; i += 4)
              if (id0 + acc_row(i, 0) < V) *reinterpret_cast<f32x4*>(out + acc_row(i, 0)) = f32x4{z[i], z[i + 1], z[i + 2], z[i + 3]};
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (id0 + acc_row(i, 0) < V) out[acc_row(i, 0)] = z[i];
          }
        }
      }
      s_max[(wave * LMH_WT + t) * WAVE + lane] = m[t];
    }
    __syncthreads();
    float sum[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float other = s_max[((wave ^ 1) * LMH_WT + t) * WAVE + lane], both = fmaxf(m[t], other);
      if (wave & 1 ? other == both : m[t] < both) best[t] = 0x7fffffff;   // of two halves that have it the first one's id is lower
      m[t] = both;
      sum[t] = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = both > -INFINITY ? __expf(acc[t][i] - both) : 0.f;
      if (!(wave & 1)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[t] += acc[t][i];
        s_sum[(pair + t) * WAVE + lane] = sum[t];
        s_id[(pair + t) * WAVE + lane] = best[t];
      }
    }
    __syncthreads();
    if (!(wave & 1)) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      sum[t] = s_sum[(pair + t) * WAVE + lane];
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[t] += acc[t][i];
      best[t] = min(best[t], s_id[(pair + t) * WAVE + lane]);
      const LmStat w = lm_combine(LmStat{m[t], sum[t], best[t]}, LmStat{__shfl_xor(m[t], 32, WAVE), __shfl_xor(sum[t], 32, WAVE), __shfl_xor(best[t], 32, WAVE)});
      const int i = t * TILE + col;
      if (half == 0 && t < nt && tok0 + i < n_rows)
        *reinterpret_cast<f32x4*>(part + ((int64_t)s_row[i] * n_parts + slot) * 4) = f32x4{w.m, w.s, __int_as_float(w.id), 0.f};
    }
  };
  if (nt > 5) run(std::integral_constant<int, 6>{}, std::integral_constant<int, 6>{});
  else if (nt == 5) run(std::integral_constant<int, 5>{}, std::integral_constant<int, 6>{});
  else run(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
}

// Up to 64 tokens: one or two token tiles per workgroup and both activation planes (trace ids 15, 14): there the weight
// stream is the bound, and sharing the activation fragments relieves the address unit, which would otherwise take every
// lane's own activation row one by one.  (33 to 64 tokens in workgroups of two tasks: 144 against 119 us, the fragments
// of 64 rows are shared by too few.)  More tokens: four tiles, high plane only (id 9).
template <int WW, int WT> constexpr size_t lm_piece_lds() { return (size_t)WW * 2 * WT * 16 * WAVE * 4; }
template <typename E> static void launch_lm_wide_t(const LmArgs& a, hipStream_t st) {
  const LmPlan p = lm_plan(a.V, a.T);
  const int groups = a.T <= 2 * TILE ? 1 : (a.T + WT * TILE - 1) / (WT * TILE);
  const int wgs = (p.whole + p.tasks - p.first_piece + XCDS - 1) / XCDS * XCDS * groups;
  const void* xn = lm_compact(Planes<E>::N > 1, a.T) ? a.xn_hi : a.xn;
  auto go = [&](auto kernel, int ww, size_t lds) {
    kernel<<<wgs, ww * WAVE, lds, st>>>((const E*)a.w, (const E*)xn, a.norm, a.T, a.H, a.V, a.scale, a.part, a.logits_out, a.rows,
                                        p, live_word());
  };
  if (a.T <= TILE) {
    if (p.ww == LM_PIECE_WW) go(lm_head_wide_kernel<E, 1, 15, LM_PIECE_WW>, LM_PIECE_WW, lm_piece_lds<LM_PIECE_WW, 1>());
    else go(lm_head_wide_kernel<E, 1, 15, LM_SMALL_WW>, LM_SMALL_WW, wide_lds<E, 15, 1>());
  } else if (a.T <= 2 * TILE) {
    if (p.ww == LM_PIECE_WW) go(lm_head_wide_kernel<E, 2, 14, LM_PIECE_WW>, LM_PIECE_WW, lm_piece_lds<LM_PIECE_WW, 2>());
    else go(lm_head_wide_kernel<E, 2, 14, LM_MID_WW>, LM_MID_WW, lm_piece_lds<LM_MID_WW, 2>());
  } else {
    if constexpr (sizeof(E) == 2) {
      if (lm_half(true, a.T)) {
        const int half_wgs = (p.parts / LMH_TASKS + XCDS - 1) / XCDS * XCDS * ((a.T + LMH_WT * TILE - 1) / (LMH_WT * TILE));
        lm_head_half_kernel<E><<<half_wgs, LMH_WW * WAVE, lm_half_lds<E>(), st>>>((const E*)a.w, (const E*)xn, a.norm, a.T, a.H, a.V, a.scale, a.part, a.logits_out,
                                                                                 a.rows, p.tasks, p.parts, live_word());
        return;
      }
    }
    go(lm_head_wide_kernel<E, WT, 9, LM_WW>, LM_WW, wide_lds<E, 9, WT>());
  }
}
void launch_lm_head_wide(bool bf16, const LmArgs& a, hipStream_t st) {
  if (bf16) launch_lm_wide_t<bf16_t>(a, st);
  else launch_lm_wide_t<float>(a, st);
}

bool configure_wide() {
  auto opt_in = [](const void* f, int bytes) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess; };
  const void* many[12] = {(const void*)expert_many_kernel<bf16_t, WT, EXPERT_WW, 25, GateUp<bf16_t>>,
                         (const void*)expert_many_kernel<float, WT, EXPERT_WW, 25, GateUp<float>>,
                         (const void*)expert_many_kernel<bf16_t, WT, EXPERT_WW, 26, Down<bf16_t>>,
                         (const void*)expert_many_kernel<float, WT, EXPERT_WW, 26, Down<float>>,
                         (const void*)expert_many_kernel<bf16_t, WT, EXPERT_WW, 10, GateUp<bf16_t>>,
                         (const void*)expert_many_kernel<float, WT, EXPERT_WW, 10, GateUp<float>>,
                         (const void*)expert_many_kernel<bf16_t, WT, EXPERT_WW, 11, Down<bf16_t>>,
                         (const void*)expert_many_kernel<float, WT, EXPERT_WW, 11, Down<float>>,
                         (const void*)expert_pieces_kernel<bf16_t, 2, GateUp<bf16_t>>, (const void*)expert_pieces_kernel<float, 2, GateUp<float>>,
                         (const void*)expert_pieces_kernel<bf16_t, 2, Down<bf16_t>>, (const void*)expert_pieces_kernel<float, 2, Down<float>>};
  for (const void* f : many)
    if (!opt_in(f, (int)many_lds<EXPERT_WW>())) return false;
  const void* pieces[4] = {(const void*)lm_head_wide_kernel<bf16_t, 1, 15, LM_PIECE_WW>, (const void*)lm_head_wide_kernel<float, 1, 15, LM_PIECE_WW>,
                           (const void*)lm_head_wide_kernel<bf16_t, 2, 14, LM_PIECE_WW>, (const void*)lm_head_wide_kernel<float, 2, 14, LM_PIECE_WW>};
  for (const void* f : pieces)
    if (!opt_in(f, 128 * 1024)) return false;
  return opt_in((const void*)lm_head_half_kernel<bf16_t>, (int)lm_half_lds<bf16_t>()) && opt_in((const void*)lm_head_wide_kernel<bf16_t, WT, 9, LM_WW>, 128 * 1024) &&
         opt_in((const void*)lm_head_wide_kernel<float, WT, 9, LM_WW>, 128 * 1024);
}

TRACE_READER(trace_read_wide)

}  // namespace dinfer
