// Bidirectional (non-causal) attention of a tile of 32 query tokens over every key of its sequence: the
// cached prefix pages plus the tokens of this forward, read through the page table.
//
// Work split: grid (split, head, query tile), ATTN_WAVES waves per workgroup.  A sequence uses as many of the
// grid's splits as its own key count asks for (attn_splits_for; the other workgroups exit at once), and its key
// tiles (32 keys) are dealt round-robin to the waves of those splits.  Each wave keeps its own online-softmax
// state; the waves of a workgroup are folded through LDS in wave order, each wave finishing its share of the
// output rows.  With one split the workgroup writes the normalised output itself; otherwise it leaves one
// partial (unnormalised output, max, sum) and takes an arrival ticket of its (query tile, head); the workgroup
// that arrives last folds the partials in split order and writes the output.
//
// MFMA mapping (32x32 tiles):  S^T[key][query] = K_tile . Q^T   (A = K rows, B = Q columns), so a lane owns
// one query column and softmax statistics are per lane;  O^T[d][query] += V^T_tile . P^T  (A = V^T rows read
// from the transposed V page, B = P^T taken from the S^T accumulator registers without any shuffle).
#include <type_traits>

#include "gemm.hpp"
#include "kernels.hpp"

namespace dinfer {

constexpr int ATTN_WAVES = 8;
constexpr int ATTN_FETCH_MAX_OWN = 64;   // launches with at most this many workgroups of their own also fetch AttnArgs::pf

size_t attn_part_floats(int n_qtiles, int n_heads, int n_splits, int head_dim) {
  return (size_t)n_qtiles * n_heads * n_splits * TILE * (head_dim + 2);
}

// B operand of the PV product for k-step s2: the G probabilities this lane holds for that step's keys, and
// the matching A operand (V^T of those keys for feature row d).  key_of_row: which of a tile's 32 keys row r of the
// score tile stands for (any assignment will do, as the softmax does not care); key_of_acc: the tile-local key of
// accumulator register v.
template <typename E> struct PvStep;
template <> struct PvStep<bf16_t> {
  // Bits 2 and 3 of the row are swapped, so that the eight registers 8*s2 .. 8*s2+7 of half h hold the consecutive keys
  // 16*s2 + 8h .. +7 and their V^T entries are one 16-byte load (with rows in key order they are two 8-byte loads
  // eight keys apart, twice as many instructions for the address unit).
  static constexpr int STEPS = 2;
  __device__ static int key_of_row(int r) { return (r & 19) | ((r & 4) << 1) | ((r & 8) >> 1); }
  __device__ static int key_of_acc(int v, int half) { return 16 * (v >> 3) + 8 * half + (v & 7); }
  // plane 0: bf16(p); plane 1: bf16(p - plane 0)
  __device__ static bf16x8 p_vec(const float (&p)[16], int s2, int plane) {
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bf16_t hi = (bf16_t)p[8 * s2 + i];
      r[i] = plane == 0 ? hi : (bf16_t)(p[8 * s2 + i] - (float)hi);
    }
    return r;
  }
  // vrow: V^T row of feature d inside the page of this step (16 slots contiguous)
  __device__ static bf16x8 v_vec(const bf16_t* vrow, int half, int /*s2*/) { return load16<bf16_t>(vrow + 8 * half); }
  __device__ static int page_of_step(int s2) { return s2; }
  __device__ static int key_of(int s2, int half, int i) { return 16 * s2 + 8 * half + i; }
};
template <> struct PvStep<float> {
  // step s2 in {0..3}: registers 4*s2 .. 4*s2+3 -> keys 8*s2 + 4h + {0..3}
  static constexpr int STEPS = 4;
  __device__ static int key_of_row(int r) { return r; }
  __device__ static int key_of_acc(int v, int half) { return acc_row(v, half); }
  __device__ static f32x4 p_vec(const float (&p)[16], int s2, int /*plane*/) {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = p[4 * s2 + i];
    return r;
  }
  __device__ static f32x4 v_vec(const float* vrow, int half, int s2) {
    return *reinterpret_cast<const f32x4*>(vrow + 8 * (s2 & 1) + 4 * half);
  }
  __device__ static int page_of_step(int s2) { return s2 >> 1; }
  __device__ static int key_of(int s2, int half, int i) { return 8 * s2 + 4 * half + i; }
};

// NS key tiles of the online softmax: scores sacc (16 keys of the lane's query each, the other half-wave holds the
// other 16) -> probabilities p, with the lane's reference maximum m_run, its sum l_run and the output o kept up.  Softmax
// statistics live in the log2 domain (c2 = scale * log2(e), one fused multiply-add in front of the exponential).  A
// lane's reference maximum moves only when a tile's maximum passes it by more than REF_SLACK: probabilities are then
// bounded by 2^REF_SLACK instead of 1, which float32 sums and the bf16 hi + lo planes hold just as well, and the output
// registers are rescaled only in the rare tile where some lane's reference moves (a wave-uniform branch), not in
// every tile.
constexpr float REF_SLACK = 6.f;
template <int DT, int NS>
__device__ inline void online_softmax(const f32x16 (&sacc)[NS], float c2, float& m_run, float& l_run, f32x16 (&o)[DT],
                                      float (&p)[NS][16]) {
  float mx = sacc[0][0];
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[n][v]);
  mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));      // the other half-wave holds the column's other keys
  const float mt = mx * c2;                       // finite: a key tile always holds at least one valid key
  const bool moves = mt > m_run + REF_SLACK;      // (m_run = -inf before the wave's first tile)
  if (__builtin_amdgcn_ballot_w64(moves)) {
    const float m_new = moves ? mt : m_run;
    const float alpha = moves ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;
    l_run *= alpha;
    m_run = m_new;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[t][v] *= alpha;
  }
  float psum = 0.f;
#pragma unroll
  for (int n = 0; n < NS; ++n)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[n][v] = __builtin_amdgcn_exp2f(fmaf(sacc[n][v], c2, -m_run));
      psum += p[n][v];
    }
  l_run += psum;
}

template <typename E, int HD>
__global__ __launch_bounds__(ATTN_WAVES * WAVE) void attention_kernel(const E* __restrict__ Q, int64_t q_plane,
                                                         const E* __restrict__ kv_layer, KvGeom geom, FwdMeta meta,
                                                         const int32_t* __restrict__ page_table, int pt_stride,
                                                         int n_splits, float* __restrict__ part,
                                                         int32_t* __restrict__ tickets, E* __restrict__ out,
                                                         int T_out, int n_qtiles, L2Prefetch pf,
                                                         const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  if ((int)blockIdx.z >= n_qtiles) {
    // not an attention workgroup: one that fetches a region of a later launch's weights into this die's L2
    const int index = (int)((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
    const int region = index - l2_prefetch_first(n_qtiles * gridDim.y * gridDim.x);
    if (region >= 0 && region < pf.n_regions) l2_fetch(pf.base + (size_t)region * pf.region_bytes, pf.region_bytes);
    return;
  }
  typedef typename ET<E>::vec vec;
  constexpr int G = ET<E>::G, KS = ET<E>::KS, DSTEPS = HD / KS, DT = HD / TILE, NP = Planes<E>::N;
  const int split = blockIdx.x, head = blockIdx.y, qt = blockIdx.z;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int seq = meta.qtile[qt * 3 + 0], tok0 = meta.qtile[qt * 3 + 1], nvalid = meta.qtile[qt * 3 + 2];
  const int n_keys = meta.seq_nkeys[seq];
  const int my_splits = min(attn_splits_for(n_keys), n_splits);   // splits this sequence uses of those the grid offers
  if (split >= my_splits) return;                                  // uniform over the workgroup
  const int D = geom.n_heads * HD;
  const float scale = rsqrtf((float)HD);
  TRACE_MARK(7, 0);
  // The sequence's page-table row goes to LDS first: a tile's K / V addresses then need no global round trip
  // of their own, and the loads of the next tile can be issued at once.
  __shared__ int32_t pt[ATTN_MAX_PAGES];
  {
    const int32_t* row = page_table + (int64_t)seq * pt_stride;
    const int n_pages_used = (n_keys + PAGE - 1) / PAGE;       // <= pt_stride, <= ATTN_MAX_PAGES (host checks)
    for (int i = threadIdx.x; i < n_pages_used; i += blockDim.x) pt[i] = row[i];
  }

  // Q^T operand (queries and probabilities enter the MFMAs as hi + lo planes when E is bf16, like every
  // activation): all waves use the same query tile, so it is staged once in LDS in operand order
  // [head_dim k-step][plane][lane] and read from there in the tile loop instead of living in registers.
  __shared__ vec qs[DSTEPS * NP * WAVE];
  {
    const E* qrow = Q + (int64_t)(tok0 + min(col, nvalid - 1)) * D + head * HD + half * G;
    for (int i = wave; i < DSTEPS * NP; i += ATTN_WAVES)
      qs[i * WAVE + lane] = load16<E>(qrow + (i % NP) * q_plane + (i / NP) * KS);
  }
  __syncthreads();
  TRACE_MARK(7, 1);
  f32x16 o[DT];
  zero_acc<DT>(o);
  float m_run = -INFINITY, l_run = 0.f;

  const int n_ktiles = (n_keys + TILE - 1) / TILE;
  const int stride = my_splits * ATTN_WAVES;             // key tiles are dealt round-robin to all its waves
  const int kt0 = split * ATTN_WAVES + wave;
  // K rows and V^T rows of one key tile, loaded straight into MFMA operand registers
  struct TileRegs {
    vec k[DSTEPS];
    vec v[PvStep<E>::STEPS][DT];
  };
  auto load_tile = [&](int kt, TileRegs& r) {
    const int key = min(kt * TILE + PvStep<E>::key_of_row(col), n_keys - 1);
    const E* krow = kv_layer + kv_k_index(geom, safe_page(geom, pt[key / PAGE]), head, key % PAGE, 0) + half * G;
#pragma unroll
    for (int s = 0; s < DSTEPS; ++s) r.k[s] = load16<E>(krow + s * (PAGE * KS));   // k-step s of this slot
#pragma unroll
    for (int s2 = 0; s2 < PvStep<E>::STEPS; ++s2) {
      const int pkey = min(kt * TILE + PvStep<E>::page_of_step(s2) * PAGE, n_keys - 1);
      const int page = safe_page(geom, pt[pkey / PAGE]);
#pragma unroll
      for (int t = 0; t < DT; ++t)
        r.v[s2][t] = PvStep<E>::v_vec(kv_layer + kv_v_index(geom, page, head, 0, t * TILE + col), half, s2);
    }
  };
  const float c2 = scale * 1.44269504088896341f;
  auto use_tile = [&](TileRegs& cur, int kt) {
    // ---- S^T = K . Q^T  (the compiler barrier keeps the query reads inside the loop: hoisted, they would
    // occupy the 64 registers that staging them in LDS is meant to free)
    asm volatile("" ::: "memory");
    f32x16 sacc[1];
    zero_acc<1>(sacc);
    {
      // the query fragments are read from LDS QD ahead of the matrix instructions that use them; the scheduling
      // barrier keeps the compiler from moving the reads back next to their use
      constexpr int QF = DSTEPS * NP, QD = 3;
      vec ring[QD];
#pragma unroll
      for (int f = 0; f < QD; ++f) ring[f] = qs[f * WAVE + lane];
#pragma unroll
      for (int f = 0; f < QF; ++f) {
        const vec b = ring[f % QD];
        if (f + QD < QF) ring[f % QD] = qs[(f + QD) * WAVE + lane];
        __builtin_amdgcn_sched_barrier(0);
        mfma32(sacc[0], cur.k[f / NP], b);
      }
    }
    if ((kt + 1) * TILE > n_keys) {
      // the sequence's last, ragged tile (wave-uniform, at most once per wave; the empty asm keeps it a branch):
      // scores of slots past the last key become -inf, and their V entries, which may hold anything (NaN * 0
      // would poison the sum), become 0
      asm volatile("" ::: "memory");
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (kt * TILE + PvStep<E>::key_of_acc(v, half) >= n_keys) sacc[0][v] = -INFINITY;
#pragma unroll
      for (int s2 = 0; s2 < PvStep<E>::STEPS; ++s2)
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int i = 0; i < G; ++i)
            if (kt * TILE + PvStep<E>::key_of(s2, half, i) >= n_keys) cur.v[s2][t][i] = (E)0.f;
    }
    float p[1][16];
    online_softmax<DT, 1>(sacc, c2, m_run, l_run, o, p);
    // ---- O^T += V^T . P^T
#pragma unroll
    for (int s2 = 0; s2 < PvStep<E>::STEPS; ++s2) {
      vec pv[NP];
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) pv[pl] = PvStep<E>::p_vec(p[0], s2, pl);
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) mfma32(o[t], cur.v[s2][t], pv[pl]);
    }
  };
  // Two tile buffers that swap roles (the loop is unrolled by two, so no registers are copied): the next tile's
  // loads are issued before this tile is used, clamped, so that no branch surrounds loads and the compiler can
  // count them; a wave's last turn re-reads its own tile.
  TileRegs ta, tb;
  if (kt0 < n_ktiles) load_tile(kt0, ta);
  for (int kt = kt0; kt < n_ktiles; kt += 2 * stride) {
    load_tile(min(kt + stride, n_ktiles - 1), tb);
    use_tile(ta, kt);
    if (kt + stride >= n_ktiles) break;
    load_tile(min(kt + 2 * stride, n_ktiles - 1), ta);
    use_tile(tb, kt + stride);
  }
  TRACE_MARK(7, 2);
  // ---- fold the waves through LDS (lane-major, conflict free): every wave leaves its state, then wave w
  // finishes RPW of the DT*16 accumulator registers, summed over the waves in wave order
  extern __shared__ float lds[];                       // [ATTN_WAVES][DT*16 + 2][64 lanes]
  constexpr int PW = (DT * 16 + 2) * WAVE, RPW = DT * 16 / ATTN_WAVES;
  static_assert(RPW % 4 == 0, "a wave finishes whole groups of four accumulator registers");
  {
    float* pb = lds + wave * PW + lane;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) pb[(t * 16 + v) * WAVE] = o[t][v];
    pb[(DT * 16) * WAVE] = m_run;
    pb[(DT * 16 + 1) * WAVE] = l_run + __shfl_xor(l_run, 32, WAVE);
  }
  __syncthreads();
  TRACE_MARK(7, 3);
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < ATTN_WAVES; ++w) M = fmaxf(M, lds[w * PW + (DT * 16) * WAVE + lane]);
  float L = 0.f;
  float r[RPW];
#pragma unroll
  for (int i = 0; i < RPW; ++i) r[i] = 0.f;
#pragma unroll
  for (int w = 0; w < ATTN_WAVES; ++w) {
    const float* pb = lds + w * PW + lane;
    const float mw = pb[(DT * 16) * WAVE];
    const float sw = mw > -INFINITY ? __builtin_amdgcn_exp2f(mw - M) : 0.f;   // a wave that saw no key tile contributes nothing
    L += sw * pb[(DT * 16 + 1) * WAVE];
#pragma unroll
    for (int i = 0; i < RPW; ++i) r[i] += sw * pb[(wave * RPW + i) * WAVE];
  }
  if (my_splits == 1) {
    // the whole key range was here: normalise and write the attention output
    if (col < nvalid) {
      const float inv = 1.f / L;
#pragma unroll
      for (int i4 = 0; i4 < RPW / 4; ++i4) {   // four accumulator registers = four consecutive features
        const int g = wave * RPW + 4 * i4;
        const f32x4 o = {r[4 * i4] * inv, r[4 * i4 + 1] * inv, r[4 * i4 + 2] * inv, r[4 * i4 + 3] * inv};
        store_actk4<E>(out, T_out, tok0 + col, head * HD + (g / 16) * TILE + acc_row(g % 16, half), o);
      }
    }
    TRACE_MARK(7, 4);
    return;
  }
  // partial of this split: O [32 q][HD] (unnormalised), (m, l) [32], handed over with device-coherent stores
  const int pair = qt * geom.n_heads + head;
  const buf_rsrc pr = coherent_buffer(part);
  const uint32_t pair_bytes = (uint32_t)pair * n_splits * TILE * (HD + 2) * 4, part_bytes = TILE * (HD + 2) * 4;
  {
    const uint32_t pb = pair_bytes + split * part_bytes;
#pragma unroll
    for (int i4 = 0; i4 < RPW / 4; ++i4) {
      const int g = wave * RPW + 4 * i4;
      const float v4[4] = {r[4 * i4], r[4 * i4 + 1], r[4 * i4 + 2], r[4 * i4 + 3]};
      coherent_store_n<4>(pr, pb + (col * HD + (g / 16) * TILE + acc_row(g % 16, half)) * 4, v4);
    }
    if (wave == 0 && half == 0) {
      const float ml[2] = {M, L};
      coherent_store_n<2>(pr, pb + (TILE * HD + 2 * col) * 4, ml);
    }
  }
  __shared__ int32_t s_flag;
  if (!last_arrival(tickets + pair, my_splits, &s_flag)) return;
  // Last to arrive: fold the partials in split order, each weighted against the maximum of all, by fused adds (as written: a product that
  // the compiler rounds first is another last bit of every row).  A thread takes ITEMS (query, 4 consecutive features) items.  The loads
  // of N splits are under way together; they bypass the L2, so that one compute unit's fetch is the bound, and no more are issued than
  // for two, four, eight or sixteen splits (sixteen clamped loads for every count -> this: two splits, 64 tokens behind 768 keys 19.0 ->
  // 16.0 us for the launch, 12 sequences of 32 40.0 -> 36.8; eight splits of 4096 keys 22.4 -> 21.0;
  // sixteen of 8000 25.6 -> 26.5, in two rounds of eight 26.7).  Nor for rows past the tile's last query: one token behind 8000 keys
  // 20.6, with the loads of all 32 rows 23.5.
  constexpr int ITEMS = TILE * HD / 4 / (ATTN_WAVES * WAVE);
  static_assert(ITEMS * ATTN_WAVES * WAVE == TILE * HD / 4, "whole items per thread");
  auto item_q = [&](int i) { return (int)(threadIdx.x + i * ATTN_WAVES * WAVE) / (HD / 4); };
  auto item_d = [&](int i) { return (int)(threadIdx.x + i * ATTN_WAVES * WAVE) % (HD / 4) * 4; };
  float Ls[ITEMS];
  f32x4 acc[ITEMS];
  auto fold = [&](auto C) {
    constexpr int N = decltype(C)::value;
    float ml[ITEMS][N][2], op[ITEMS][N][4];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (item_q(i) >= nvalid) continue;
#pragma unroll
      for (int p = 0; p < N; ++p) {
        const uint32_t pb = pair_bytes + min(p, my_splits - 1) * part_bytes;
        coherent_load_n<2>(pr, pb + (TILE * HD + 2 * item_q(i)) * 4, ml[i][p]);
        coherent_load_n<4>(pr, pb + (item_q(i) * HD + item_d(i)) * 4, op[i][p]);
      }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      Ls[i] = 0.f;
      acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (item_q(i) >= nvalid) continue;
      float Mx = -INFINITY;
#pragma unroll
      for (int p = 0; p < N; ++p) Mx = p < my_splits ? fmaxf(Mx, ml[i][p][0]) : Mx;
#pragma unroll
      for (int p = 0; p < N; ++p) {
        if (p < my_splits && ml[i][p][0] > -INFINITY) {   // (a split whose waves saw no key tile contributes nothing)
          const float w = __builtin_amdgcn_exp2f(ml[i][p][0] - Mx);
          Ls[i] = __builtin_fmaf(w, ml[i][p][1], Ls[i]);
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[i][k] = __builtin_fmaf(w, op[i][p][k], acc[i][k]);
        }
      }
    }
  };
  if (my_splits == 2) fold(std::integral_constant<int, 2>{});
  else if (my_splits <= 4) fold(std::integral_constant<int, 4>{});
  else if (my_splits <= 8) fold(std::integral_constant<int, 8>{});
  else fold(std::integral_constant<int, ATTN_MAX_SPLITS>{});
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (item_q(i) >= nvalid) continue;
    const float inv = 1.f / Ls[i];
    store_actk4<E>(out, T_out, tok0 + item_q(i), head * HD + item_d(i), acc[i] * inv);
  }
}

// ------------------------------------------------------------------------------------------------
// Many query tiles of one sequence (prompts), bf16: a workgroup takes one head and ROWS_WAVES consecutive query tiles,
// one per wave, walks all keys of the sequence, and every key tile goes through LDS once for all of its waves (two
// tiles a turn, double buffered, the turn after next on its way in registers).  In the kernel above every query tile is a workgroup of its
// own whose waves split the keys: each fetches all K and V again (1.6 GB through the L2s for prompts of 1811, 333, 825
// and 1318 tokens: 169 us per layer, 136 in this form), and the waves' partial outputs meet in a fold through 136 KB of LDS.  Here a wave
// keeps its queries (both planes) and output in registers, nothing is folded, and two workgroups of four waves share
// a compute unit, so that one multiplies while the other waits at its barrier or works on its softmax.
// ------------------------------------------------------------------------------------------------
constexpr int ROWS_TOK = ROWS_WAVES * TILE;
static_assert(ROWS_TILE == TILE, "attn_rows_groups counts tiles of this size");

template <int HD>
__global__ __launch_bounds__(ROWS_WAVES * WAVE, 2) void attention_rows_kernel(
    const bf16_t* __restrict__ Q, int64_t q_plane, const bf16_t* __restrict__ kv_layer, KvGeom geom, FwdMeta meta, SeqSpan span,
    const int32_t* __restrict__ page_table, int pt_stride, bf16_t* __restrict__ out, int T_out, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef bf16_t E;
  typedef ET<E>::vec vec;
  constexpr int G = ET<E>::G, KS = ET<E>::KS, DSTEPS = HD / KS, DT = HD / TILE, NP = Planes<E>::N, STEPS = PvStep<E>::STEPS;
  constexpr int WF = DSTEPS;      // fragments a wave fetches of every pair of tiles: the K or the V fragments of one tile
  static_assert(DSTEPS == STEPS * DT && STEPS == 2 && ROWS_WAVES == 4, "two key tiles have four such sets");
  const int head = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  int seq = 0, group = blockIdx.y;
  for (; seq < span.n_seq - 1; ++seq) {      // uniform: which sequence the workgroup's queries belong to
    const int n = (span.off[seq + 1] - span.off[seq] + ROWS_TOK - 1) / ROWS_TOK;
    if (group < n) break;
    group -= n;
  }
  const int tok0 = span.off[seq] + group * ROWS_TOK + wave * TILE, nvalid = span.off[seq + 1] - tok0;   // <= 0: nothing for this wave
  const int n_keys = meta.seq_nkeys[seq], n_turns = (n_keys + 2 * TILE - 1) / (2 * TILE);
  const int D = geom.n_heads * HD;
  __shared__ int32_t pt[ATTN_MAX_PAGES];
  extern __shared__ __align__(16) char lds_kv[];
  auto kv = reinterpret_cast<vec(*)[4][WF][WAVE]>(lds_kv);   // [buffer][K of tile 0, K of tile 1, V of 0, V of 1][fragment][lane]
  {
    const int32_t* row = page_table + (int64_t)seq * pt_stride;
    const int n_pages_used = (n_keys + PAGE - 1) / PAGE;       // <= pt_stride, <= ATTN_MAX_PAGES (host checks)
    for (int i = threadIdx.x; i < n_pages_used; i += ROWS_WAVES * WAVE) pt[i] = row[i];
  }
  vec q[DSTEPS][NP];
  {
    const E* qrow = Q + (int64_t)max(span.off[seq], min(tok0 + col, span.off[seq + 1] - 1)) * D + head * HD + half * G;
#pragma unroll
    for (int s = 0; s < DSTEPS; ++s)
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) q[s][pl] = load16<E>(qrow + pl * q_plane + s * KS);
  }
  __syncthreads();
  // A turn takes two key tiles: one barrier, one reduction over the half-waves and one test of the reference maximum for
  // 64 keys, and two independent chains of score products.
  // A wave fetches the K (waves 0, 1) or the V fragments of one tile of the turn, in two halves: one is on its way
  // during the score products, the other during softmax and output products (all of them at once do not fit the 256
  // registers beside scores, queries and output).
  constexpr int HF = WF / 2;
  vec next[HF];
  const int sub = wave & 1;
  const bool fetch_k = wave < 2;
  auto fetch = [&](int turn, int h) {
    const int key0 = (2 * min(turn, n_turns - 1) + sub) * TILE;
    if (fetch_k) {
      const int key = min(key0 + PvStep<E>::key_of_row(col), n_keys - 1);
      const E* krow = kv_layer + kv_k_index(geom, safe_page(geom, pt[key / PAGE]), head, key % PAGE, 0) + half * G;
#pragma unroll
      for (int j = 0; j < HF; ++j) next[j] = load16<E>(krow + (h * HF + j) * (PAGE * KS));
    } else {   // half h of the V fragments is k-step h: the tile's page h
      const int page = safe_page(geom, pt[min(key0 + PvStep<E>::page_of_step(h) * PAGE, n_keys - 1) / PAGE]);
#pragma unroll
      for (int t = 0; t < HF; ++t) next[t] = PvStep<E>::v_vec(kv_layer + kv_v_index(geom, page, head, 0, t * TILE + col), half, h);
    }
  };
  auto put = [&](int turn, int h) {
    const int key0 = (2 * turn + sub) * TILE;
    if (!fetch_k && key0 + TILE > n_keys) {
      // the last, ragged tile: V entries past the last key may hold anything (NaN * 0 would poison the sum)
#pragma unroll
      for (int j = 0; j < HF; ++j)
#pragma unroll
        for (int i = 0; i < G; ++i)
          if (key0 + PvStep<E>::key_of(h, half, i) >= n_keys) next[j][i] = (E)0.f;
    }
#pragma unroll
    for (int j = 0; j < HF; ++j) kv[turn & 1][wave][h * HF + j][lane] = next[j];
  };
  f32x16 o[DT];
  zero_acc<DT>(o);
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = rsqrtf((float)HD) * 1.44269504088896341f;
  fetch(0, 0);
  put(0, 0);
  fetch(0, 1);
  put(0, 1);
  fetch(1, 0);
  // (past the last turn the fetches repeat it, and their fragments go to the buffer that is not read any more)
  for (int turn = 0; turn < n_turns; ++turn) {
    __syncthreads();       // this turn's tiles are in their buffer, and every wave has done with the other one
    const auto& tiles = kv[turn & 1];
    // LDS fragments are read RD ahead of the matrix instructions that use them (pinned by the scheduling barriers)
    constexpr int RD = 4, NF = 2 * DSTEPS;
    vec ring[RD];
    f32x16 sacc[2];
    zero_acc<2>(sacc);
#pragma unroll
    for (int f = 0; f < RD; ++f) ring[f] = tiles[f & 1][f >> 1][lane];
#pragma unroll
    for (int f = 0; f < NF; f += 2) {      // k-step f / 2 of both tiles
      const vec a0 = ring[f % RD], a1 = ring[(f + 1) % RD];
#pragma unroll
      for (int i = 0; i < 2; ++i) {        // behind the last K fragments the first of V
        const int n = f + i + RD;
        ring[(f + i) % RD] = n < NF ? tiles[n & 1][n >> 1][lane] : tiles[2][n - NF][lane];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) {
        mfma32(sacc[0], a0, q[f / 2][pl]);
        mfma32(sacc[1], a1, q[f / 2][pl]);
      }
    }
    put(turn + 1, 0);
    fetch(turn + 1, 1);
    if ((turn + 1) * 2 * TILE > n_keys) {
      asm volatile("" ::: "memory");       // keeps the rare turn behind a branch
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if ((2 * turn + n) * TILE + PvStep<E>::key_of_acc(v, half) >= n_keys) sacc[n][v] = -INFINITY;
    }
    float p[2][16];
    online_softmax<DT, 2>(sacc, c2, m_run, l_run, o, p);
#pragma unroll
    for (int u = 0; u < 2 * STEPS; ++u) {  // k-step u % STEPS of tile u / STEPS
      vec pv[NP];
#pragma unroll
      for (int pl = 0; pl < NP; ++pl) pv[pl] = PvStep<E>::p_vec(p[u / STEPS], u % STEPS, pl);
#pragma unroll
      for (int pl = 0; pl < NP; ++pl)      // plane by plane: neighbouring products go to different accumulators
#pragma unroll
        for (int t = 0; t < DT; ++t) {
          const int f = u * DT + t;
          mfma32(o[t], ring[f % RD], pv[pl]);
          if (pl == NP - 1 && f + RD < NF) ring[f % RD] = tiles[2 + (f + RD) / WF][(f + RD) % WF][lane];
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    put(turn + 1, 1);
    fetch(turn + 2, 0);
  }
  if (col < nvalid) {
    const float inv = 1.f / (l_run + __shfl_xor(l_run, 32, WAVE));
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 r = {o[t][4 * g] * inv, o[t][4 * g + 1] * inv, o[t][4 * g + 2] * inv, o[t][4 * g + 3] * inv};
        store_actk4<E>(out, T_out, tok0 + col, head * HD + t * TILE + acc_row(4 * g, half), r);
      }
  }
}

template <int HD> constexpr size_t attn_lds() { return (size_t)ATTN_WAVES * ((HD / TILE) * 16 + 2) * WAVE * 4; }

template <typename E, int HD> static void launch_attention_t(const AttnArgs& a, hipStream_t st) {
  // With few workgroups of its own the launch gets layers of the grid behind the query tiles that fetch a.pf (a
  // workgroup fills a compute unit, so with many of its own the fetching ones would only queue up behind them).
  const int per_layer = a.n_splits * a.geom.n_heads, real = per_layer * a.n_qtiles;
  const bool fetch = a.pf.base != nullptr && real <= ATTN_FETCH_MAX_OWN;
  const int last = fetch ? l2_prefetch_first(real) + a.pf.n_regions : real;   // one past the last index in use
  attention_kernel<E, HD><<<dim3(a.n_splits, a.geom.n_heads, (last + per_layer - 1) / per_layer), ATTN_WAVES * WAVE,
                            attn_lds<HD>(), st>>>(
      (const E*)a.q, a.q_plane, (const E*)a.kv_layer, a.geom, a.meta, a.page_table, a.pt_stride, a.n_splits, a.part,
      a.tickets, (E*)a.out, a.T, a.n_qtiles, fetch ? a.pf : L2Prefetch{nullptr, 0, 0}, live_word());
}

template <int HD> constexpr size_t rows_lds() { return (size_t)2 * 4 * (HD / ET<bf16_t>::KS) * WAVE * 16; }
template <int HD> static void launch_attention_rows(const AttnArgs& a, int groups, hipStream_t st) {
  attention_rows_kernel<HD><<<dim3(a.geom.n_heads, groups), ROWS_WAVES * WAVE, rows_lds<HD>(), st>>>(
      (const bf16_t*)a.q, a.q_plane, (const bf16_t*)a.kv_layer, a.geom, a.meta, a.span, a.page_table, a.pt_stride, (bf16_t*)a.out,
      a.T, live_word());
}

bool configure_attention() {
  const void* fns[4] = {(const void*)attention_kernel<bf16_t, 128>, (const void*)attention_kernel<float, 128>,
                        (const void*)attention_kernel<bf16_t, 64>, (const void*)attention_kernel<float, 64>};
  bool ok = true;
  for (const void* fn : fns)
    ok = ok && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)attn_lds<128>()) == hipSuccess;
  ok = ok && hipFuncSetAttribute((const void*)attention_rows_kernel<128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rows_lds<128>()) == hipSuccess &&
       hipFuncSetAttribute((const void*)attention_rows_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)rows_lds<64>()) == hipSuccess;
  (void)hipGetLastError();
  return ok;
}

void launch_attention(bool bf16, const AttnArgs& a, hipStream_t st) {
  const int hd = a.geom.head_dim;
  const int groups = bf16 ? attn_rows_groups(a.span.off, a.span.n_seq, a.geom.n_heads, a.from_zero) : 0;
  if (groups > 0) {
    if (hd == 128) launch_attention_rows<128>(a, groups, st);
    else launch_attention_rows<64>(a, groups, st);
  } else if (bf16) {
    if (hd == 128) launch_attention_t<bf16_t, 128>(a, st);
    else launch_attention_t<bf16_t, 64>(a, st);
  } else {
    if (hd == 128) launch_attention_t<float, 128>(a, st);
    else launch_attention_t<float, 64>(a, st);
  }
}

TRACE_READER(trace_read_attention)

}  // namespace dinfer
