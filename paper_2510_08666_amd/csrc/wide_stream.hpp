// Shared-operand weight streaming for forwards with many token rows: a workgroup of WW waves covers WW tasks
// (64 output features each) and WT tiles of 32 token rows.  Each wave streams the weights of its task from memory
// into registers for the whole K range; the activation fragments of the WT token tiles go through LDS, staged
// chunk by chunk, so that every fragment is fetched once per workgroup.
#pragma once
#include <type_traits>

#include "gemm.hpp"

namespace dinfer {

// Kinds of kernels by trace id (the ids: common.hpp).
constexpr bool wide_dense(int kid) { return kid == 12 || kid == 13; }                // dense projections
constexpr bool wide_expert(int kid) { return kid == 10 || kid == 11; }               // expert GEMMs of four tiles: an item for itself,
constexpr bool wide_expert_shared(int kid) { return kid == 25 || kid == 26; }        // or beside its expert's others (expert_plan.hpp)
constexpr bool wide_smooth(int kid) { return kid == 24; }                            // smoothing contraction of four tiles

// How a kernel (by its trace id) with WT token tiles moves its operands.  KC: k-steps per chunk; PRE: chunks of weights in
// the registers of a wave; BD: chunks of activation fragments in its registers on their way to LDS; NB: chunks of fragments
// in LDS; AGAIN: other workgroups read the weights again soon.  Those are loaded as ordinary lines, which stay in the L2 (the
// dense projections' few MB, an expert's between its items); what is streamed once goes by non-temporal loads, which push
// nothing else out of the caches.
// The forms of four tiles and eight waves have one workgroup per compute unit and 128 accumulator registers per lane.  Where
// the matrix cores are the bound (LM head, prompts), short chunks with one barrier each let several of them be under way in the
// registers that two of four k-steps took, and a third LDS buffer carries a wave over the barrier (see the ring below).  Bit
// for bit the sums of the longer chunks; LM head at 512 / 160 tokens 366 -> 342 / 220 -> 195 us, gate/up + down at 4287
// tokens 534 + 312 -> 526 + 308, no spills (2 registers before); with chunks of four k-steps and three buffers 539 + 318.
// Three chunks of weights, not more: loads return in order, so the rows on their way to LDS wait for the weights asked for before
// them (4287 tokens, QKV / gate/up / down 229.7 / 537.8 / 300.6 us with four, 226.9 / 531.3 / 296.0 with three, 228.7 / 535.5 / 300.3 with two,
// 305.7 / 739 / 408 with six; LM head at 512 tokens 300.4 with four, 296.7 with three).  The
// expert GEMMs of up to two items per expert on average (wide_expert) keep four k-steps and two buffers: they are bound by
// their weights (12 sequences of 32, whole refresh: 569 us, 573 with short chunks).  Two workgroups of four waves per compute
// unit stage the fragments twice: LM head 404.
template <int KID, int WT> struct WideShape {
  static constexpr int KC = 4, PRE = 2, BD = wide_smooth(KID) || wide_expert(KID) ? 1 : 2, NB = 2;
  static constexpr bool AGAIN = wide_dense(KID);
};
template <int KID> struct WideShape4x8 {
  static constexpr int KC = 2, PRE = 3, BD = 1, NB = 3;
  static constexpr bool AGAIN = wide_dense(KID) || wide_expert_shared(KID);
};
// Two token tiles, likewise in short chunks over three buffers (chunks of four k-steps over two -> this): dense projections, QKV at 512
// tokens 43.1 -> 40.5 us, 384 41.3 -> 38.8; the forms of 33 to 64 tokens, with rows asked for three chunks ahead, gate/up + down at 64 tokens
// 82.4 + 47.9 -> 81.4 + 46.4, LM head 118.8 -> 117.8 (with four chunks of weights and rows two ahead 82.1 + 47.5, 118.2).  The expert GEMMs of
// few rows per expert, whose weights stream at the chip's rate, keep chunks of four: 64 experts of width 1024 at 160 tokens gain 1 us
// (96.3 + 59.7 -> 95.1 + 58.7), but with two rounds of workgroups (width 1536, 290 tokens) gate/up goes from 139 to 149.
template <int KID, int P, int B> struct WideShape2 {
  static constexpr int KC = 2, PRE = P, BD = B, NB = 3;
  static constexpr bool AGAIN = wide_dense(KID);
};
template <> struct WideShape<12, 2> : WideShape2<12, 4, 2> {};
template <> struct WideShape<13, 2> : WideShape2<13, 4, 2> {};
template <> struct WideShape<14, 2> : WideShape2<14, 3, 3> {};
template <> struct WideShape<17, 2> : WideShape2<17, 3, 3> {};
template <> struct WideShape<19, 2> : WideShape2<19, 3, 3> {};
template <> struct WideShape<9, 4> : WideShape4x8<9> {};
template <> struct WideShape<12, 4> : WideShape4x8<12> {};
template <> struct WideShape<13, 4> : WideShape4x8<13> {};
template <> struct WideShape<25, 4> : WideShape4x8<25> {};
template <> struct WideShape<26, 4> : WideShape4x8<26> {};
constexpr int WKC = 4;     // K is cut in units of this many k-steps

// Planes of the activations a kernel (by its trace id) feeds to the matrix cores.  The LM head with hundreds of
// token rows is bound by the matrix cores, and its rounding error is not carried into later layers: it takes the
// high bf16 plane only, that is activations rounded to bf16 as in the paper's arithmetic (bf16 inputs, float32
// accumulation); the low plane would double its matrix work.  The expert GEMMs stay bound by their weight streams
// and keep both planes (one plane: 7 % faster, but the error carried through 16 layers reaches the test bars).
template <typename E, int KID> struct WidePlanes { static constexpr int N = Planes<E>::N; };
template <> struct WidePlanes<bf16_t, 9> { static constexpr int N = 1; };

template <int N, class F, int I = 0> __device__ inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}

// One k-step of a token tile in LDS: 32 rows of PIECES 16-byte pieces, as they lie in memory (plane by plane, half by half).
// A load covers 64 / PIECES whole rows: neighbouring lanes take the pieces of one row, so that the address unit finds them in
// one cache line.  In LDS a row's pieces are permuted by the row number (in groups of 16 / PIECES rows), so that neither the
// writes nor the fragment reads (one piece of 32 rows each) meet in a bank: SQ_LDS_BANK_CONFLICT is 0.
template <typename E, int KID> struct WidePieces {
  static constexpr int N = 2 * WidePlanes<E, KID>::N, TILE_VECS = TILE * N, ROWS = WAVE / N;
  __device__ static int slot(int row, int piece) { return row * N + (piece ^ ((row / (16 / N)) & (N - 1))); }
};
template <typename E, int KID, int WT> constexpr size_t wide_lds() {
  return (size_t)WideShape<KID, WT>::NB * WideShape<KID, WT>::KC * WT * WidePieces<E, KID>::TILE_VECS * 16;
}

// Accumulate ksteps k-steps (a multiple of KC).  w: this wave's task (k-step 0).  act: the k-major activations (k-step
// 0), bkstride: their k-step stride; row_of(r): the activation row that row r of token tile `wave % WT` stands for.
// sb: LDS [buffers][KC][WT][32 rows][pieces].  NT: token tiles that hold rows.  wave: 0 .. WW-1 (uniform), the
// wave's rank among the WW waves that share sb (every wave of the workgroup must make the call: it holds the
// workgroup's barriers).
template <typename E, int WT, int NT, int WW, int KID, class RowOf>
__device__ inline void wide_stream_nt(const E* __restrict__ w, int ksteps, const E* __restrict__ act, RowOf&& row_of, int64_t bkstride,
                                      typename ET<E>::vec* sb, f32x16 (&acc0)[WT], f32x16 (&acc1)[WT], int wave) {
  typedef typename ET<E>::vec vec;
  typedef WidePieces<E, KID> Pc;
  typedef WideShape<KID, WT> Sh;
  constexpr int KC = Sh::KC, PRE = Sh::PRE, BD = Sh::BD, NB = Sh::NB;
  constexpr int NP = WidePlanes<E, KID>::N, ROW_BYTES = NP * ET<E>::KS * (int)sizeof(E);   // planes; a row's k-step
  constexpr int STEP = 2 * WAVE * 16;              // bytes of a task's k-step
  static_assert(PRE % BD == 0 && (NB == 2 || NB == 3), "register sets are taken from the unrolled index");
  static_assert(WW % WT == 0 && (KC * WT) % WW == 0, "every wave stages whole k-steps of one token tile");
  const int lane = threadIdx.x & 63;
  const int n_chunks = ksteps / KC, last = n_chunks - 1;
  TRACE_MARK(KID, 0);
  constexpr int SKS = KC * WT / WW;                // k-steps of a chunk this wave stages (of token tile wave % WT)
  const int st = wave % WT, sk0 = (wave / WT) * SKS;
  constexpr int BUF = KC * WT * Pc::TILE_VECS;
  // bf16 operands are addressed by a scalar base per k-step, float32 ones by a pointer per lane: there the scalar arithmetic in
  // front of every chunk's loads cost the matrix instructions 6 to 18 % (QKV of 1500 tokens, hidden 1024: 276 us with scalar bases,
  // 249 with a pointer per lane for the weights, 239 for the rows as well; LM head of 32 tokens, hidden 3584, 476, 463 and 452).
  // bf16 gains nothing, and two planes of row pointers cost registers (384 tokens 260 -> 264 us a layer).
  constexpr bool LANES = sizeof(E) == 4;
  const uint32_t wlane = lane * 16;
  const char* wl = (const char*)w + wlane;
  auto wload = [&](int c, int ks, int tile) {
    const int64_t at = (int64_t)(min(c, last) * KC + ks) * STEP + tile * (WAVE * 16);
    const E* p = (const E*)(LANES ? wl + at : (const char*)w + at + wlane);
    return Sh::AGAIN ? load16<E>(p) : load16_stream<E>(p);
  };
  vec wa0[PRE][KC], wa1[PRE][KC];
  vec bset[BD][SKS][NP];                           // fragments of later chunks, on their way to LDS
  // what this lane stages: piece lane % N of NP rows
  uint32_t src[NP];                                // byte offset in a k-step
  int dst[NP];
  // (asked for before the weights: for the experts they hang on the permutation, and loads return in order)
#pragma unroll
  for (int j = 0; j < NP; ++j) src[j] = (uint32_t)row_of(j * Pc::ROWS + lane / Pc::N);
#pragma unroll
  for (int i = 0; i < PRE; ++i)
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) {
      wa0[i][ks] = wload(i, ks, 0);
      wa1[i][ks] = wload(i, ks, 1);
    }
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int r = j * Pc::ROWS + lane / Pc::N;
    src[j] = src[j] * (uint32_t)ROW_BYTES + (lane % Pc::N) * 16;
    dst[j] = (sk0 * WT + st) * Pc::TILE_VECS + Pc::slot(r, lane % Pc::N);
  }
  const int64_t step = bkstride * (int64_t)sizeof(E);
  const char* row[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) row[j] = (const char*)act + sk0 * step + src[j];
  auto fetch = [&](int c, vec (&b)[SKS][NP]) {
    const int64_t at = (int64_t)(min(c, last) * KC) * step;
    const char* base = (const char*)(act + (int64_t)(min(c, last) * KC + sk0) * bkstride);
#pragma unroll
    for (int ks = 0; ks < SKS; ++ks)
#pragma unroll
      for (int j = 0; j < NP; ++j) b[ks][j] = load16<E>((const E*)(LANES ? row[j] + at + ks * step : base + ks * step + src[j]));
  };
  auto put = [&](int buf, const vec (&b)[SKS][NP]) {
#pragma unroll
    for (int ks = 0; ks < SKS; ++ks)
#pragma unroll
      for (int j = 0; j < NP; ++j) sb[buf + ks * WT * Pc::TILE_VECS + dst[j]] = b[ks][j];
  };
  {
    vec b0[NB - 1][SKS][NP];
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) fetch(i, b0[i]);
#pragma unroll
    for (int i = 0; i < BD; ++i) fetch(NB - 1 + i, bset[(NB - 1 + i) % BD]);
#pragma unroll
    for (int i = 0; i < NB - 1; ++i) put(i * BUF, b0[i]);
  }
  int rd[NP];                                      // this lane's vector of plane q in a k-step of a tile
#pragma unroll
  for (int q = 0; q < NP; ++q) rd[q] = Pc::slot(lane & 31, 2 * q + (lane >> 5));
  // Fragments in the order (k-step, token tile, plane).  The LDS read of fragment f + FD is issued before the matrix
  // instructions of fragment f, and a scheduling barrier keeps the compiler from sinking it back next to its use (left
  // alone it keeps only two reads in flight and the matrix pipe waits for LDS after every four instructions; measured at
  // 512 tokens: LM head 362 -> 322 us, QKV 41.7 -> 38.7 us, expert gate/up 118 -> 113 us).  With three buffers the ring runs
  // on over the barrier.
  constexpr int F = KC * NT * NP;
  constexpr int FD = F % 4 == 0 ? 4 : F % 3 == 0 ? 3 : 2;
  static_assert(F % FD == 0, "the ring goes on over chunks");
  vec ring[FD];
  auto frag = [&](int buf, int f) { return sb[buf + ((f / (NT * NP)) * WT + (f / NP) % NT) * Pc::TILE_VECS + rd[f % NP]]; };
  int cur = 0;                                     // buffer of chunk c
  if constexpr (NB == 3) {
    __syncthreads();
    static_for<FD>([&](auto J) { ring[decltype(J)::value] = frag(0, decltype(J)::value); });
  }
  // One chunk; i = c % PRE picks the registers at compile time.  Barrier; the fragments of chunk c + NB - 1 go from registers
  // to LDS and a later chunk's take their place; chunk c is multiplied; the weights of chunk c + PRE are requested.  Loads
  // past the end are clamped to the last chunk (never used), so the loop body has no branch around a load.
  auto chunk = [&](auto I, int c) {
    constexpr int i = decltype(I)::value;
    __syncthreads();
    if (c == 0) TRACE_MARK(KID, 1);
    if (c == 1) TRACE_MARK(KID, 2);
    if (c == 16) TRACE_MARK(KID, 4);
    if (c == 32) TRACE_MARK(KID, 5);
    const int nxt = cur + BUF < NB * BUF ? cur + BUF : 0;
    auto& b = bset[(i + NB - 1) % BD];
    if constexpr (NB == 3) put(nxt + BUF < NB * BUF ? nxt + BUF : 0, b);
    else put(nxt, b);
    fetch(c + NB - 1 + BD, b);
    if constexpr (NB == 2) static_for<FD>([&](auto J) { ring[decltype(J)::value] = frag(cur, decltype(J)::value); });
    static_for<F>([&](auto Fi) {
      constexpr int f = decltype(Fi)::value, ks = f / (NT * NP), t = (f / NP) % NT;
      const vec b = ring[f % FD];
      if constexpr (f + FD < F) ring[f % FD] = frag(cur, f + FD);
      else if constexpr (NB == 3) ring[f % FD] = frag(nxt, f + FD - F);
      __builtin_amdgcn_sched_barrier(0);
      mfma32(acc0[t], wa0[i][ks], b);
      mfma32(acc1[t], wa1[i][ks], b);
    });
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) {
      wa0[i][ks] = wload(c + PRE, ks, 0);
      wa1[i][ks] = wload(c + PRE, ks, 1);
    }
    cur = nxt;
  };
  // Whole rounds of PRE chunks run without a test between the chunks: a branch there gives the compiler a path from
  // one chunk straight back to the loop top, for which it drains every load in flight at each iteration.
  // The first round stands in front of the loop: the prologue leaves the loads in another order than a round does
  // (all weights first, then the fragments), and the wait counts the compiler puts at the loop top are the smaller
  // of what its two ways in allow -- entered straight from the prologue, every chunk waited until all but four of
  // the loads in flight had returned, the weights requested one chunk earlier included, and a wave had one chunk
  // of weights under way instead of PRE.
  int c0 = 0;
  if (n_chunks >= PRE) {
    static_for<PRE>([&](auto I) { chunk(I, decltype(I)::value); });
    for (c0 = PRE; c0 + PRE <= n_chunks; c0 += PRE) static_for<PRE>([&](auto I) { chunk(I, c0 + decltype(I)::value); });
  }
  static_for<PRE - 1>([&](auto I) {
    if (c0 + decltype(I)::value < n_chunks) chunk(I, c0 + decltype(I)::value);   // uniform over the workgroup
  });
  TRACE_MARK(KID, 6);
}

// nt: token tiles that hold rows (the others are skipped); the tile count is a compile-time constant of the loop.
template <typename E, int WT, int WW, int KID, class RowOf>
__device__ inline void wide_stream(const E* __restrict__ w, int ksteps, const E* __restrict__ act, RowOf&& row_of, int64_t bkstride,
                                   typename ET<E>::vec* sb, int nt, f32x16 (&acc0)[WT], f32x16 (&acc1)[WT], int wave) {
  if constexpr (WT >= 4) {
    if (nt >= 4) return wide_stream_nt<E, WT, 4, WW, KID>(w, ksteps, act, row_of, bkstride, sb, acc0, acc1, wave);
    if (nt == 3) return wide_stream_nt<E, WT, 3, WW, KID>(w, ksteps, act, row_of, bkstride, sb, acc0, acc1, wave);
  }
  if constexpr (WT >= 2) {
    if (nt >= 2) return wide_stream_nt<E, WT, 2, WW, KID>(w, ksteps, act, row_of, bkstride, sb, acc0, acc1, wave);
  }
  wide_stream_nt<E, WT, 1, WW, KID>(w, ksteps, act, row_of, bkstride, sb, acc0, acc1, wave);
}

}  // namespace dinfer
