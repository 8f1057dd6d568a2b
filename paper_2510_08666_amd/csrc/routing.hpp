// Reductions over a whole wavefront, and what the expert kernels of up to 64 tokens read off the routing themselves.
#pragma once
#include "common.hpp"

namespace dinfer {

// Cross-lane moves inside rows of 16 lanes on the data-parallel-primitive path (no LDS round trip).  The four
// controls below form a butterfly: after them (the first three) every lane of a 16-lane (8-lane) group holds the group's
// result, provided the combining step is symmetric.
template <int CTRL> __device__ inline int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
template <int CTRL> __device__ inline float dpp_f(float v) { return __int_as_float(dpp_i<CTRL>(__float_as_int(v))); }
constexpr int DPP_SWAP1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int DPP_SWAP2 = 0x4E;         // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141;  // lane i <- lane 7-i of its group of 8
constexpr int DPP_MIRROR = 0x140;       // lane i <- lane 15-i of its row

// f over all 64 lanes; every lane ends with the same bits where f commutes.  Behind the butterfly of a row, two exchanges of
// rows and of half-waves: of a pair of equal registers each swap leaves one side's values in the first and the other's in
// the second, in every lane.
template <class F> __device__ inline int wave_all(int v, F f) {
  v = f(v, dpp_i<DPP_SWAP1>(v));
  v = f(v, dpp_i<DPP_SWAP2>(v));
  v = f(v, dpp_i<DPP_HALF_MIRROR>(v));
  v = f(v, dpp_i<DPP_MIRROR>(v));
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = f((int)r[0], (int)r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return f((int)h[0], (int)h[1]);
}
__device__ inline float wave_all_max(float v) {
  return __int_as_float(wave_all(__float_as_int(v), [](int a, int b) { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); }));
}
__device__ inline float wave_all_sum(float v) {
  return __int_as_float(wave_all(__float_as_int(v), [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }));
}
// The sum as lanes with four consecutive values each would form it: those in order, then a butterfly over the sixteen sums.
__device__ inline float wave_all_sum_by_fours(float v) {
  float s = dpp_f<0x00>(v) + dpp_f<0x55>(v);      // quad_perm: the same lane of four to all of them
  s += dpp_f<0xAA>(v);
  s += dpp_f<0xFF>(v);
  s += dpp_f<DPP_HALF_MIRROR>(s);
  s += dpp_f<DPP_MIRROR>(s);
  const int i = __float_as_int(s);
  const auto r = __builtin_amdgcn_permlane16_swap(i, i, false, false);
  s = __int_as_float(r[0]) + __int_as_float(r[1]);
  const int k = __float_as_int(s);
  const auto h = __builtin_amdgcn_permlane32_swap(k, k, false, false);
  return __int_as_float(h[0]) + __int_as_float(h[1]);
}
// ... as lanes with eight consecutive values each would form it.
__device__ inline float wave_all_sum_by_eights(float v) {
  float s = dpp_f<0x00>(v) + dpp_f<0x55>(v);      // the first four of the eight lanes
  s += dpp_f<0xAA>(v);
  s += dpp_f<0xFF>(v);
  float t = dpp_f<DPP_HALF_MIRROR>(s);            // ... in the lanes of the other four, which go on from them
  t += dpp_f<0x00>(v);
  t += dpp_f<0x55>(v);
  t += dpp_f<0xAA>(v);
  t += dpp_f<0xFF>(v);
  const float back = dpp_f<DPP_HALF_MIRROR>(t);
  s = threadIdx.x & 4 ? t : back;
  s += dpp_f<DPP_MIRROR>(s);
  const int i = __float_as_int(s);
  const auto r = __builtin_amdgcn_permlane16_swap(i, i, false, false);
  s = __int_as_float(r[0]) + __int_as_float(r[1]);
  const int k = __float_as_int(s);
  const auto h = __builtin_amdgcn_permlane32_swap(k, k, false, false);
  return __int_as_float(h[0]) + __int_as_float(h[1]);
}
// OR over the wave, as a scalar
__device__ inline uint64_t wave_all_or(uint64_t v) {
  auto all = [](int x) { return (uint32_t)__builtin_amdgcn_readfirstlane(wave_all(x, [](int a, int b) { return a | b; })); };
  return (uint64_t)all((int)(v >> 32)) << 32 | all((int)v);
}
// Set bits of a wave-uniform mask below this lane
__device__ inline int bits_below_lane(uint64_t m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)); }
// Position of the n-th set bit (n from 0, less than the number of set bits) of a wave-uniform mask
__device__ inline int nth_bit(uint64_t m, int n) {
  const bool mine = ((m >> (threadIdx.x & 63)) & 1) && bits_below_lane(m) == n;
  return __builtin_ctzll(__ballot(mine) | 1ull << 63);
}

// Up to 64 tokens the kernels of the routed experts sort the (token, slot) pairs themselves: a wave holds all pairs, N in a
// lane, and reads off what it needs by ballots: which experts have rows, and the rows of one of them, in pair order.  That is a
// load and some two hundred instructions beside the weights' first loads, where a sort in front of the launch was one
// more hand-off between workgroups (in the router: 2.2 us) and another 1.2 us for the permutation.
template <int N> struct PairIds {
  int id[N];       // expert of pair j * 64 + lane, MAX_EXPERTS past the end
  __device__ void load(const int32_t* __restrict__ expert_of_pair, int n_pairs) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < N; ++j) id[j] = expert_of_pair[min(j * WAVE + lane, n_pairs - 1)];
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (j * WAVE + lane >= n_pairs) id[j] = MAX_EXPERTS;
  }
  __device__ uint64_t experts() const {
    uint64_t m = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) m |= id[j] < MAX_EXPERTS ? 1ull << id[j] : 0ull;
    return wave_all_or(m);
  }
  // {e, first sorted row, rows, 0} of expert e; s_pair (64 entries of LDS): its pairs, in order, once the caller has passed a
  // barrier (a token is routed to an expert at most once, so there are no more than 64)
  __device__ int4 rows_of(int e, int32_t* s_pair) const {
    const int lane = threadIdx.x & 63;
    int first = 0, rows = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      first += __popcll(__ballot(id[j] < e));
      const uint64_t mine = __ballot(id[j] == e);
      if (id[j] == e) s_pair[rows + bits_below_lane(mine)] = j * WAVE + lane;
      rows += __popcll(mine);
    }
    return make_int4(e, first, rows, 0);
  }
};

// Up to 32 tokens, where a wave wants the rows of all tokens for a few experts: lane = token (both half-waves alike).
struct TokenExperts {
  int e[MAX_TOPK], top_k;       // (the last one again past top_k)
  bool is_tok;
  __device__ void load(const int32_t* __restrict__ topk_idx, int T, int k) {
    const int col = threadIdx.x & 31;
    top_k = k;
    is_tok = col < T;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) e[j] = topk_idx[min(col, T - 1) * k + min(j, k - 1)];
  }
  __device__ uint64_t experts() const {
    uint64_t m = 0;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) m |= 1ull << e[j];
    return wave_all_or(m);
  }
  // Place of the lane's token for expert x among the pairs sorted by expert, then token; -1: not routed to it
  __device__ int row_of(int x) const {
    const int half = (threadIdx.x >> 5) & 1, col = threadIdx.x & 31;
    int before = 0;
    bool here = false;
#pragma unroll
    for (int j = 0; j < MAX_TOPK; ++j) {
      const bool pair = is_tok && half == 0 && j < top_k;
      before += __popcll(__ballot(pair && e[j] < x));
      here |= e[j] == x;
    }
    const uint32_t toks = (uint32_t)__ballot(is_tok && here);   // bit per token, from the lower half-wave
    return is_tok && here ? before + __popc(toks & ((1u << col) - 1)) : -1;
  }
};

}  // namespace dinfer
