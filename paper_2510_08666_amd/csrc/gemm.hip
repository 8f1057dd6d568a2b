// The dense contractions of the step as weight-streaming MFMA kernels (core in gemm.hpp):
//   QKV projection + rotary embedding + KV-page write, output projection + residual,
//   router + top-k, the fused down projection of the routed experts, iteration smoothing's contraction.
// (The other expert GEMMs and the LM head: wide.hip.)
// RMSNorm is never materialised.  Whoever produces a residual row also stores it multiplied by the gain of the
// norm that follows, as MFMA-ready planes ("normalised-input planes", without the 1/rms factor); the consumers
// feed those planes to the matrix cores and scale their accumulators by the row's 1/rms in the epilogue.
#include "gemm.hpp"
#include "kernels.hpp"
#include "routing.hpp"
#include "wide_stream.hpp"

namespace dinfer {

// ------------------------------------------------------------------------------------------------
// Split-K kernel for the attention-side projections.  A task (64 output features) of one token group is shared
// by `slices` workgroups of KW waves; every wave streams its own K range.  The partial tiles of a workgroup are
// summed through LDS in wave order; with more than one slice the workgroup sums go to global memory and the
// workgroup that arrives last adds them in slice order (so the result does not depend on scheduling) and runs
// the epilogue.  At small token counts the host picks the slices so that a wave's whole K range is in flight at
// once: these kernels are bound by memory latency, not bandwidth, and every further dependent round trip
// costs microseconds.
// ------------------------------------------------------------------------------------------------
// Epilogues receive, for one token (lane) and one accumulator tile pair, PER consecutive accumulator registers
// v0 .. v0+PER-1 of tile 0 (a0) and tile 1 (a1): rows acc_row(v0, half) .. +PER-1 of each tile, which are PER
// consecutive features (v0 is a multiple of PER, PER divides 4).  apply() returns the lane's contribution to the
// row statistic of the epilogue (ROWSUM), which the kernel sums over the task and hands to row_sum().
template <typename E> struct QkvEpi {
  static constexpr bool ROWSUM = false;
  E* q;
  int64_t q_plane;
  E* kv_layer;
  KvGeom geom;
  const int32_t* tok_seq;
  const int32_t* tok_pos;
  const int32_t* page_table;
  int pt_stride;
  const float* cos_tab;
  const float* sin_tab;
  RowNorm norm;        // statistics of the tokens' residual rows
  int T, H;
  int D;               // n_heads * head_dim

  // What the epilogue needs from memory besides the accumulators.  prefetch() runs before the weight stream
  // starts and issues only loads whose addresses are known then; prefetch2() runs behind the stream and issues
  // the loads that depend on the first ones, so that they are under way while the partial sums are folded.
  template <int PER> struct Pre {
    int pos, seq, page, tok;
    float r;
    float c[PER], s[PER];
  };
  template <int PER> __device__ Pre<PER> prefetch(int, int tok, bool valid, int, int) const {
    Pre<PER> p;
    const int t = valid ? tok : 0;
    p.pos = tok_pos[t];
    p.seq = tok_seq[t];
    p.tok = t;
    return p;
  }
  template <int PER> __device__ void prefetch2(Pre<PER>& p, int task, int half, int v0) const {
    const int hd = geom.head_dim;
    p.r = row_rinv(norm.ssq, norm.n_ssq, T, p.tok, H, norm.eps);   // up to 32 loads: kept behind the weight stream
    p.page = page_table[(int64_t)p.seq * pt_stride + p.pos / PAGE];
    const int j0 = (task % (hd / 64)) * TILE + acc_row(v0, half);
    const bool rot = task < 2 * geom.n_heads * (hd / 64);
    if constexpr (PER == 4) {   // j0 is a multiple of 4: one 16-byte load per table
      const f32x4 c4 = *reinterpret_cast<const f32x4*>(cos_tab + (int64_t)p.pos * (hd / 2) + (rot ? j0 : 0));
      const f32x4 s4 = *reinterpret_cast<const f32x4*>(sin_tab + (int64_t)p.pos * (hd / 2) + (rot ? j0 : 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p.c[i] = rot ? c4[i] : 1.f;
        p.s[i] = rot ? s4[i] : 0.f;
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        p.c[i] = rot ? cos_tab[(int64_t)p.pos * (hd / 2) + j0 + i] : 1.f;
        p.s[i] = rot ? sin_tab[(int64_t)p.pos * (hd / 2) + j0 + i] : 0.f;
      }
    }
  }

  template <int PER>
  __device__ float apply(const Pre<PER>& pre, int task, int tok, bool valid, int half, int v0, const float (&a0)[PER],
                         const float (&a1)[PER], bool) const {
    if (!valid) return 0.f;
    const int hd = geom.head_dim;
    const int per_head = hd / 64;
    const int qk_tasks = geom.n_heads * per_head;
    const int page = safe_page(geom, pre.page);
    const int slot = pre.pos % PAGE;
    const float r = pre.r;
    const int row0 = acc_row(v0, half);
    if (task < 2 * qk_tasks) {
      // rotary pair: a0 holds feature j of the head, a1 feature j + hd/2
      const bool is_k = task >= qk_tasks;
      const int rr = is_k ? task - qk_tasks : task;
      const int head = rr / per_head, jt = rr % per_head;
      const int j0 = jt * TILE + row0;
      float lo[PER], hi[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const float a = a0[i] * r, b = a1[i] * r;
        lo[i] = a * pre.c[i] - b * pre.s[i];
        hi[i] = b * pre.c[i] + a * pre.s[i];
      }
      if (is_k) {
        // (PER consecutive features starting at a multiple of PER stay inside one 32-byte block of the K layout)
        E* dst = kv_layer + kv_k_index(geom, page, head, slot, j0);
        E* dst_hi = kv_layer + kv_k_index(geom, page, head, slot, j0 + hd / 2);
        if constexpr (PER == 4) {
          store_elems4<E>(dst, f32x4{lo[0], lo[1], lo[2], lo[3]});
          store_elems4<E>(dst_hi, f32x4{hi[0], hi[1], hi[2], hi[3]});
        } else {
#pragma unroll
          for (int i = 0; i < PER; ++i) {
            dst[i] = from_f32<E>(lo[i]);
            dst_hi[i] = from_f32<E>(hi[i]);
          }
        }
      } else {
        const int64_t dst = (int64_t)tok * D + head * hd + j0;
        if constexpr (PER == 4) {
          store_act4<E>(q, dst, q_plane, f32x4{lo[0], lo[1], lo[2], lo[3]});
          store_act4<E>(q, dst + hd / 2, q_plane, f32x4{hi[0], hi[1], hi[2], hi[3]});
        } else {
#pragma unroll
          for (int i = 0; i < PER; ++i) {
            store_act<E>(q, dst + i, q_plane, lo[i]);
            store_act<E>(q, dst + hd / 2 + i, q_plane, hi[i]);
          }
        }
      }
    } else {
      const int t = task - 2 * qk_tasks;   // adjacent tiles 2t, 2t+1 of V
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int f0 = (2 * t) * TILE + row0 + i;
        const int f1 = f0 + TILE;
        kv_layer[kv_v_index(geom, page, f0 / hd, slot, f0 % hd)] = from_f32<E>(a0[i] * r);
        kv_layer[kv_v_index(geom, page, f1 / hd, slot, f1 % hd)] = from_f32<E>(a1[i] * r);
      }
    }
    return 0.f;
  }
  __device__ void row_sum(int, int, float) const {}
};

// Eight features' contribution to the router's logits in float32, straight from the registers of an epilogue: a lane holds four of
// them for its token, rows 8 * step + 4 * half .. +3 of weight tile `tile` of the 64-feature task, which is the B operand of
// two matrix instructions as it stands.  Result as for mfma32: experts along the rows.
struct RouterStep {
  // packed router weights: the lane's expert (of 32 from 32 * et on), the four features above
  __device__ static f32x4 load(const float* w, int task, int tile, int step, int et, int lane) {
    return *reinterpret_cast<const f32x4*>(w + (((int64_t)task * 8 + tile * 4 + step) * 2 + et) * (WAVE * 4) + lane * 4);
  }
  __device__ static void add(f32x16& acc, const f32x4& a, const f32x4& v) { mfma32(acc, a, v); }
};

// x += result; the new row also goes out as normalised-input planes for the expert half (times its norm's gain),
// and the task's share of the row's sum of squares to ssq[task][token].
template <typename E> struct ResidualEpi {
  static constexpr bool ROWSUM = true;
  float* x;
  int H;
  const float* gain;   // [H] gain of the norm that follows
  E* xn;               // [T][H] k-major planes
  float* ssq;          // [H/64][T]
  int T;
  const E* w_router;   // null: no shares of the router's logits
  float* shares;       // [H/64][T][MAX_EXPERTS]

  template <int PER> struct Pre {
    float x0[PER], x1[PER], g0[PER], g1[PER];
  };
  template <int PER> __device__ Pre<PER> prefetch(int task, int tok, bool valid, int half, int v0) const {
    Pre<PER> p;
    const int col = (2 * task) * TILE + acc_row(v0, half);
    const float* p0 = x + (int64_t)(valid ? tok : 0) * H + col;
    if constexpr (PER == 4) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(p0), b = *reinterpret_cast<const f32x4*>(p0 + TILE);
      const f32x4 c = *reinterpret_cast<const f32x4*>(gain + col), d = *reinterpret_cast<const f32x4*>(gain + col + TILE);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p.x0[i] = a[i];
        p.x1[i] = b[i];
        p.g0[i] = c[i];
        p.g1[i] = d[i];
      }
      return p;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      p.x0[i] = p0[i];
      p.x1[i] = p0[TILE + i];
      p.g0[i] = gain[col + i];
      p.g1[i] = gain[col + TILE + i];
    }
    return p;
  }
  template <int PER> __device__ void prefetch2(Pre<PER>&, int, int, int) const {}

  // Two squares, the first of which is rounded by itself.  Which of a tile pair's that is was the compiler's choice for each kernel, and
  // another one is another 1/rms for every product that follows: so it is written down (first0; a constant for the callers).
  __device__ static float two_squares(float n0, float n1, bool first0) {
    return first0 ? __builtin_fmaf(n1, n1, n0 * n0) : __builtin_fmaf(n0, n0, n1 * n1);
  }
  template <int PER>
  __device__ float apply(const Pre<PER>& pre, int task, int tok, bool valid, int half, int v0, const float (&a0)[PER],
                         const float (&a1)[PER], bool first0) const {
    if (!valid) return 0.f;
    const int col = (2 * task) * TILE + acc_row(v0, half);
    float* p0 = x + (int64_t)tok * H + col;
    float ss = 0.f;
    if constexpr (PER == 4) {
      f32x4 n0, n1, m0, m1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        n0[i] = pre.x0[i] + a0[i];
        n1[i] = pre.x1[i] + a1[i];
        m0[i] = n0[i] * pre.g0[i];
        m1[i] = n1[i] * pre.g1[i];
        ss += two_squares(n0[i], n1[i], first0);
      }
      *reinterpret_cast<f32x4*>(p0) = n0;
      *reinterpret_cast<f32x4*>(p0 + TILE) = n1;
      store_actk4<E>(xn, T, tok, col, m0);
      store_actk4<E>(xn, T, tok, col + TILE, m1);
      return ss;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const float n0 = pre.x0[i] + a0[i], n1 = pre.x1[i] + a1[i];
      p0[i] = n0;
      p0[TILE + i] = n1;
      store_actk<E>(xn, T, tok, col + i, n0 * pre.g0[i]);
      store_actk<E>(xn, T, tok, col + TILE + i, n1 * pre.g1[i]);
      ss += two_squares(n0, n1, first0);
    }
    return ss;
  }
  __device__ void row_sum(int task, int tok, float s) const { ssq[(int64_t)task * T + tok] = s; }
  // the values that apply() stores as planes, four features of each tile
  __device__ static void normed(const Pre<4>& pre, const float (&a0)[4], const float (&a1)[4], f32x4 (&m)[2]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[0][i] = (pre.x0[i] + a0[i]) * pre.g0[i];
      m[1][i] = (pre.x1[i] + a1[i]) * pre.g1[i];
    }
  }
  __device__ void store_share(int task, int tok, int expert, const f32x4& v) const {
    *reinterpret_cast<f32x4*>(shares + ((int64_t)task * T + tok) * MAX_EXPERTS + expert) = v;
  }
};

// The workgroup's sums leave for / come back from the cross-workgroup buffer.  A thread holds PER consecutive
// accumulator registers (v0 .. v0+PER-1) of each tile; they travel as one PER-float piece:
//   part[unit][slice][token tile][weight tile][v0 / PER][lane][PER]
// Writer and reader are the same (wave, lane) of their workgroups, so each reads what its counterpart wrote.
template <int TT, int PER> __device__ inline uint32_t slice_piece(int64_t unit_slice, int t, int tile, int v0, int lane) {
  return (uint32_t)(((((unit_slice * TT + t) * 2 + tile) * (16 / PER) + v0 / PER) * WAVE + lane) * PER * sizeof(float));
}
template <int TT, int PER>
__device__ inline void put_slice(float* part, int64_t unit_slice, int lane, int v0, const float (&a0)[TT][PER],
                                 const float (&a1)[TT][PER]) {
  const buf_rsrc r = coherent_buffer(part);
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    coherent_store_n<PER>(r, slice_piece<TT, PER>(unit_slice, t, 0, v0, lane), a0[t]);
    coherent_store_n<PER>(r, slice_piece<TT, PER>(unit_slice, t, 1, v0, lane), a1[t]);
  }
}
// The loads of CH slices are issued together before any of them is added (a loop that loads and adds slice by
// slice pays one memory round trip per slice); the sum still runs in slice order.
template <int TT, int PER, int CH = 4>
__device__ inline void sum_slices(const float* part, int64_t unit, int n_slices, int lane, int v0, float (&a0)[TT][PER],
                                  float (&a1)[TT][PER]) {
  const buf_rsrc r = coherent_buffer(part);
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      a0[t][i] = 0.f;
      a1[t][i] = 0.f;
    }
  for (int s0 = 0; s0 < n_slices; s0 += CH) {
    float b0[CH][TT][PER], b1[CH][TT][PER];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int64_t us = unit * n_slices + min(s0 + c, n_slices - 1);
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        coherent_load_n<PER>(r, slice_piece<TT, PER>(us, t, 0, v0, lane), b0[c][t]);
        coherent_load_n<PER>(r, slice_piece<TT, PER>(us, t, 1, v0, lane), b1[c][t]);
      }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const bool on = s0 + c < n_slices;
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          a0[t][i] += on ? b0[c][t][i] : 0.f;
          a1[t][i] += on ? b1[c][t][i] : 0.f;
        }
    }
  }
}

template <typename E, int TT, int KW, class Epi>
__global__ __launch_bounds__(KW * WAVE) void gemm_ksplit_kernel(const E* __restrict__ W, int ksteps,
                                                                 const E* __restrict__ B, int T, int K,
                                                                 float* __restrict__ part, int32_t* __restrict__ tickets,
                                                                 Epi epi, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  extern __shared__ float red[];   // [KW][2*TT*16][64]
  __shared__ int32_t s_flag;
  __shared__ float s_ss[Epi::ROWSUM ? KW * TT * TILE : 1];
  constexpr int ROWS = 2 * TT * 16, PER = 16 / KW;
  [[maybe_unused]] constexpr int KID = Epi::ROWSUM ? 2 : 1;
  const int slice = blockIdx.x, n_slices = gridDim.x, task = blockIdx.y, group = blockIdx.z;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5;
  const int tok0 = group * TT * TILE;
  TRACE_MARK(KID, 0);
  const int v0 = wave * PER;
  typename Epi::template Pre<PER> pre[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const int tok = tok0 + t * TILE + (lane & 31);
    pre[t] = epi.template prefetch<PER>(task, tok, tok < T, half, v0);
  }
  f32x16 acc0[TT], acc1[TT];
  zero_acc<TT>(acc0);
  zero_acc<TT>(acc1);
  const int per = (ksteps + n_slices * KW - 1) / (n_slices * KW);
  const int ks0 = min(ksteps, (slice * KW + wave) * per), ks1 = min(ksteps, ks0 + per);
  PlaneLoader<E, TT> ld;
#pragma unroll
  for (int t = 0; t < TT; ++t) ld.set(t, B, T, min(tok0 + t * TILE + (lane & 31), T - 1), half);
  stream_task<E, TT, (TT == 1 ? 8 : 4)>(W + (int64_t)task * task_stride_elems<E>(ksteps), ks0, ks1, ld, acc0, acc1);
  TRACE_MARK(KID, 1);
#pragma unroll
  for (int t = 0; t < TT; ++t) epi.template prefetch2<PER>(pre[t], task, half, v0);
  // Shares of the router's logits: of up to 64 tokens, in float32 a wave's eight features of either tile straight from its registers; in
  // bfloat16, two token tiles (one: oproj_pair_kernel), a chain of the task's four k-steps on the planes as they are stored.
  constexpr bool STEPS = Epi::ROWSUM && sizeof(E) == 4 && TT <= 2, CHAIN = Epi::ROWSUM && sizeof(E) == 2 && TT == 2;
  [[maybe_unused]] f32x4 rw[2][2];   // [tile][experts from 0, from 32]
  if constexpr (STEPS) {
    if (epi.w_router) {
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int et = 0; et < 2; ++et) rw[f][et] = RouterStep::load(epi.w_router, task, f, wave, et, lane);
    }
  }
  spill_partials<TT, ROWS>(red, wave, lane, acc0, acc1);
  __syncthreads();
  TRACE_MARK(KID, 2);
  float a0[TT][PER], a1[TT][PER];
  fold_partials<TT, KW, PER>(red, lane, v0, a0, a1);
  if (n_slices > 1) {
    const int64_t unit = (int64_t)task * gridDim.z + group;
    put_slice<TT, PER>(part, unit * n_slices + slice, lane, v0, a0, a1);
    if (!last_arrival(tickets + unit, n_slices, &s_flag)) return;
    TRACE_MARK(KID, 3);
    sum_slices<TT, PER>(part, unit, n_slices, lane, v0, a0, a1);
  }
  [[maybe_unused]] typename ET<E>::vec rc[4];   // the chain's router weights: experts of half wave & 1, for token tile wave / 2
  if constexpr (CHAIN) {
    if (epi.w_router) {
#pragma unroll
      for (int i = 0; i < 4; ++i) rc[i] = load16<E>(epi.w_router + (((int64_t)task * 4 + i) * 2 + (wave & 1)) * (WAVE * ET<E>::G) + lane * ET<E>::G);
    }
  }
  float ss[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const int tok = tok0 + t * TILE + (lane & 31);
    ss[t] = epi.template apply<PER>(pre[t], task, tok, tok < T, half, v0, a0[t], a1[t], TT == 1);
  }
  if constexpr (Epi::ROWSUM) {
    // the task's row statistic: both half-waves of a column, then the KW waves in order
    const bool routed = (STEPS || CHAIN) && epi.w_router != nullptr;
    if constexpr (STEPS) {
      if (routed) {
        // wave w holds features 8w .. 8w + 7 of both tiles, the depth of two instructions each; summed over the waves like the statistic
        static_assert(PER == 4, "RouterStep");
        f32x16 r0[TT], r1[TT];
        zero_acc<TT>(r0);
        zero_acc<TT>(r1);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          f32x4 m[2];
          Epi::normed(pre[t], a0[t], a1[t], m);
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            RouterStep::add(r0[t], rw[f][0], m[f]);
            RouterStep::add(r1[t], rw[f][1], m[f]);
          }
        }
        __syncthreads();   // the partials in `red` are consumed
        spill_partials<TT, ROWS>(red, wave, lane, r0, r1);
      }
    }
    [[maybe_unused]] E* planes = reinterpret_cast<E*>(red);   // [token tile][k-step][plane][half-lane][token][8], an operand fragment each
    if constexpr (CHAIN) {
      if (routed) {
        static_assert(Planes<E>::N == 2 && ET<E>::KS == 16 && KW == 4, "a wave's registers are half a k-step of each tile");
        __syncthreads();   // the partials in `red` are consumed
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          f32x4 m[2];
          Epi::normed(pre[t], a0[t], a1[t], m);
#pragma unroll
          for (int f = 0; f < 2; ++f)   // features 32 f + 8 wave + 4 half ..
            store_act4<E>(planes, ((((t * 4 + 2 * f + (wave >> 1)) * 2) * 2 + (wave & 1)) * TILE + (lane & 31)) * 8 + 4 * half, 2 * TILE * 8, m[f]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const float s2 = ss[t] + __shfl_xor(ss[t], 32, WAVE);
      if (half == 0) s_ss[(wave * TT + t) * TILE + lane] = s2;
    }
    __syncthreads();
    if constexpr (STEPS) {
      if (routed) {
        float b0[TT][PER], b1[TT][PER];
        fold_partials<TT, KW, PER>(red, lane, v0, b0, b1);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          const int tok = tok0 + t * TILE + (lane & 31);
          if (tok < T) {
            epi.store_share(task, tok, acc_row(v0, half), f32x4{b0[t][0], b0[t][1], b0[t][2], b0[t][3]});
            epi.store_share(task, tok, TILE + acc_row(v0, half), f32x4{b1[t][0], b1[t][1], b1[t][2], b1[t][3]});
          }
        }
      }
    }
    if constexpr (CHAIN) {
      if (routed) {
        typedef typename ET<E>::vec vec;
        f32x16 z;
#pragma unroll
        for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            mfma32(z, rc[i], *reinterpret_cast<const vec*>(planes + (((((wave >> 1) * 4 + i) * 2 + q) * 2 + half) * TILE + (lane & 31)) * 8));
        const int tok = tok0 + (wave >> 1) * TILE + (lane & 31);
        if (tok < T) {
#pragma unroll
          for (int g = 0; g < 4; ++g)
            epi.store_share(task, tok, (wave & 1) * TILE + acc_row(4 * g, half), f32x4{z[4 * g], z[4 * g + 1], z[4 * g + 2], z[4 * g + 3]});
        }
      }
    }
    for (int i = threadIdx.x; i < TT * TILE; i += KW * WAVE) {
      float s = 0.f;
      for (int w = 0; w < KW; ++w) s += s_ss[w * TT * TILE + i];
      const int tok = tok0 + i;
      if (tok < T) epi.row_sum(task, tok, s);
    }
  }
  TRACE_MARK(KID, 4);
}

template <int TT, int KW> constexpr size_t ksplit_lds() { return (size_t)KW * 2 * TT * 16 * WAVE * 4; }

template <typename E, class Epi>
static void launch_ksplit(bool bf16, const E* W, int ksteps, const E* B, int T, int K, int n_tasks,
                          float* part, int32_t* tickets, const Epi& epi, hipStream_t st) {
  const int slices = single_slice() ? 1 : ksplit_slices(bf16, K, T, n_tasks);
  if (T <= 32) {
    gemm_ksplit_kernel<E, 1, 4, Epi><<<dim3(slices, n_tasks, 1), 4 * WAVE, ksplit_lds<1, 4>(), st>>>(W, ksteps, B, T, K, part, tickets, epi, live_word());
  } else if (T <= 64) {
    gemm_ksplit_kernel<E, 2, 4, Epi><<<dim3(slices, n_tasks, 1), 4 * WAVE, ksplit_lds<2, 4>(), st>>>(W, ksteps, B, T, K, part, tickets, epi, live_word());
  } else {
    const int groups = (T + 4 * TILE - 1) / (4 * TILE);
    gemm_ksplit_kernel<E, 4, 4, Epi><<<dim3(1, n_tasks, groups), 4 * WAVE, ksplit_lds<4, 4>(), st>>>(W, ksteps, B, T, K, part, tickets, epi, live_word());
  }
}

// ------------------------------------------------------------------------------------------------
// Output projection of up to 32 tokens in bfloat16 that leaves the router's shares of 128 features (router_share_features).  The
// contraction of the router adds in chains of eight k-steps, two tasks, and a sum that runs on from the first task's into the second's
// cannot be put together from two.  So the slices of two tasks meet in one workgroup, which runs the epilogue of both and then the
// chain: the planes of the 128 features as operands in LDS, a wave per 32 experts.  Everything else, and every sum, as in the split-K kernel.
// The operands of the epilogues are asked for with the slices, behind the hand-off (in front of the stream: 0.4 us more).  Bound by the
// hand-off and by what one compute unit fetches behind it; with the events around the launches, hidden 2048 and 32 tokens: output projection
// 13.2 us and selection 6.7; with a task's shares 11.2 and 6.7, in another order; without shares 10.1, and 13.3 for the router's contraction.
// ------------------------------------------------------------------------------------------------
template <typename E, int KW>
__global__ __launch_bounds__(KW * WAVE) void oproj_pair_kernel(const E* __restrict__ W, int ksteps, const E* __restrict__ B, int T,
                                                               float* __restrict__ part, int32_t* __restrict__ tickets, ResidualEpi<E> epi,
                                                               const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  constexpr int ROWS = 32, PER = 16 / KW, KS = ET<E>::KS, G = ET<E>::G, CHAIN = ROUTER_CHAIN;
  static_assert(Planes<E>::N == 2 && KS == 16 && KW == 4 && CHAIN * KS == 128, "a wave's registers are half a k-step of each tile");
  extern __shared__ __align__(16) float red[];   // [KW][ROWS][64], then the chain's operands
  __shared__ int32_t s_flag;
  __shared__ float s_ss[KW * 2 * TILE];
  const int slice = blockIdx.x, n_slices = gridDim.x, task = blockIdx.y, pair = task >> 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int v0 = wave * PER;
  const bool valid = col < T;
  TRACE_MARK(2, 0);
  float a0[1][PER], a1[1][PER];
  {
    f32x16 acc0[1], acc1[1];
    zero_acc<1>(acc0);
    zero_acc<1>(acc1);
    const int per = (ksteps + n_slices * KW - 1) / (n_slices * KW);
    const int ks0 = min(ksteps, (slice * KW + wave) * per), ks1 = min(ksteps, ks0 + per);
    PlaneLoader<E, 1> ld;
    ld.set(0, B, T, min(col, T - 1), half);
    stream_task<E, 1, 8>(W + (int64_t)task * task_stride_elems<E>(ksteps), ks0, ks1, ld, acc0, acc1);
    TRACE_MARK(2, 1);
    spill_partials<1, ROWS>(red, wave, lane, acc0, acc1);
    __syncthreads();
    TRACE_MARK(2, 2);
    fold_partials<1, KW, PER>(red, lane, v0, a0, a1);
  }
  // the slices of two token tiles of one task (sum_slices) are here those of one tile of two tasks
  const buf_rsrc out = coherent_buffer(part);
  const int64_t piece = (int64_t)pair * n_slices + slice;
  coherent_store_n<PER>(out, slice_piece<2, PER>(piece, task & 1, 0, v0, lane), a0[0]);
  coherent_store_n<PER>(out, slice_piece<2, PER>(piece, task & 1, 1, v0, lane), a1[0]);
  if (!last_arrival(tickets + pair, 2 * n_slices, &s_flag)) return;
  TRACE_MARK(2, 3);
  vec rw[CHAIN];   // router weights of the wave's 32 experts
  if (wave < 2) {
#pragma unroll
    for (int i = 0; i < CHAIN; ++i) rw[i] = load16<E>(epi.w_router + ((int64_t)(pair * CHAIN + i) * 2 + wave) * (WAVE * G) + lane * G);
  }
  typename ResidualEpi<E>::template Pre<PER> pre[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) pre[p] = epi.template prefetch<PER>(2 * pair + p, col, valid, half, v0);
  float s0[2][PER], s1[2][PER];
  sum_slices<2, PER>(part, pair, n_slices, lane, v0, s0, s1);
  E* planes = reinterpret_cast<E*>(red);   // [k-step][plane][half-lane][token][8], an operand fragment each
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const float ss = epi.template apply<PER>(pre[p], 2 * pair + p, col, valid, half, v0, s0[p], s1[p], true);
    const float s2 = ss + __shfl_xor(ss, 32, WAVE);
    if (half == 0) s_ss[(wave * 2 + p) * TILE + col] = s2;
    f32x4 m[2];
    ResidualEpi<E>::normed(pre[p], s0[p], s1[p], m);
#pragma unroll
    for (int f = 0; f < 2; ++f) {          // features 64 p + 32 f + 8 wave + 4 half ..
      const int ks = 4 * p + 2 * f + (wave >> 1);
      store_act4<E>(planes, (((ks * 2) * 2 + (wave & 1)) * TILE + col) * 8 + 4 * half, 2 * TILE * 8, m[f]);
    }
  }
  __syncthreads();
  if (wave < 2) {
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
#pragma unroll
    for (int i = 0; i < CHAIN; ++i)
#pragma unroll
      for (int q = 0; q < 2; ++q) mfma32(z, rw[i], *reinterpret_cast<const vec*>(planes + (((i * 2 + q) * 2 + half) * TILE + col) * 8));
    if (valid) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        epi.store_share(pair, col, wave * TILE + acc_row(4 * g, half), f32x4{z[4 * g], z[4 * g + 1], z[4 * g + 2], z[4 * g + 3]});
    }
  } else if (wave == 2 && valid) {         // the tasks' row statistics: the KW waves in order
    float s = 0.f;
    for (int w = 0; w < KW; ++w) s += s_ss[(w * 2 + half) * TILE + col];
    epi.row_sum(2 * pair + half, col, s);
  }
  TRACE_MARK(2, 4);
}

// ------------------------------------------------------------------------------------------------
// QKV projection of up to 32 tokens with 32 features (half a task) per workgroup (rule and figures: half_applies): HALF_KW waves
// cut the whole K range, every wave has its share in flight at once, and the sums meet in LDS.  Bound by memory latency like the
// split-K kernel, whose two slices per task need a hand-off between workgroups (about 3 us) to get as many bytes under way.
// The matrix instruction's 32 rows are 16 of each of the task's two tiles, so that an epilogue still finds its pairs (feature
// j and its rotary partner, rows r and r + 16) in one lane: registers v and v + 8.  Sums in the order of the split-K kernel
// with two slices, bit for bit.
// ------------------------------------------------------------------------------------------------
template <typename E, class Epi>
__global__ __launch_bounds__(HALF_KW * WAVE) __attribute__((amdgpu_waves_per_eu(2))) void gemm_half_kernel(const E* __restrict__ W, int ksteps, const E* __restrict__ B, int T,
                                                                   Epi epi, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  constexpr int G = ET<E>::G, NP = Planes<E>::N, PER = 4, EW = 2;   // the first EW waves run the epilogue
  __shared__ float red[HALF_KW * 16 * WAVE];
  const int task = blockIdx.x >> 1, sub = blockIdx.x & 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int v0 = (wave < EW ? wave : 0) * PER, tok = col;
  TRACE_MARK(1, 0);
  auto pre = epi.template prefetch<PER>(task, tok, tok < T, half, 8 * sub + v0);
  const int per = ksteps / HALF_KW, ks0 = wave * per;    // per: HALF_PF or half of it
  // lane l of the operand: row l % 16 of this half, tile (l / 16) % 2, k half l / 32
  const E* wp = W + (int64_t)task * task_stride_elems<E>(ksteps) + (int64_t)ks0 * (2 * WAVE * G) +
                ((lane >> 4 & 1) * WAVE + half * TILE + sub * 16 + (lane & 15)) * G;
  PlaneLoader<E, 1> ld;
  ld.set(0, B, T, min(tok, T - 1), half);
  f32x16 acc[1];
  zero_acc<1>(acc);
  auto stream = [&](auto N) {
    constexpr int PF = decltype(N)::value;
    vec a[PF];
    typename PlaneLoader<E, 1>::Raw raw[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) a[i] = load16_stream<E>(wp + (int64_t)i * (2 * WAVE * G));
#pragma unroll
    for (int i = 0; i < PF; ++i) raw[i] = ld.issue(0, ks0 + i);
    __builtin_amdgcn_sched_barrier(0);   // all of them before the first product
#pragma unroll
    for (int i = 0; i < PF; ++i)
#pragma unroll
      for (int q = 0; q < NP; ++q) mfma32(acc[0], a[i], raw[i].p[q]);
  };
  if (per == HALF_PF) stream(std::integral_constant<int, HALF_PF>{});
  else stream(std::integral_constant<int, HALF_PF / 2>{});
  TRACE_MARK(1, 1);
  if (wave < EW) epi.template prefetch2<PER>(pre, task, half, 8 * sub + v0);
#pragma unroll
  for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * WAVE + lane] = acc[0][v];
  __syncthreads();
  TRACE_MARK(1, 2);
  if (wave >= EW) return;
  float a0[PER], a1[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) a0[i] = a1[i] = 0.f;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    float b0[PER], b1[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) b0[i] = b1[i] = 0.f;
#pragma unroll
    for (int w = 0; w < HALF_KW / 2; ++w) {
      const float* r = red + ((s * (HALF_KW / 2) + w) * 16 + v0) * WAVE + lane;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        b0[i] += r[i * WAVE];
        b1[i] += r[(8 + i) * WAVE];
      }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      a0[i] += b0[i];
      a1[i] += b1[i];
    }
  }
  epi.template apply<PER>(pre, task, tok, tok < T, half, 8 * sub + v0, a0, a1, true);
  TRACE_MARK(1, 4);
}

// Static + dynamic LDS of these kernels can pass the 64 KiB default: opt in to the 160 KiB LDS of gfx950
// (dynamic limit = what the kernel's static LDS leaves).  Returns false if the runtime refuses.
static bool opt_in_lds(const void* fn) {
  hipFuncAttributes fa;
  if (hipFuncGetAttributes(&fa, fn) != hipSuccess) return false;
  const int room = 160 * 1024 - (int)fa.sharedSizeBytes;
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, room) == hipSuccess;
}
template <typename E, class Epi> static bool configure_ksplit() {
  return opt_in_lds((const void*)gemm_ksplit_kernel<E, 1, 4, Epi>) &&
         opt_in_lds((const void*)gemm_ksplit_kernel<E, 2, 4, Epi>) &&
         opt_in_lds((const void*)gemm_ksplit_kernel<E, 4, 4, Epi>);
}
static_assert(ksplit_lds<1, 4>() >= ROUTER_CHAIN * 2 * 2 * TILE * 16, "the chain's operands take the place of the partial sums");

// ------------------------------------------------------------------------------------------------
// Down projection of the routed experts fused with the weighted combine, the residual add and the statistics of
// the norm that follows, for at most 32 tokens.  The sum over a token's k experts is a contraction like any other:
//   x[t][f] += sum_e sum_i  y[e][t][i] * Wd[e][f][i]      (y already carries the routing weight; y[e][t] = 0
//                                                           for tokens that were not routed to expert e)
// so a task (64 output features) runs over the "long K" of all experts that received rows, 64 k-steps each, with
// the token tile as the MFMA columns: a lane whose token is not among an expert's rows feeds zeros.  The long K is
// cut into pieces for n_slices x KW waves; wave sums are folded through LDS, workgroup sums through the
// cross-workgroup hand-off of the split-K kernel, in fixed order, and the last workgroup of a task runs the
// residual epilogue.  No per-(token, expert) output rows are stored and no separate combine pass runs; and because
// the work is cut by weight bytes, a layer that touches 8 experts fills the chip as well as one that touches 60.
// ------------------------------------------------------------------------------------------------
template <typename E, int TT, int KW, int PF>
__global__ __launch_bounds__(KW * WAVE) void expert_down_fused_kernel(const E* __restrict__ W, const E* __restrict__ Y,
                                                                       int64_t y_rows, const int32_t* __restrict__ topk_idx, int T,
                                                                       int I, int top_k, int n_tasks,
                                                                       float* __restrict__ part,
                                                                       int32_t* __restrict__ tickets, ResidualEpi<E> epi, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  extern __shared__ float red[];   // [KW][2*TT*16][64]
  __shared__ int32_t s_flag;
  constexpr int G = ET<E>::G, KS = ET<E>::KS, NP = Planes<E>::N, ROWS = 2 * TT * 16;
  constexpr int EW = 4, PER = 16 / EW;   // the first EW waves run the epilogue, four accumulator registers each
  static_assert(KW >= EW && MAX_EXPERTS <= WAVE, "epilogue waves; one lane per listed expert");
  constexpr int64_t STEP = 2 * WAVE * G;
  const int slice = blockIdx.x, n_slices = gridDim.x, task = blockIdx.y;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  TRACE_MARK(5, 0);
  TRACE_MARK_WAVE(55, 0, KW);
  // The first loads hang on the routing alone: this lane's tokens' experts, from which the wave reads off the list of
  // experts with rows and, for the two of them it meets, where its tokens' rows sit in Y (sorted by expert, then token).
  static_assert(TT == 1, "TokenExperts");
  TokenExperts tokens;
  tokens.load(topk_idx, T, top_k);
  const uint64_t experts = tokens.experts();
  const int n_act = __popcll(experts);
  // The long K: experts with rows in list order, ksteps_e k-steps each, in groups of PF k-steps; this wave's
  // contiguous share [g0, g1).  A share is never longer than one expert's groups, so it meets at most two experts.  Float32: shares of
  // equal length rounded down or up, so that each workgroup has the same number of groups within one; shares all rounded up leave the
  // last ones short (the float32 test model 14.5 against 12.3 us with events around the launch).  In bfloat16 they are all rounded up: the cut
  // is the order of the sum, and in another order outputs of sixteen layers differ where an expert is a tie (router_share_features).
  // It costs 42.0 against 40.1 us on average over batch-1 layers of 21 to 58 experts (50 experts: 57 of 64 waves have seven groups each).
  constexpr bool EVEN = sizeof(E) == 4;
  const int ksteps_e = I / KS, groups_e = ksteps_e / PF, total = n_act * groups_e;
  const int units = n_slices * KW, unit = slice * KW + wave, per = (total + units - 1) / units;
  const int g0 = EVEN ? total * unit / units : min(total, unit * per), g1 = EVEN ? total * (unit + 1) / units : min(total, g0 + per);
  const int i0 = g0 / groups_e;
  const int e_first = nth_bit(experts, min(i0, n_act - 1)), e_second = nth_bit(experts, min(i0 + 1, n_act - 1));
  const E* wbase = W + (int64_t)task * task_stride_elems<E>(ksteps_e) + lane * G;
  const int64_t wexpert = (int64_t)n_tasks * task_stride_elems<E>(ksteps_e);
  auto weights_of = [&](int g) { return wbase + (g / groups_e == i0 ? e_first : e_second) * wexpert + (g % groups_e) * PF * STEP; };
  // Which Y row this lane reads for group g (byte offset of its first k-step) and how far it moves per k-step.
  // Y is read through a buffer descriptor with hardware range checking: a lane whose token was not routed to the
  // group's expert is given an offset past the end, for which the load returns zeros without touching memory --
  // exactly the operand such a token contributes.
  const __amdgpu_buffer_rsrc_t ybuf = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<E*>(Y), 0, (uint32_t)(y_rows * I * NP * sizeof(E)), 0x00020000);
  constexpr uint32_t ROW_BYTES = NP * KS * sizeof(E), PAST_END = 0x80000000u;
  const uint32_t ykstride = (uint32_t)y_rows * ROW_BYTES;
  int row_first = 0, row_second = 0;   // set behind the first weights
  auto rows_of = [&](int g, uint32_t (&yoff)[TT], uint32_t (&ystep)[TT]) {
    const int kk = (g % groups_e) * PF, row = g / groups_e == i0 ? row_first : row_second;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      yoff[t] = row >= 0 ? ((uint32_t)kk * (uint32_t)y_rows + row) * ROW_BYTES + half * 16 : PAST_END;
      ystep[t] = row >= 0 ? ykstride : 0;
    }
  };
  f32x16 acc0[TT], acc1[TT];
  zero_acc<TT>(acc0);
  zero_acc<TT>(acc1);
  vec a0[PF], a1[PF], yr[PF][TT][NP];
  auto issue_w = [&](int i, const E* wp) {
    a0[i] = load16_stream<E>(wp + i * STEP);
    a1[i] = load16_stream<E>(wp + i * STEP + WAVE * G);
  };
  auto issue_y = [&](int i, const uint32_t (&yoff)[TT], const uint32_t (&ystep)[TT]) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int q = 0; q < NP; ++q)
        yr[i][t][q] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(
                                                  ybuf, yoff[t] + i * ystep[t] + q * (uint32_t)(KS * sizeof(E)), 0, 0));
  };
  auto use = [&](int i) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        mfma32(acc0[t], a0[i], yr[i][t][q]);
        mfma32(acc1[t], a1[i], yr[i][t][q]);
      }
  };
  if (g0 < g1) {
    {
      const E* wp = weights_of(g0);
      TRACE_MARK_WAVE(55, 1, KW);
#pragma unroll
      for (int i = 0; i < PF; ++i) issue_w(i, wp);
      row_first = tokens.row_of(e_first);
      row_second = tokens.row_of(e_second);
      uint32_t yoff[TT], ystep[TT];
      rows_of(g0, yoff, ystep);
#pragma unroll
      for (int i = 0; i < PF; ++i) issue_y(i, yoff, ystep);
    }
    auto group = [&](int g) {
      if (g == g0 + 1) TRACE_MARK(5, 5);
      if (g == g0 + 2) TRACE_MARK(5, 6);
      if (g == g0 + 4) TRACE_MARK(5, 7);
      if (g == g0) TRACE_MARK_WAVE(55, 2, KW);
      if (g == g0 + 1) TRACE_MARK_WAVE(55, 3, KW);
      if (g == g0 + 3) TRACE_MARK_WAVE(55, 4, KW);
      const E* wn = weights_of(g + 1);
      uint32_t yn[TT], ynstep[TT];
      rows_of(g + 1, yn, ynstep);
      // k-step by k-step: multiply, then request the same slot of the next group.  The scheduling barriers keep
      // the compiler from collecting the requests at the end of the iteration (it then waits for all of them at
      // the top of the next one and the memory pipe idles while the group is multiplied).
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        use(i);
        __builtin_amdgcn_sched_barrier(0);
        issue_w(i, wn);
        issue_y(i, yn, ynstep);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // The first group stands in front of the loop: it meets the loads in the prologue's order (all weights, then
    // all rows), the later ones in the order the groups leave them (slot by slot), and wait counts at the top of a
    // loop that is entered both ways are the smaller of the two: slot 0 then waited for half the group in flight.
    if (g0 + 1 < g1) {
      group(g0);
      for (int g = g0 + 1; g + 1 < g1; ++g) group(g);
    }
#pragma unroll
    for (int i = 0; i < PF; ++i) use(i);
  }
  // Epilogue by the first EW waves (the others only keep the workgroup's barriers company).
  const bool worker = wave < EW;
  const int v0 = (worker ? wave : 0) * PER;
  typename ResidualEpi<E>::template Pre<PER> pre[TT];
  if (worker) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int tok = t * TILE + col;
      pre[t] = epi.template prefetch<PER>(task, tok, tok < T, half, v0);
    }
  }
  TRACE_MARK(5, 1);
  TRACE_MARK_WAVE(55, 5, KW);
  spill_partials<TT, ROWS>(red, wave, lane, acc0, acc1);
  __syncthreads();
  TRACE_MARK(5, 2);
  float s0[TT][PER], s1[TT][PER];
  if (worker) fold_partials<TT, KW, PER>(red, lane, v0, s0, s1);
  if (n_slices > 1) {
    if (worker) put_slice<TT, PER>(part, (int64_t)task * n_slices + slice, lane, v0, s0, s1);
    if (!last_arrival(tickets + task, n_slices, &s_flag)) return;
    TRACE_MARK(5, 3);
    if (worker) sum_slices<TT, PER, 8>(part, task, n_slices, lane, v0, s0, s1);
  }
  float ss[TT];
  if (worker) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int tok = t * TILE + col;
      ss[t] = epi.template apply<PER>(pre[t], task, tok, tok < T, half, v0, s0[t], s1[t], true);
    }
  }
  __syncthreads();   // the partials in `red` are consumed
  if (worker) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const float s2 = ss[t] + __shfl_xor(ss[t], 32, WAVE);
      if (half == 0) red[(wave * TT + t) * TILE + lane] = s2;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < TT * TILE; i += KW * WAVE) {
    float s = 0.f;
    for (int w = 0; w < EW; ++w) s += red[w * TT * TILE + i];
    if (i < T) epi.row_sum(task, i, s);
  }
  TRACE_MARK(5, 4);
}

// ------------------------------------------------------------------------------------------------
// Dense projections over many token rows (more than 64).  A workgroup takes TASKS (eight, four or two) tasks and up to WT token
// tiles; its TASKS * KH waves are KH teams, each team with its own share of the K range, its own LDS staging area for the
// activation fragments (wide_stream.hpp) and one wave per task, which streams that task's weights once and keeps
// the accumulators of 64 features x WT*32 rows.  The teams' sums are folded through LDS at the end, each
// team taking a part of them through the epilogue (those of the split-K kernel, called for four accumulator registers at a time).  KH > 1 puts
// several waves on every SIMD, so that one multiplies while another waits for LDS or memory, without asking the
// launch for more workgroups than there are (task, token) tiles.
// Grid (task groups, token groups): with a multiple of eight task groups the workgroups of one die always take the
// same tasks, so the weights (a few MB per die) are read from HBM once and then served by that die's L2.
// ------------------------------------------------------------------------------------------------
// Measured at 512 tokens (QKV / output projection, microseconds): one team 58 / 34, two teams 58 / 34 before and
// 41 / 29 after the epilogue stores were widened, four teams of one token tile 94 / 37; four token tiles per
// workgroup 102 / 95 (too few workgroups); two tasks per workgroup 57 / 19 (the output projection, with 32 tasks,
// then fills the chip with 256 workgroups).
constexpr int DENSE_KH = 2;
static_assert(DENSE_TILE == TILE, "dense_plan.hpp counts in these units");

template <typename E, int KID, int WT, int TASKS, int KH> constexpr size_t dense_lds() {
  const size_t stage = KH * wide_lds<E, KID, WT>();
  const size_t fold = KH > 1 ? (size_t)KH * TASKS * 32 * WAVE * 4 : 0;   // at most 32 registers a wave from either team
  return stage > fold ? stage : fold;
}

// The token tiles go to the gridDim.y token groups WT by WT, with four tiles evenly (at most four each).
template <typename E, int WT, int TASKS, int KH, class Epi>
__global__ __launch_bounds__(TASKS * KH * WAVE) void gemm_dense_kernel(const E* __restrict__ W, int ksteps,
                                                                       const E* __restrict__ B, int T, int n_tasks,
                                                                       Epi epi, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  constexpr int G = ET<E>::G, KS = ET<E>::KS, NP = Planes<E>::N, PER = 4;
  constexpr int KID = Epi::ROWSUM ? 13 : 12;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int team = wave / TASKS, rank = wave % TASKS;
  const int slot = blockIdx.x * TASKS + rank, task = min(slot, n_tasks - 1);
  // (divisions only where the groups are unequal: they cost the small forms 0.6 us a launch; tiles * groups fits 32 bits)
  const uint32_t tiles = (T + TILE - 1) / TILE;
  const int tile0 = WT < 4 ? blockIdx.y * WT : tiles * blockIdx.y / gridDim.y;
  const int nt = WT < 4 ? min(WT, (int)tiles - tile0) : (int)(tiles * (blockIdx.y + 1) / gridDim.y) - tile0;
  const int tok0 = tile0 * TILE;
  const int ks_team = ksteps / (WKC * KH) * WKC, ks0 = team * ks_team;
  vec* sb = reinterpret_cast<vec*>(lds_raw + team * wide_lds<E, KID, WT>());
  auto row_of = [&](int r) { return min(tok0 + (rank % WT) * TILE + r, T - 1); };
  f32x16 acc0[WT], acc1[WT];
  zero_acc<WT>(acc0);
  zero_acc<WT>(acc1);
  wide_stream<E, WT, TASKS, KID>(
      W + (int64_t)task * task_stride_elems<E>(ksteps) + (int64_t)ks0 * (2 * WAVE * G), ks_team, B + (int64_t)ks0 * T * (NP * KS), row_of,
      (int64_t)T * (NP * KS), sb, nt, acc0, acc1, rank);
  constexpr int NG = 16 / PER;
  // Epilogue of register groups G0 .. G0 + GN - 1 of token tile t, in three sweeps over them, so that the loads of one sweep are
  // all in flight together: what is addressed by the token, what is addressed by what those loads return, then the arithmetic.
  auto finish = [&](auto Tile, auto First, auto Count) {
    constexpr int t = decltype(Tile)::value, G0 = decltype(First)::value, GN = decltype(Count)::value;
    const int tok = tok0 + t * TILE + col;
    const bool valid = t < nt && tok < T;
    typename Epi::template Pre<PER> pre[GN];
#pragma unroll
    for (int g = 0; g < GN; ++g) pre[g] = epi.template prefetch<PER>(task, tok, valid, half, (G0 + g) * PER);
#pragma unroll
    for (int g = 0; g < GN; ++g) epi.template prefetch2<PER>(pre[g], task, half, (G0 + g) * PER);
    constexpr bool SHARES = Epi::ROWSUM && WT == 1 && sizeof(E) == 4;   // (with more tiles they do not fit the registers)
    [[maybe_unused]] f32x4 rw[2][GN][2];   // [tile][eight features][experts from 0, from 32]
    [[maybe_unused]] f32x16 r0[1], r1[1];
    bool routed = false;
    if constexpr (SHARES) {
      zero_acc<1>(r0);
      zero_acc<1>(r1);
      routed = epi.w_router != nullptr;
      if (routed) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int g = 0; g < GN; ++g)
#pragma unroll
            for (int et = 0; et < 2; ++et) rw[f][g][et] = RouterStep::load(epi.w_router, task, f, G0 + g, et, lane);
      }
    }
    float ss = 0.f;
#pragma unroll
    for (int g = 0; g < GN; ++g) {
      float a0[PER], a1[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        a0[i] = acc0[t][(G0 + g) * PER + i];
        a1[i] = acc1[t][(G0 + g) * PER + i];
      }
      ss += epi.template apply<PER>(pre[g], task, tok, valid, half, (G0 + g) * PER, a0, a1, WT == 4 && G0 + g == 0);
      if constexpr (SHARES) {
        if (routed) {
          f32x4 m[2];
          Epi::normed(pre[g], a0, a1, m);
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            RouterStep::add(r0[0], rw[f][g][0], m[f]);
            RouterStep::add(r1[0], rw[f][g][1], m[f]);
          }
        }
      }
    }
    if constexpr (SHARES) {
      if (routed && valid) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          epi.store_share(task, tok, acc_row(4 * g, half), f32x4{r0[0][4 * g], r0[0][4 * g + 1], r0[0][4 * g + 2], r0[0][4 * g + 3]});
          epi.store_share(task, tok, TILE + acc_row(4 * g, half), f32x4{r1[0][4 * g], r1[0][4 * g + 1], r1[0][4 * g + 2], r1[0][4 * g + 3]});
        }
      }
    }
    if (Epi::ROWSUM) {   // the wave holds the whole task: the row statistic is the sum over its two half-waves
      static_assert(!Epi::ROWSUM || GN == NG, "all features of the task");
      ss += __shfl_xor(ss, 32, WAVE);
      if (half == 0 && valid) epi.row_sum(task, tok, ss);
    }
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, NG> All;
  if constexpr (KH > 1) {
    // fold through red[sender][rank][register][lane].  The teams share the epilogue where it can be cut: each takes a token tile, or
    // half of the registers of the only one, gets the other's sums of those and adds them to its own.  (Team 0 alone: QKV at 512 tokens
    // 44.1 us, 42.9 with both; 384 41.5 and 40.8; 160 21.0 and 19.7; 256 26.1 and 25.7; asking for the epilogue's operands in front of the
    // fold gains nothing more.)
    static_assert(KH == 2 && WT <= 2, "two teams, a tile each");
    constexpr bool CUT = WT == 2 || !Epi::ROWSUM;                  // (a row statistic needs all features of the tile)
    constexpr int REGS = WT == 2 || !CUT ? 32 : 16, HG = NG / 2;   // registers a team sends
    float* red = reinterpret_cast<float*>(lds_raw) + (int64_t)rank * REGS * WAVE + lane;
    constexpr int SENDER = TASKS * REGS * WAVE;
    auto send = [&](auto Tile, auto First) {
      constexpr int t = decltype(Tile)::value, v = decltype(First)::value;
      float* r = red + team * SENDER;
#pragma unroll
      for (int i = 0; i < REGS / 2; ++i) {
        r[i * WAVE] = acc0[t][v + i];
        r[(REGS / 2 + i) * WAVE] = acc1[t][v + i];
      }
    };
    auto receive = [&](auto Tile, auto First) {
      constexpr int t = decltype(Tile)::value, v = decltype(First)::value;
      const float* r = red + (1 - team) * SENDER;
#pragma unroll
      for (int i = 0; i < REGS / 2; ++i) {
        acc0[t][v + i] += r[i * WAVE];
        acc1[t][v + i] += r[(REGS / 2 + i) * WAVE];
      }
    };
    typedef std::integral_constant<int, 8> I8;
    typedef std::integral_constant<int, HG> IH;
    __syncthreads();   // the staging areas are done with
    if constexpr (!CUT) {
      if (team > 0) send(I0{}, I0{});
    } else if constexpr (WT == 2) {
      if (team == 0) send(I1{}, I0{});
      else send(I0{}, I0{});
    } else {
      if (team == 0) send(I0{}, I8{});
      else send(I0{}, I0{});
    }
    __syncthreads();
    if (slot >= n_tasks) return;
    if (team == 0) {
      receive(I0{}, I0{});
      if constexpr (CUT && WT == 1) finish(I0{}, I0{}, IH{});
      else finish(I0{}, I0{}, All{});
    } else if constexpr (CUT && WT == 2) {
      receive(I1{}, I0{});
      finish(I1{}, I0{}, All{});
    } else if constexpr (CUT) {
      receive(I0{}, I8{});
      finish(I0{}, IH{}, IH{});
    }
  } else {
    if (slot >= n_tasks) return;
    static_for<WT>([&](auto I) { finish(I, I0{}, All{}); });   // (the accumulators of four tiles leave no room for all at once)
  }
  TRACE_MARK(KID, 7);
}

// True when the dense form takes the call (many rows, K a whole number of staged chunks per team).
// (Above 64 tokens.  With two token tiles the split-K form of the QKV projection used to hand 12.6 MB of partial
// sums between workgroups, 8 slices per task, and the dense form was faster, 19.1 against 27.9 us; with the two
// slices that ksplit_slices() now gives a launch of 96 tasks it takes 14.9 us.  For the output projection, a third
// of the weights, split-K was ahead all along, 11.5 against 17.1.)
static bool dense_applies(int T, int ksteps) { return T > 2 * TILE && ksteps % (WKC * DENSE_KH) == 0; }
int router_share_features(bool bf16, int D, int H, int T) {
  if (single_slice()) return 0;
  if (bf16) {
    const int features = T <= TILE ? ROUTER_CHAIN * 16 : T <= 2 * TILE ? ROUTER_CHAIN * 8 : 0;
    return features && H % (ROUTER_WAVES * features) == 0 ? features : 0;
  }
  if (T <= 2 * TILE) return 64;
  return T <= ROUTER_SHARES_T && dense_applies(T, D / 8) && dense_form(false, H / 64, T).tiles == 1 ? 64 : 0;
}

template <typename E, int WT, int TASKS, int KH, class Epi>
static void launch_dense_as(const E* W, int ksteps, const E* B, int T, int n_tasks, int groups, const Epi& epi, hipStream_t st) {
  constexpr int KID = Epi::ROWSUM ? 13 : 12;
  gemm_dense_kernel<E, WT, TASKS, KH, Epi><<<dim3((n_tasks + TASKS - 1) / TASKS, groups),
                                            TASKS * KH * WAVE, dense_lds<E, KID, WT, TASKS, KH>(), st>>>(W, ksteps, B, T, n_tasks,
                                                                                                       epi, live_word());
}
// More tasks and token tiles per workgroup cut the operand traffic, but only while the launch still fills the chip.
template <typename E, class Epi>
static void launch_dense(const E* W, int ksteps, const E* B, int T, int n_tasks, const Epi& epi, hipStream_t st) {
  const DenseForm f = dense_form(sizeof(E) == 2, n_tasks, T);
  if (f.tasks == DENSE_WIDE_TASKS) {
    if constexpr (sizeof(E) == 2) launch_dense_as<E, DENSE_WIDE_TILES, DENSE_WIDE_TASKS, 1, Epi>(W, ksteps, B, T, n_tasks, f.groups, epi, st);
  } else if (f.tiles == 2) launch_dense_as<E, 2, 4, DENSE_KH, Epi>(W, ksteps, B, T, n_tasks, f.groups, epi, st);
  else if (f.tasks == 4) launch_dense_as<E, 1, 4, DENSE_KH, Epi>(W, ksteps, B, T, n_tasks, f.groups, epi, st);
  else launch_dense_as<E, 1, 2, DENSE_KH, Epi>(W, ksteps, B, T, n_tasks, f.groups, epi, st);
}

template <typename E, class Epi> static bool configure_dense() {
  if constexpr (sizeof(E) == 2)
    if (!opt_in_lds((const void*)gemm_dense_kernel<E, DENSE_WIDE_TILES, DENSE_WIDE_TASKS, 1, Epi>)) return false;
  return opt_in_lds((const void*)gemm_dense_kernel<E, 2, 4, DENSE_KH, Epi>) && opt_in_lds((const void*)gemm_dense_kernel<E, 1, 4, DENSE_KH, Epi>) &&
         opt_in_lds((const void*)gemm_dense_kernel<E, 1, 2, DENSE_KH, Epi>);
}

template <typename E> static void launch_qkv_t(bool bf16, const QkvArgs& a, hipStream_t st) {
  const int D = a.geom.n_heads * a.geom.head_dim;
  QkvEpi<E> epi{(E*)a.q, a.q_plane, (E*)a.kv_layer, a.geom, a.meta.tok_seq, a.meta.tok_pos, a.page_table,
                a.pt_stride, a.cos_tab, a.sin_tab, a.norm, a.T, a.H, D};
  if (dense_applies(a.T, a.H / ET<E>::KS))
    launch_dense<E>((const E*)a.w, a.H / ET<E>::KS, (const E*)a.xn, a.T, 3 * D / 64, epi, st);
  else if (!single_slice() && half_applies(bf16, a.H, a.T, 3 * D / 64)) {
    if constexpr (sizeof(E) == 2)
      gemm_half_kernel<E, QkvEpi<E>><<<2 * (3 * D / 64), HALF_KW * WAVE, 0, st>>>((const E*)a.w, a.H / ET<E>::KS, (const E*)a.xn, a.T, epi, live_word());
  } else
    launch_ksplit<E>(bf16, (const E*)a.w, a.H / ET<E>::KS, (const E*)a.xn, a.T, a.H, 3 * D / 64, a.part,
                     a.tickets, epi, st);
}
void launch_qkv(bool bf16, const QkvArgs& a, hipStream_t st) {
  if (bf16) launch_qkv_t<bf16_t>(true, a, st);
  else launch_qkv_t<float>(false, a, st);
}

template <typename E> static void launch_oproj_t(bool bf16, const OprojArgs& a, hipStream_t st) {
  ResidualEpi<E> epi{a.x, a.H, a.gain, (E*)a.xn, a.ssq, a.T, (const E*)a.w_router, a.shares};
  if (dense_applies(a.T, a.D / ET<E>::KS))
    launch_dense<E>((const E*)a.w, a.D / ET<E>::KS, (const E*)a.a, a.T, a.H / 64, epi, st);
  else {
    if constexpr (sizeof(E) == 2) {
      if (a.w_router && a.share_features == 2 * 64) {
        oproj_pair_kernel<E, 4><<<dim3(ksplit_slices(true, a.D, a.T, a.H / 64), a.H / 64), 4 * WAVE, ksplit_lds<1, 4>(), st>>>(
            (const E*)a.w, a.D / ET<E>::KS, (const E*)a.a, a.T, a.part, a.tickets, epi, live_word());
        return;
      }
    }
    launch_ksplit<E>(bf16, (const E*)a.w, a.D / ET<E>::KS, (const E*)a.a, a.T, a.D, a.H / 64, a.part, a.tickets,
                     epi, st);
  }
}
// What the workgroups of the split-K launch stream: workgroup (slice, task) has index task * slices + slice and takes
// the slice's share of the task's k-steps, 2 KB of packed weights each, so region i starts at i * region_bytes.
L2Prefetch oproj_prefetch_plan(bool bf16, const void* w, int D, int H, int T) {
  const int ksteps = D / (bf16 ? 16 : 8), n_tasks = H / 64;
  if (T > 2 * TILE || single_slice()) return L2Prefetch{nullptr, 0, 0};   // more tokens: the dense form
  const int slices = ksplit_slices(bf16, D, T, n_tasks);
  if (ksteps % (slices * 4) != 0) return L2Prefetch{nullptr, 0, 0};       // slices of unequal length
  return L2Prefetch{(const char*)w, (uint32_t)(ksteps / slices) * 2048u, n_tasks * slices};
}
void launch_oproj(bool bf16, const OprojArgs& a, hipStream_t st) {
  if (bf16) launch_oproj_t<bf16_t>(true, a, st);
  else launch_oproj_t<float>(false, a, st);
}

// ------------------------------------------------------------------------------------------------
// Iteration smoothing: delta = probabilities . W_emb, a contraction over the whole vocabulary with few output features
// (32 tasks at hidden 2048), so the launch is filled by cutting the contraction: a workgroup takes SMOOTH_TASKS tasks,
// up to WT token tiles and one K slice, which its two teams of waves halve (as in gemm_dense_kernel), and leaves its
// sums in part[slice][token][feature]; smooth_reduce_kernel adds the slices in order and writes the rows of masked
// positions.  A single slice (many tokens) writes them itself.
// Bound: the stream of the transposed embedding matrix (644 MB at vocabulary 157184; 32 tokens: 149 -> 119 us, 5.4 TB/s).
// The activation fragments of a slice go through LDS once per SMOOTH_TASKS tasks: in the split-K form, where every wave
// fetched its own, they took as many of a compute unit's outstanding requests as the weights (4.3 TB/s), and above
// 64 tokens the unsliced shared-operand form had 24 workgroups at 160 tokens.
// ------------------------------------------------------------------------------------------------
static_assert(SMOOTH_TILE == TILE && SMOOTH_CHUNK == WKC, "smooth_plan counts in these units");
template <typename E, int KID, int WT> constexpr size_t smooth_lds() {
  const size_t stage = SMOOTH_KH * wide_lds<E, KID, WT>();
  const size_t fold = (size_t)(SMOOTH_KH - 1) * SMOOTH_TASKS * 2 * WT * 16 * WAVE * 4;
  return stage > fold ? stage : fold;
}

template <typename E, int WT, int KID>
__global__ __launch_bounds__(SMOOTH_TASKS * SMOOTH_KH * WAVE) void smooth_partial_kernel(const E* __restrict__ W, int ksteps,
                                                                                       const E* __restrict__ B, int T, int H,
                                                                                       int n_slices, int pairs, float* __restrict__ part,
                                                                                       const uint64_t* __restrict__ mask, int block_len,
                                                                                       float* __restrict__ delta,
                                                                                       const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  typedef typename ET<E>::vec vec;
  extern __shared__ __align__(16) char lds_raw[];   // 16-byte aligned: staged fragments move as 128-bit LDS accesses
  constexpr int G = ET<E>::G, KS = ET<E>::KS, NP = Planes<E>::N;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const int team = wave / SMOOTH_TASKS, rank = wave % SMOOTH_TASKS;
  const int n_tasks = H / (2 * TILE), tgroups = (n_tasks + SMOOTH_TASKS - 1) / SMOOTH_TASKS;
  const int tiles = (T + TILE - 1) / TILE, groups = (tiles + WT - 1) / WT, per_group = (tiles + groups - 1) / groups;
  const SmoothItem item = smooth_item(blockIdx.x, groups, tgroups, n_slices);
  if (!item.valid) return;                              // uniform over the workgroup
  const int slice = item.slice, tgroup = item.task_group;
  const int nt = min(per_group, tiles - item.token_group * per_group);
  if (nt <= 0) return;
  const int tok0 = item.token_group * per_group * TILE;
  const int slot = tgroup * SMOOTH_TASKS + rank, task = min(slot, n_tasks - 1);
  // the slice's chunks, the same number for both teams (they share the workgroup's barriers); see smooth_kpad
  const int p0 = (int)((int64_t)pairs * slice / n_slices), p1 = (int)((int64_t)pairs * (slice + 1) / n_slices);
  const int chunks = p1 - p0;
  const int64_t ks0 = ((int64_t)p0 * SMOOTH_KH + (int64_t)team * chunks) * WKC;
  vec* sb = reinterpret_cast<vec*>(lds_raw + team * wide_lds<E, KID, WT>());
  auto row_of = [&](int r) { return min(tok0 + (rank % WT) * TILE + r, T - 1); };
  f32x16 acc0[WT], acc1[WT];
  zero_acc<WT>(acc0);
  zero_acc<WT>(acc1);
  wide_stream<E, WT, SMOOTH_TASKS, KID>(
      W + (int64_t)task * task_stride_elems<E>(ksteps) + ks0 * (2 * WAVE * G), chunks * WKC, B + ks0 * T * (NP * KS), row_of,
      (int64_t)T * (NP * KS), sb, nt, acc0, acc1, rank);
  float* red = reinterpret_cast<float*>(lds_raw);
  float* r = red + (int64_t)rank * (2 * WT * 16) * WAVE + lane;
  __syncthreads();   // the staging areas are done with
  if (team > 0) {
#pragma unroll
    for (int t = 0; t < WT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        r[(t * 32 + v) * WAVE] = acc0[t][v];
        r[(t * 32 + 16 + v) * WAVE] = acc1[t][v];
      }
  }
  __syncthreads();
  if (team > 0 || slot >= n_tasks) return;
#pragma unroll
  for (int t = 0; t < WT; ++t) {
    const int tok = tok0 + t * TILE + col;
    if (t < nt && tok < T) {
      float* out = part + ((int64_t)slice * T + tok) * H + (2 * task) * TILE;
      const bool wanted = n_slices > 1 || ((mask[tok / block_len] >> (tok % block_len)) & 1ull);
      float* row = delta + (int64_t)tok * H + (2 * task) * TILE;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (!wanted) continue;
        f32x4 a, b;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[i] = acc0[t][4 * g + i] + r[(t * 32 + 4 * g + i) * WAVE];
          b[i] = acc1[t][4 * g + i] + r[(t * 32 + 16 + 4 * g + i) * WAVE];
        }
        if (n_slices > 1) {
          *reinterpret_cast<f32x4*>(out + acc_row(4 * g, half)) = a;
          *reinterpret_cast<f32x4*>(out + TILE + acc_row(4 * g, half)) = b;
        } else {           // the caller's buffer: only 4-byte alignment is known
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            row[acc_row(4 * g, half) + i] = a[i];
            row[TILE + acc_row(4 * g, half) + i] = b[i];
          }
        }
      }
    }
  }
}

// delta[t][f] = sum over the slices, in slice order, for the rows of masked positions (the others are left alone).
__global__ __launch_bounds__(256) void smooth_reduce_kernel(const float* __restrict__ part, int n_slices, int T, int H,
                                                             const uint64_t* __restrict__ mask, int block_len,
                                                             float* __restrict__ delta, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4, n = (int64_t)T * H;
  if (i >= n) return;
  const int t = (int)(i / H);
  if (!((mask[t / block_len] >> (t % block_len)) & 1ull)) return;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int k = 0; k < n_slices; ++k) s += *reinterpret_cast<const f32x4*>(part + k * n + i);
#pragma unroll
  for (int q = 0; q < 4; ++q) delta[i + q] = s[q];   // the caller's buffer: only 4-byte alignment is known
}

// The vocabulary in whole multiples of 512 k-steps (zero weights and probabilities past its end): every slice of the
// kernel above gets whole chunks for both of its teams.
int smooth_kpad(bool bf16, int V) {
  const int unit = (bf16 ? 16 : 8) * 512;
  return (V + unit - 1) / unit * unit;
}
template <typename E, int WT, int KID> static void launch_smooth_as(const SmoothArgs& a, int Kpad, const SmoothPlan& p, hipStream_t st) {
  // the partial sums live where the logits were (T * V floats), which the probabilities have replaced, or if these leave
  // too little room in the workspace
  const int slices = single_slice() ? 1 : p.slices, wgs = (p.task_groups * p.token_groups * slices + 7) / 8 * 8;
  float* part = p.in_logits ? a.logits : a.part;
  smooth_partial_kernel<E, WT, KID><<<wgs, SMOOTH_TASKS * SMOOTH_KH * WAVE, smooth_lds<E, KID, WT>(), st>>>(
      (const E*)a.w_emb_t, Kpad / ET<E>::KS, (const E*)a.probs, a.T, a.H, slices, p.pairs, part, a.mask, a.block_len, a.delta, live_word());
  if (slices == 1) return;
  const int64_t quads = (int64_t)a.T * a.H / 4;
  smooth_reduce_kernel<<<(unsigned)((quads + 255) / 256), 256, 0, st>>>(part, slices, a.T, a.H, a.mask, a.block_len, a.delta,
                                                                        live_word());
}
template <typename E> static void launch_smooth_t(const SmoothArgs& a, int Kpad, hipStream_t st) {
  const SmoothPlan p = smooth_plan(a.H, a.V, ET<E>::KS, a.T);
  if (p.wt == 1) launch_smooth_as<E, 1, 23>(a, Kpad, p, st);
  else if (p.wt == 2) launch_smooth_as<E, 2, 23>(a, Kpad, p, st);
  else launch_smooth_as<E, 4, 24>(a, Kpad, p, st);
}
void launch_expected_embedding(bool bf16, const SmoothArgs& a, hipStream_t st) {
  const int Kpad = smooth_kpad(bf16, a.V);
  launch_prob_planes(bf16, a.logits, a.stats, a.T, a.V, Kpad, a.probs, st);
  if (bf16) launch_smooth_t<bf16_t>(a, Kpad, st);
  else launch_smooth_t<float>(a, Kpad, st);
}
template <typename E> static bool configure_smooth() {
  return opt_in_lds((const void*)smooth_partial_kernel<E, 1, 23>) && opt_in_lds((const void*)smooth_partial_kernel<E, 2, 23>) &&
         opt_in_lds((const void*)smooth_partial_kernel<E, 4, 24>);
}

// ------------------------------------------------------------------------------------------------
// Router where the output projection leaves shares of the logits (router_share_features): a wave per token, a lane per expert.  The
// logits are the sum of the shares (in the order of their features), times the row's 1/rms, which comes from the sums of squares of the
// output projection's tasks; then softmax and the k selection rounds (ties to the lower expert id).  No sum between workgroups is left; up to 64
// tokens the pairs are sorted by whoever needs them (PairIds).  Bound by one dependent round trip and the rounds' cross-lane steps.
// Until the output projection left shares, one or two token tiles were contracted with the whole of K here by up to eight workgroups, with
// a hand-off between them, and the last one selected and sorted: with events around the launch 14.0 -> 6.8 us at 32 tokens, 16.1 -> 7.2
// at 64 (hidden 2048, bfloat16), the float32 test model 10.8 -> 6.7; the output projection takes 2.9 and 2.4 longer in bfloat16, 1.1 and 2.7 in
// float32, the expert kernels up to 0.8.
// More tokens (float32): as the router kernel below and the permutation take it 34.0 us at 160 tokens and 35.9 at 512, with this kernel 11.9
// and 12.8 (hidden 2048, the output projection +2.4; hidden 256 14.5 and 15.5 -> 12.0 and 11.4, +2.5), as long as the projection takes its
// forms of one token tile (beyond, shares of 8 KB a token would cost more than the contraction).  Eight tokens a workgroup: with 32, one
// compute unit fetches 256 KB.
// ------------------------------------------------------------------------------------------------
constexpr int SELECT_WAVES = 4;
// HIST (more than 64 tokens): the workgroup leaves its tokens' pairs per expert for the permutation.  PARTS (bfloat16, shares that are
// chains): every sum in the order of the router kernel below, whose waves, workgroups and lanes these are: eight chains to a
// workgroup, sums of squares in PARTS parts (16, or 8 with two token tiles), 64 / PARTS experts to a lane.  0: no order kept.
template <int WAVES, bool HIST, int PARTS>
__global__ __launch_bounds__(WAVES * WAVE) void router_select_kernel(const float* __restrict__ shares, const float* __restrict__ ssq, int n_tasks, int n_shares,
                                                                     float eps, int T, int H, int n_exp, int top_k, int norm_topk,
                                                                     float* __restrict__ rinv, int32_t* __restrict__ topk_idx,
                                                                     float* __restrict__ topk_w, int32_t* __restrict__ hist, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  static_assert(MAX_EXPERTS == WAVE && MAX_HIDDEN / 64 <= WAVE, "a lane per expert, and per task for the sums of squares");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tok = blockIdx.x * WAVES + wave;
  __shared__ int32_t s_cnt[HIST ? MAX_EXPERTS : 1];
  if constexpr (HIST) {
    if (wave == 0) s_cnt[lane] = 0;
    __syncthreads();
  }
  if (tok < T) {                        // uniform over the wave
    constexpr int SS = PARTS ? WAVE / PARTS : 1;
    float ss[SS];
#pragma unroll
    for (int i = 0; i < SS; ++i) {
      const int j = PARTS ? lane % PARTS + PARTS * i : lane;
      ss[i] = j < n_tasks ? ssq[(int64_t)j * T + tok] : 0.f;
    }
    float z = 0.f;
    for (int j0 = 0; j0 < n_shares; j0 += 32) {   // 32 independent loads at a time
      float v[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = shares[((int64_t)min(j0 + i, n_shares - 1) * T + tok) * MAX_EXPERTS + lane];
      if constexpr (PARTS) {                      // (a multiple of eight)
#pragma unroll
        for (int i = 0; i < 32; i += ROUTER_WAVES) {
          float part = 0.f;
#pragma unroll
          for (int k = 0; k < ROUTER_WAVES; ++k) part += v[i + k];
          z += j0 + i < n_shares ? part : 0.f;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 32; ++i) z += j0 + i < n_shares ? v[i] : 0.f;
      }
    }
    float row_ss = 0.f;
    if constexpr (PARTS) {
      float part = ss[0];
#pragma unroll
      for (int i = 1; i < SS; ++i) part += ss[i];
#pragma unroll
      for (int q = 0; q < PARTS; ++q) row_ss += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(part), q));
    } else
      row_ss = wave_all_sum(ss[0]);
    const float r = rsqrtf(row_ss / H + eps);
    const bool on = lane < n_exp;
    z *= r;
    asm("" : "+v"(z));                            // rounded here, not in a sum with the maximum
    z = on ? z : -INFINITY;
    const float m = wave_all_max(z);
    const float ez = on ? expf(z - m) : 0.f;
    float sum;
    if constexpr (PARTS == 16) sum = wave_all_sum_by_fours(ez);
    else if constexpr (PARTS == 8) sum = wave_all_sum_by_eights(ez);
    else sum = wave_all_sum(ez);
    const float inv = 1.f / sum;
    // a row of NaN (fmaxf takes the number) selects the first experts and gets NaN weights: without a selection its expert ids
    // would be no ids, and the expert kernels would index with them
    float p = on ? fmaxf(ez * inv, 0.f) : -1.f;
    float wsel = 0.f, sel_sum = 0.f;    // lane j keeps the j-th selection
    int isel = 0;
    for (int j = 0; j < top_k; ++j) {
      const float best = wave_all_max(p);
      const int e = __builtin_ctzll(__ballot(p == best) | 1ull << 63);
      if (lane == e) p = -1.f;
      if (lane == j) {
        wsel = best;
        isel = e;
      }
      sel_sum += best;
    }
    if (lane < top_k) {
      topk_idx[tok * top_k + lane] = isel;
      topk_w[tok * top_k + lane] = norm_topk ? wsel / sel_sum : wsel;
      if constexpr (HIST) atomicAdd(&s_cnt[isel], 1);
    }
    if (lane == 0) rinv[tok] = r;
  }
  if constexpr (HIST) {
    __syncthreads();
    if (wave == 0) hist[blockIdx.x * MAX_EXPERTS + lane] = s_cnt[lane];
  }
}

// ------------------------------------------------------------------------------------------------
// Router without shares.  The single weight task holds experts 0-31 (tile 0) and 32-63 (tile 1); a workgroup takes a token
// tile, its KW waves the K range, and the partial tiles meet in LDS.  It turns the sums into logits[token][expert] (times the
// row's 1/rms, which it derives from the per-task sums of squares the output projection left), then groups of 16 or 8 lanes take one
// token each through softmax and the k selection rounds (ties to the lower expert id).
// ------------------------------------------------------------------------------------------------
// L (8 or 16) lanes form a group; every lane ends with the same bits (each step combines the same two values on both sides).
template <int L> __device__ inline float group_max(float v) {
  v = fmaxf(v, dpp_f<DPP_SWAP1>(v));
  v = fmaxf(v, dpp_f<DPP_SWAP2>(v));
  v = fmaxf(v, dpp_f<DPP_HALF_MIRROR>(v));
  return L == 16 ? fmaxf(v, dpp_f<DPP_MIRROR>(v)) : v;
}
template <int L> __device__ inline float group_sum(float v) {
  v += dpp_f<DPP_SWAP1>(v);
  v += dpp_f<DPP_SWAP2>(v);
  v += dpp_f<DPP_HALF_MIRROR>(v);
  return L == 16 ? v + dpp_f<DPP_MIRROR>(v) : v;
}
template <int L> __device__ inline int group_min(int v) {
  v = min(v, dpp_i<DPP_SWAP1>(v));
  v = min(v, dpp_i<DPP_SWAP2>(v));
  v = min(v, dpp_i<DPP_HALF_MIRROR>(v));
  return L == 16 ? min(v, dpp_i<DPP_MIRROR>(v)) : v;
}
// Largest value of the group and the lowest id that holds it: the largest value first, then the lowest id among
// the lanes whose own best equals it (two plain butterflies instead of one with a compound comparison).
template <int L> __device__ inline void group_argmax(float& bv, int& bi) {
  const float mx = group_max<L>(bv);
  bi = group_min<L>(bv == mx ? bi : 0x7fffffff);
  bv = mx;
}

// TT: one token tile per workgroup, or two (33 to 64 tokens).
template <typename E, int TT, int KW>
__global__ __launch_bounds__(KW * WAVE) void router_kernel(const E* __restrict__ W, const E* __restrict__ xn,
                                                            const float* __restrict__ ssq, int n_ssq,
                                                            float eps, int T, int H, int n_exp, int top_k, int norm_topk,
                                                            float* __restrict__ rinv, int32_t* __restrict__ topk_idx,
                                                            float* __restrict__ topk_w, int32_t* __restrict__ hist, const int32_t* __restrict__ live) {
  if (step_is_dead(live)) return;
  extern __shared__ float red[];   // [KW][2*TT*16][64] partials
  constexpr int ROWS = 2 * TT * 16, NTOK = TT * TILE, NTHREADS = KW * WAVE, PER = 16 / KW;
  constexpr int SS_PARTS = NTHREADS / NTOK;                       // threads per token for the sums of squares
  constexpr int SS_PER = (MAX_HIDDEN / 64 + SS_PARTS - 1) / SS_PARTS;
  constexpr int LOGIT_STRIDE = MAX_EXPERTS + 1;   // padded: the transposed writes spread over the banks
  __shared__ float s_logit[NTOK * LOGIT_STRIDE];
  __shared__ float s_ssp[SS_PARTS * NTOK];
  __shared__ float s_rinv[NTOK];
  __shared__ int32_t s_cnt[MAX_EXPERTS];                     // pairs per expert
  const int group = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane >> 5;
  const int tok0 = group * NTOK;
  const int ksteps = H / ET<E>::KS;
  TRACE_MARK(3, 0);
  // shares of the rows' sums of squares (one per 64-feature task of the producer), loaded before the stream
  float ssv[SS_PER];
  {
    const int tok = min(tok0 + (int)threadIdx.x % NTOK, T - 1), part0 = threadIdx.x / NTOK;
#pragma unroll
    for (int i = 0; i < SS_PER; ++i) {
      const int j = part0 + i * SS_PARTS;
      ssv[i] = j < n_ssq ? ssq[(int64_t)j * T + tok] : 0.f;
    }
  }
  f32x16 acc0[TT], acc1[TT];
  zero_acc<TT>(acc0);
  zero_acc<TT>(acc1);
  PlaneLoader<E, TT> ld;
#pragma unroll
  for (int t = 0; t < TT; ++t) ld.set(t, xn, T, min(tok0 + t * TILE + (lane & 31), T - 1), half);
  const int per = (ksteps + KW - 1) / KW;
  const int ks0 = min(ksteps, wave * per), ks1 = min(ksteps, ks0 + per);
  stream_task<E, TT, (TT == 1 ? 8 : 4), false>(W, ks0, ks1, ld, acc0, acc1);
  TRACE_MARK(3, 1);
  spill_partials<TT, ROWS>(red, wave, lane, acc0, acc1);
  {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < SS_PER; ++i) s += ssv[i];
    s_ssp[threadIdx.x] = s;     // [part][token]
  }
  __syncthreads();
  TRACE_MARK(3, 2);
  const int v0 = wave * PER;
  float a0[TT][PER], a1[TT][PER];
  fold_partials<TT, KW, PER>(red, lane, v0, a0, a1);
  if (threadIdx.x < MAX_EXPERTS) s_cnt[threadIdx.x] = 0;
  if (threadIdx.x < NTOK) {
    float row_ss = 0.f;
    for (int q = 0; q < SS_PARTS; ++q) row_ss += s_ssp[q * NTOK + threadIdx.x];
    const float r = rsqrtf(row_ss / H + eps);
    s_rinv[threadIdx.x] = r;
    if (tok0 + (int)threadIdx.x < T) rinv[tok0 + threadIdx.x] = r;
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const int tl = t * TILE + (lane & 31);
    const float r = s_rinv[tl];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      s_logit[tl * LOGIT_STRIDE + acc_row(v0 + i, half)] = a0[t][i] * r;
      s_logit[tl * LOGIT_STRIDE + TILE + acc_row(v0 + i, half)] = a1[t][i] * r;
    }
  }
  __syncthreads();
  TRACE_MARK(3, 3);
  // 16 lanes per token with 4 consecutive experts each; with 64 tokens 8 lanes and 8 experts
  constexpr int LPT = NTHREADS / NTOK, EPL = MAX_EXPERTS / LPT;
  static_assert((LPT == 16 || LPT == 8) && LPT >= MAX_TOPK, "lane j keeps the j-th selection");
  const int grp = threadIdx.x / LPT, sub = threadIdx.x % LPT;
  for (int tl = grp; tl < NTOK; tl += NTHREADS / LPT) {
    float p[EPL];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      p[i] = EPL * sub + i < n_exp ? s_logit[tl * LOGIT_STRIDE + EPL * sub + i] : -INFINITY;
      m = fmaxf(m, p[i]);
    }
    m = group_max<LPT>(m);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      p[i] = EPL * sub + i < n_exp ? expf(p[i] - m) : 0.f;
      sum += p[i];
    }
    const float inv = 1.f / group_sum<LPT>(sum);
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      // a row of NaN (fmaxf takes the number) selects the first experts and gets NaN weights: without a selection its
      // expert ids would be no ids, and the permutation would index with them
      p[i] = EPL * sub + i < n_exp ? fmaxf(p[i] * inv, 0.f) : -1.f;
    }
    float wsel = 0.f, sel_sum = 0.f;   // lane j of the group keeps the j-th selection
    int isel = 0;
    for (int j = 0; j < top_k; ++j) {
      float bv = -1.f;
      int bi = 0x7fffffff;
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (p[i] > bv) {               // ids ascend with i: strict '>' keeps the lowest id
          bv = p[i];
          bi = EPL * sub + i;
        }
      group_argmax<LPT>(bv, bi);
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        if (EPL * sub + i == bi) p[i] = -1.f;
      if (sub == j) {
        wsel = bv;
        isel = bi;
      }
      sel_sum += bv;
    }
    if (sub < top_k && tok0 + tl < T) {
      const int tok = tok0 + tl;
      topk_idx[tok * top_k + sub] = isel;
      topk_w[tok * top_k + sub] = norm_topk ? wsel / sel_sum : wsel;
      atomicAdd(&s_cnt[isel], 1);
    }
  }
  TRACE_MARK(3, 4);
  __syncthreads();
  if (threadIdx.x < MAX_EXPERTS) hist[group * MAX_EXPERTS + threadIdx.x] = s_cnt[threadIdx.x];   // for the permutation
  TRACE_MARK(3, 5);
}

template <typename E> static void launch_router_t(const RouterArgs& a, hipStream_t st) {
  auto select = [&](auto kernel, int waves) {
    kernel<<<(a.T + waves - 1) / waves, waves * WAVE, 0, st>>>(a.shares, a.ssq, a.H / 64, a.H / a.share_features, a.eps, a.T, a.H, a.E, a.top_k, a.norm_topk,
                                                               a.rinv, a.topk_idx, a.topk_w, a.hist, live_word());
  };
  const bool few = a.T <= 2 * TILE;   // the expert kernels sort the pairs
  auto contract = [&](auto kernel, int tiles, size_t lds) {
    kernel<<<(a.T + tiles * TILE - 1) / (tiles * TILE), ROUTER_WAVES * WAVE, lds, st>>>((const E*)a.w, (const E*)a.xn, a.ssq, a.H / 64, a.eps, a.T, a.H, a.E,
                                                                                        a.top_k, a.norm_topk, a.rinv, a.topk_idx, a.topk_w, a.hist, live_word());
  };
  constexpr bool CHAINS = sizeof(E) == 2;
  if (!a.share_features) {
    if (few && a.T > TILE) contract(router_kernel<E, 2, ROUTER_WAVES>, 2, ksplit_lds<2, ROUTER_WAVES>());
    else contract(router_kernel<E, 1, ROUTER_WAVES>, 1, ksplit_lds<1, ROUTER_WAVES>());
  } else if (CHAINS && a.T <= TILE) select(router_select_kernel<SELECT_WAVES, false, CHAINS ? 16 : 0>, SELECT_WAVES);
  else if (few) select(router_select_kernel<SELECT_WAVES, false, CHAINS ? 8 : 0>, SELECT_WAVES);
  else select(router_select_kernel<HIST_TOKENS, true, 0>, HIST_TOKENS);
  if (few) return;
  launch_permute(a.topk_idx, a.T * a.top_k, a.top_k, a.hist, a.share_features ? HIST_TOKENS : TILE, a.E, a.cnt, a.off, a.perm, a.work,
                 expert_group_tiles(a.E, a.T * a.top_k), expert_round_items(a.E, a.T * a.top_k, a.H, a.I), st);
}
void launch_router(bool bf16, const RouterArgs& a, hipStream_t st) {
  if (bf16) launch_router_t<bf16_t>(a, st);
  else launch_router_t<float>(a, st);
}

// Fused down projection: DOWN_SLICES workgroups of DOWN_KW waves share a task's long K.
constexpr int DOWN_SLICES = 8, DOWN_KW = 8;
int down_fused_slices() { return DOWN_SLICES; }
template <typename E> static void launch_down_fused_t(const ExpertArgs& a, const OprojArgs& r, hipStream_t st) {
  ResidualEpi<E> epi{r.x, r.H, r.gain, (E*)r.xn, r.ssq, r.T, nullptr, nullptr};
  const int n_tasks = a.H / 64, ksteps_e = a.I / ET<E>::KS;
  const dim3 grid(DOWN_SLICES, n_tasks);
  const E *w = (const E*)a.w_down, *y = (const E*)a.y;
  const int64_t y_rows = (int64_t)a.T * a.top_k;
  if (ksteps_e % 8 == 0)
    expert_down_fused_kernel<E, 1, DOWN_KW, 8><<<grid, DOWN_KW * WAVE, ksplit_lds<1, DOWN_KW>(), st>>>(
        w, y, y_rows, a.topk_idx, a.T, a.I, a.top_k, n_tasks, r.part, r.tickets, epi, live_word());
  else
    expert_down_fused_kernel<E, 1, DOWN_KW, 4><<<grid, DOWN_KW * WAVE, ksplit_lds<1, DOWN_KW>(), st>>>(
        w, y, y_rows, a.topk_idx, a.T, a.I, a.top_k, n_tasks, r.part, r.tickets, epi, live_word());
}
void launch_expert_down_fused(bool bf16, const ExpertArgs& a, const OprojArgs& res, hipStream_t st) {
  if (bf16) launch_down_fused_t<bf16_t>(a, res, st);
  else launch_down_fused_t<float>(a, res, st);
}

// The routed-expert GEMMs and the LM head live in wide.hip (shared-operand forms for every token count).
void launch_expert_gate_up(bool bf16, const ExpertArgs& a, hipStream_t st) { launch_expert_gate_up_wide(bf16, a, st); }
void launch_expert_down(bool bf16, const ExpertArgs& a, hipStream_t st) { launch_expert_down_wide(bf16, a, st); }
void launch_lm_head(bool bf16, const LmArgs& a, hipStream_t st) { launch_lm_head_wide(bf16, a, st); }

bool configure_kernels() {
  bool ok = configure_ksplit<bf16_t, QkvEpi<bf16_t>>() && configure_ksplit<float, QkvEpi<float>>() &&
            configure_ksplit<bf16_t, ResidualEpi<bf16_t>>() && configure_ksplit<float, ResidualEpi<float>>() &&
            configure_smooth<bf16_t>() && configure_smooth<float>();
  ok = ok && configure_dense<bf16_t, QkvEpi<bf16_t>>() && configure_dense<float, QkvEpi<float>>() &&
       configure_dense<bf16_t, ResidualEpi<bf16_t>>() && configure_dense<float, ResidualEpi<float>>();
  ok = ok && opt_in_lds((const void*)expert_down_fused_kernel<bf16_t, 1, DOWN_KW, 8>) &&
       opt_in_lds((const void*)expert_down_fused_kernel<bf16_t, 1, DOWN_KW, 4>) &&
       opt_in_lds((const void*)expert_down_fused_kernel<float, 1, DOWN_KW, 8>) &&
       opt_in_lds((const void*)expert_down_fused_kernel<float, 1, DOWN_KW, 4>);
  ok = ok && opt_in_lds((const void*)router_kernel<bf16_t, 1, ROUTER_WAVES>) && opt_in_lds((const void*)router_kernel<float, 1, ROUTER_WAVES>) &&
       opt_in_lds((const void*)router_kernel<bf16_t, 2, ROUTER_WAVES>) && opt_in_lds((const void*)router_kernel<float, 2, ROUTER_WAVES>);
  (void)hipGetLastError();
  return ok;
}

TRACE_READER(trace_read_gemm)

}  // namespace dinfer
