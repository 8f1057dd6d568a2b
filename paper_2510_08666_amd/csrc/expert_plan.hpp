// How the routed rows of more than 64 tokens are dealt out to the expert GEMMs.  Host C++, and device code where a function
// says so.
#pragma once

#include "host_device.hpp"

namespace dinfer {

constexpr int EXPERT_TILE = 32;   // rows of a token tile
constexpr int EXPERT_DIES = 8;     // workgroup i of a launch runs on die i % 8
constexpr int EXPERT_CUS = 256;   // compute units; eight waves of these kernels fill one
// An item is a run of an expert's sorted rows, up to expert_group_tiles tiles; a workgroup takes it with EXPERT_WW tasks (one
// per wave) and four tiles, or, up to MID_ROWS rows per expert on average, with MID_WW tasks and two tiles, so that two
// workgroups share a compute unit.  With eight tasks an expert is four workgroups of a whole compute unit each, and a step
// whose masked rows touch half of the experts leaves half of the chip idle (gate/up + down in microseconds at 96 / 128 /
// 160 tokens of a fully masked block batch: 73 + 46, 91 + 55, 89 + 53 with eight tasks, 45 + 31, 71 + 44, 72 + 46 with
// four; where all 64 experts have rows, 92 + 52 against 87 + 52 at 96 tokens and 98 + 59 against 95 + 59 at 160).  Beyond,
// the rows weigh more than the balance: every workgroup fetches its expert's rows for itself (256 tokens: 102 + 64 with
// eight tasks, 120 + 73 with four).
constexpr int EXPERT_WW = 8, EXPERT_WT = 4;
constexpr int MID_WW = 4, MID_WT = 2, MID_ROWS = 24;

inline int expert_group_tiles(int E, int n_pairs) { return n_pairs <= MID_ROWS * E ? MID_WT : EXPERT_WT; }
// Items that the groups can add up to for n_pairs routed pairs.
inline int expert_work_items(int E, int n_pairs, int group_tiles) { return E + n_pairs / (group_tiles * EXPERT_TILE); }
// Items whose workgroups fill the chip once: a round.
inline int expert_round_items(int E, int n_pairs, int H, int I) {
  const int ww = expert_group_tiles(E, n_pairs) == MID_WT ? MID_WW : EXPERT_WW, slots = EXPERT_CUS * (EXPERT_WW / ww);
  const int up = (I / 32 + ww - 1) / ww, down = (H / 64 + ww - 1) / ww, most = up > down ? up : down;
  return most < slots ? slots / most : 1;
}
// Of `items` items, sorted by weight, of which the last `light` have one or two tiles: those at the end that would begin
// another, mostly empty round of the chip.  They are handed out task by task instead (pieces), if they are light and few:
// at most three eighths of a round (one layer, 16 experts of width 4096, items beyond a round of 16: 4 of them 428 -> 421
// us, 7 of them 622 -> 628).
constexpr int PIECES_NUM = 3, PIECES_DEN = 8;
DINFER_HOST_DEVICE inline int expert_piece_items(int items, int light, int round) {
  const int over = items > round ? items % round : 0;
  return over <= light && over <= round * PIECES_NUM / PIECES_DEN ? over : 0;
}
// The most of them any routing of n_pairs pairs can give (grid sizing).
inline int expert_most_piece_items(int E, int n_pairs, int H, int I) {
  const int round = expert_round_items(E, n_pairs, H, I), few = round * PIECES_NUM / PIECES_DEN;
  const int beyond = expert_work_items(E, n_pairs, expert_group_tiles(E, n_pairs)) - round;
  return beyond <= 0 ? 0 : beyond < few ? beyond : few;
}

// From two full items per expert on average (prompts), the items of an expert run on one die, and each with its task groups
// one after the other, so that the expert's weights and the item's rows come to that die's L2 once: the work list is dealt out
// over the dies (item i to die i % 8), its full items lie EXPERT_DIES places apart, and the weights are loaded as ordinary
// lines (non-temporal ones do not stay in the L2: 32 workgroups of a die that read 16 MB side by side get 11 to 14 TB/s over
// all dies, with ordinary loads 23 to 33).  4287 tokens, about five items per expert: L2 misses of gate/up + down 20.8 + 12.7 ->
// 13.0 + 7.5 million lines, 546 + 319 -> 535 + 299 us.  With fewer items nothing is shared, and ordinary loads only push
// other data out of the caches (gate/up at 160 tokens 93 -> 103 us).
inline bool expert_shared(int E, int n_pairs) { return n_pairs >= 2 * EXPERT_WT * EXPERT_TILE * E; }
inline int expert_item_stride(int E, int n_pairs) { return expert_shared(E, n_pairs) ? EXPERT_DIES : 1; }
// Place of item i of n: items 0, 1, ... take the places 0, stride, 2 * stride, ... below n, then 1, 1 + stride, ...
DINFER_HOST_DEVICE inline int expert_item_place(int i, int n, int stride) {
  const int q = n / stride, r = n % stride, front = r * (q + 1);   // r classes of q + 1 places, then classes of q
  return i < front ? i % (q + 1) * stride + i / (q + 1) : (i - front) % (q > 0 ? q : 1) * stride + r + (i - front) / (q > 0 ? q : 1);
}
// The place behind place p.
DINFER_HOST_DEVICE inline int expert_next_place(int p, int n, int stride) { return p + stride < n ? p + stride : p % stride + 1; }

}  // namespace dinfer
