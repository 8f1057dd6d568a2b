// How the routed rows of more than 64 tokens are dealt out to the expert GEMMs.  Host C++, and device code where a function
// says so.
#pragma once

#include "host_device.hpp"

namespace dinfer {

constexpr int EXPERT_TILE = 32;   // rows of a token tile
constexpr int EXPERT_DIES = 8;    // workgroup i of a launch runs on die i % 8
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

// From two full items per expert on average (prompts), the shared form: an item's task groups run on one die one after the other,
// then its expert's other items, so that the expert's weights and the item's rows come to that die's L2 once, and the weights
// are loaded as ordinary lines (non-temporal ones do not stay in the L2: 32 workgroups of a die that read 16 MB side by side get
// 11 to 14 TB/s over all dies, with ordinary loads 23 to 33).  64 experts of width 1024, hidden 2048, bf16, plain -> shared: 4287
// tokens gate/up + down 544 + 323 -> 523 + 294 us (L2 misses 20.8 + 12.7 -> 13.0 + 7.5 million lines), 2048 tokens (the line) 311 +
// 185 -> 290 + 162; float32, 8 experts of width 1408 at the line 506 + 350 -> 480 + 332.  Below the line these two launches
// gain as well, but ordinary loads push other data out of the caches, and a whole layer gains or loses with the model (1500 tokens:
// 64 experts of width 1024 453 -> 446, 32 of 768 at hidden 4096 424 -> 432; 1100 tokens 376 -> 379).
// bf16 with 32 groups or more, a multiple of the dies: an item alone fills its die, so nothing runs beside it that could share its
// weights, while in plain order every item's group g runs on die g % 8 (four experts of width 8192, 32 groups, 3000 tokens: 359 us
// plain, 363 shared and a layer 807 -> 823; two experts of width 14336, 1500 tokens: 616 and 626).
inline bool expert_shared(bool bf16, int E, int n_pairs, int groups) {
  return n_pairs >= 2 * EXPERT_WT * EXPERT_TILE * E && !(bf16 && groups >= EXPERT_CUS / EXPERT_DIES && groups % EXPERT_DIES == 0);
}
// Which item and task group workgroup wg of the shared form takes.  The list's items lie by weight: `heavy` of four tiles (an
// expert's one behind the other), then to `full` those of three, then the light ones.  Each kind's (item, task group) pairs go to
// the dies in equal runs, so that every die has its share of the work within a workgroup, the heavy ones first.  Items dealt
// whole, i to die i % 8, left some dies a round more than the others (8 experts of width 2816, gate/up of 1200 tokens, 23 or 24
// items of 11 groups: 126 us in plain order, 156 with whole items, 109 with equal runs), and items dealt in one run a die some
// dies without any lighter item (float32, 16 experts of width 2816, 3000 tokens: 675, 748, 639).
struct ExpertUnit {
  int item, group;   // item -1: nothing to do
};
DINFER_HOST_DEVICE inline int expert_unit_wgs(int n, int groups) { return (n * groups + EXPERT_DIES - 1) / EXPERT_DIES * EXPERT_DIES; }
DINFER_HOST_DEVICE inline ExpertUnit expert_unit(int wg, int heavy, int full, int n, int groups) {
  const int ends[3] = {heavy < n ? heavy : n, full < n ? full : n, n};
  int turn = wg / EXPERT_DIES, start = 0, dealt = 0;   // turn of the die; items of the kinds before; runs with a pair more so far
  for (int k = 0; k < 3; ++k) {
    const int pairs = (ends[k] - start) * groups, each = pairs / EXPERT_DIES, more = pairs % EXPERT_DIES;
    const int run = (wg - dealt) & (EXPERT_DIES - 1);  // the first `more` runs have a pair more, from where the last kind's ended
    if (turn < each + (run < more ? 1 : 0)) {
      const int pair = run * each + (run < more ? run : more) + turn;
      return ExpertUnit{start + pair / groups, pair % groups};
    }
    turn -= each + (run < more ? 1 : 0);
    start = ends[k];
    dealt = (dealt + more) & (EXPERT_DIES - 1);
  }
  return ExpertUnit{-1, 0};
}

}  // namespace dinfer
