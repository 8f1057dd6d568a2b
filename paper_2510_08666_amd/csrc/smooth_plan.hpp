// How the expected-embedding contraction of iteration smoothing is cut into workgroups.  Host C++, and device code where a
// function says so.
#pragma once
#include <stddef.h>

#include "host_device.hpp"

namespace dinfer {

// A workgroup takes SMOOTH_TASKS tasks (64 output features each), one group of token tiles and one K slice, which
// SMOOTH_KH teams of waves halve; a slice is a whole number of pairs of chunks.
constexpr int SMOOTH_TASKS = 4, SMOOTH_KH = 2, SMOOTH_WGS = 256, SMOOTH_TILE = 32, SMOOTH_CHUNK = 4;
// Pairs of chunks a slice has at least: one leaves more partial sums than it saves, eight leave compute units idle
// (float32, hidden 256, 4096 ids, a step of 32 / 512 tokens: 102.1 / 332 us with one, 101.7 / 338 with two, 107.6 / 355
// with four, 115.6 / 382 with eight; bf16 hidden 1024, 5000 ids, 64 tokens: 112.4, 108.3, 109.6, 114.4).
constexpr int SMOOTH_MIN_PAIRS = 2;

struct SmoothPlan {
  int wt;             // token tiles per workgroup, at most: 1, 2 or 4
  int task_groups, token_groups;
  int pairs;          // pairs of chunks that hold ids of the vocabulary (what it is padded to beyond them is zeros)
  int slices;         // 1: the workgroups write the rows themselves
  bool in_logits;     // the partial sums [slices][T][H] fit where the logits [T][V] were
};
// ks: features of a k-step.  The vocabulary is stored padded (smooth_kpad) and contracted as far as it goes: 497 ids padded
// to 8192, 2240 tokens at hidden 1216, took 500 us a step, 353 without the padding.
// About one workgroup per compute unit (two waves on every SIMD); a multiple of eight slices keeps a slice on one die.
// The number of slices does not follow the room the logits leave: limited to that, 32000 ids at hidden 2048 had eight
// slices, 64 workgroups (a bf16 step of 32 tokens 167 us, 144 with 32 slices; float32 354 and 254).
inline SmoothPlan smooth_plan(int H, int V, int ks, int T) {
  SmoothPlan p;
  const int tiles = (T + SMOOTH_TILE - 1) / SMOOTH_TILE;
  p.wt = tiles <= 2 ? tiles : 4;
  p.task_groups = (H / 64 + SMOOTH_TASKS - 1) / SMOOTH_TASKS;
  p.token_groups = (tiles + p.wt - 1) / p.wt;
  const int pair = ks * SMOOTH_CHUNK * SMOOTH_KH;
  p.pairs = (V + pair - 1) / pair;
  int s = SMOOTH_WGS / (p.task_groups * p.token_groups);
  const int most = p.pairs / SMOOTH_MIN_PAIRS;
  s = s < most ? s : most;
  p.slices = s < 1 ? 1 : s >= 8 ? s / 8 * 8 : s;
  p.in_logits = p.slices <= V / H;
  return p;
}
// Bytes for the partial sums of any forward of up to max_tokens tokens whose logits leave too little room (a vocabulary
// of few rows of features: 0 at 157184 ids and hidden 2048, 8 MB at 32000).
inline size_t smooth_part_bytes(int H, int V, int ks, int max_tokens) {
  size_t most = 0;
  for (int t = SMOOTH_TILE; t < max_tokens + SMOOTH_TILE; t += SMOOTH_TILE) {
    const int T = t < max_tokens ? t : max_tokens;
    const SmoothPlan p = smooth_plan(H, V, ks, T);
    const size_t bytes = p.slices > 1 && !p.in_logits ? (size_t)p.slices * T * H * 4 : 0;
    most = bytes > most ? bytes : most;
  }
  return most;
}

// Workgroup i = die (i % 8), turn (i / 8).  Up to 128 tokens the slices vary fastest over the dies, so that a die's task
// groups share the probabilities of its slices.  With several token groups a die takes an eighth of the list [slice][task
// group][token group] in its order: the token groups of one (slice, task group) are consecutive turns and share its
// weights in the L2, and no die has more than one workgroup more than another (whole (slice, task group) units dealt out
// to the dies in turn: 20 of them with 12 token groups each, hidden 2368 and 1536 tokens, put 36 workgroups on the 32
// compute units of four dies; with 25022 ids the step took 1400 us, now 1010).
struct SmoothItem {
  int token_group, task_group, slice;
  bool valid;
};
DINFER_HOST_DEVICE inline SmoothItem smooth_item(int i, int token_groups, int task_groups, int slices) {
  const int total = token_groups * task_groups * slices, per_die = (total + 7) / 8;
  if (token_groups == 1) return SmoothItem{0, i / slices, i % slices, i < total};
  const int at = (i % 8) * per_die + i / 8;
  return SmoothItem{at % token_groups, at / token_groups % task_groups, at / (token_groups * task_groups), at < total};
}

}  // namespace dinfer
