// How the LM head deals the vocabulary out to workgroups, and with it how many softmax partials it leaves per token row.
// Plain host C++: the launcher, the kernel (as an argument) and the merge behind it all take the numbers from here.
#pragma once

namespace dinfer {

constexpr int LM_TASK_IDS = 64;                 // vocabulary ids of a task
constexpr int LM_CUS = 256;                     // compute units
// Tasks per workgroup (one per wave).  Up to 32 tokens all workgroups are resident at once and the dispatcher deals them
// evenly, so a launch lasts as long as the compute units with one workgroup more than the others: 614 workgroups of
// four tasks put 3 MB on some units and 2 MB on others (112 us), 1228 of two tasks 2.5 or 2 MB (108 us).  Above 64 tokens
// eight waves share the activation fragments of 128 rows (four in the LM head at 512 tokens: 450 us against 352).
constexpr int LM_SMALL_WW = 2, LM_MID_WW = 4;   // up to 32, up to 64 tokens
constexpr int LM_WW = 8;                        // more tokens
constexpr int LM_PIECE_WW = 8;                  // waves per task of a small vocabulary
constexpr int LM_SMALL_T = 32, LM_MID_T = 64;

// Workgroups 0 .. whole-1 take ww consecutive tasks each (the last one possibly fewer), together the tasks in front of
// first_piece; every task from there on has a workgroup of its own, which cuts the K range over its waves.
struct LmPlan {
  int tasks;          // of the vocabulary
  int ww;             // tasks per whole group, or waves per task where all are pieces
  int whole;          // whole groups
  int first_piece;    // = tasks where there are no pieces
  int parts;          // partials per token row: one per workgroup up to LM_MID_T tokens, one per wave above
};
//  - Few tasks (one per compute unit or less): all in pieces, since a wave alone with a task is bound by its chain of
//    loads and matrix instructions (4096 ids of float32, hidden 256: 16.5 -> 11 us at 32 tokens, 27 -> 13.4 at 64).
//  - 33 to 64 tokens: two workgroups of four waves fill a compute unit, so the groups beyond 512 would begin a second
//    round of the chip; they go out in pieces where these are at most a fifth of a round.  A piece fetches the activation
//    rows for itself, so that more of them cost as much as the round would (one layer and LM head in bf16 at hidden 2048,
//    35 / 64 tokens, whole groups -> pieces: 2 groups beyond 192 / 198 -> 177 / 186 us, 102 of them 202 / 202 -> 196 / 202,
//    150 of them 198 / 204 -> 204 / 221, 220 of them 207 / 214 -> 219 / 238; 157184 ids are 102 beyond).
//  - Up to 32 tokens: three waves per SIMD (168 registers) hold all workgroups of 157184 ids at once (114 -> 108 us
//    against two per SIMD, where 1024 of 1228 fit).  More than 64 tokens: whole groups.
inline LmPlan lm_plan(int V, int T) {
  LmPlan p;
  p.tasks = (V + LM_TASK_IDS - 1) / LM_TASK_IDS;
  const bool few = T <= LM_MID_T && p.tasks <= LM_CUS;
  p.ww = few ? LM_PIECE_WW : T <= LM_SMALL_T ? LM_SMALL_WW : T <= LM_MID_T ? LM_MID_WW : LM_WW;
  p.whole = few ? 0 : (p.tasks + p.ww - 1) / p.ww;
  const int round = LM_CUS * (8 / LM_MID_WW), over = p.whole % round;
  if (p.ww == LM_MID_WW && p.whole > round && 5 * over <= round) p.whole -= over;
  p.first_piece = p.whole * p.ww < p.tasks ? p.whole * p.ww : p.tasks;
  p.parts = T <= LM_MID_T ? p.whole + p.tasks - p.first_piece : p.whole * p.ww;
  return p;
}
// Above LM_MID_T tokens the LM head multiplies the high plane of bf16 activations only, and reads it as a matrix of its own ([K
// step][row][16]): out of the interleaved planes every fetched cache line is half of no use (512 / 160 tokens 315 -> 308 / 187 ->
// 175 us).  The last combine of a forward with a head writes it (+0.3 us at 512 tokens; a prompt of 4287 tokens, which has no
// head, would store 17.6 MB for nothing).
inline bool lm_compact(bool bf16, int T) { return bf16 && T > LM_MID_T; }
// bf16 rows of 129 to 192 and of 289 to 320 tokens: half a task per wave, so that five or six token tiles fit a workgroup's
// registers and the vocabulary's weights go to one workgroup where four tiles at most (or two, beyond 256 tokens, where they are three)
// would take two of them.  While all compute units stream, each takes in about 27 GB/s, from its L2 as well, and at 160 tokens
// two thirds of that was the second delivery.  LM head in us, four tiles and whole tasks -> this: 130 tokens 163 -> 137, 160 168 -> 142,
// 192 172 -> 150, 288 219 -> 214 (the call is no faster), 320 223 -> 212, 352 230 -> 234, 384 238 -> 238, 480 286 -> 322, 512 288 -> 317 (with
// eight tiles in a workgroup: every fragment read from LDS feeds one matrix instruction instead of two, and LDS is the bound).
// The call's tokens choose, not its undecided ones, which only the device knows; the kernel deals the tiles of the list.  Lists that need no
// second delivery either way gain too, since the head's last round of workgroups is shorter: of 160 tokens 16 undecided 135 -> 123, 97 to 128
// 145 -> 133, 129 170 -> 140; of 320 tokens 97 149 -> 140, 128 150 -> 144, 160 183 -> 154, 192 185 -> 158, 193 to 256 184 to 188 -> 183 to 185, 257
// 222 -> 211, all 223 -> 207 (events around the stage; 1 to 2 us more since the two halves' statistics are those of a whole task).
inline bool lm_half(bool bf16, int T) {
  const int tiles = (T + 31) / 32;
  return bf16 && (tiles == 5 || tiles == 6 || tiles == 10);
}
// Upper bound of the partials per token row, whatever the token count (workspace sizing): one per task, rounded up.
inline int lm_head_most_parts(int V) { return ((V + LM_TASK_IDS - 1) / LM_TASK_IDS + LM_WW - 1) / LM_WW * LM_WW; }
inline int lm_head_parts(int V, int T) { return lm_plan(V, T).parts; }

}  // namespace dinfer
