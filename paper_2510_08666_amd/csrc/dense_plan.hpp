// Which form the dense projections (QKV and output) take.  Plain host C++.
#pragma once

namespace dinfer {

constexpr int DENSE_TILE = 32;    // token rows of a tile
constexpr int DENSE_CUS = 256;    // compute units: a workgroup fills one
constexpr int DENSE_FILL = 140;   // workgroups a launch of four tasks and one tile each must keep

struct DenseForm {
  int tasks, tiles;               // per workgroup: 4 and 2, 4 and 1, 2 and 1, 8 and up to 4
  int groups;                     // token groups, which share the tiles evenly
};
// bf16: one round of the chip takes 41 us (QKV of the 2048-wide model, four tasks and two tiles), 25 (four tasks, one tile)
// or 20 (two tasks, one tile): four tasks and one tile while their workgroups are one round (352 tokens: 264 of them, two
// rounds, 46 us; with two tiles 39; output projection at 1100 tokens 46 and 38), two tasks where four would leave nearly
// half the chip idle (192 tokens: 288 workgroups of two tasks, two rounds, 28 us; 144 of four, 26.7).
// float32: the matrix instructions bound a workgroup, so that one with two tiles takes twice as long as one with one, and
// a few workgroups beyond a round cost no more than two tiles each (hidden 1024, QKV: 704 tokens 80.6 us with one tile,
// 264 workgroups, 87.8 with two; 256 tokens of 3072 features 81.4 and 89.2): two tiles from 160 workgroups of them on.
// bf16, where the form of four tasks and two tiles would begin a second round of the chip: eight tasks and up to four tiles
// with one wave for a task's whole K range.  A workgroup of the smaller forms multiplies for a third of its time (QKV at 4287
// tokens: 17 of 44 us, the rest prologue, fold and epilogue) and every task group fetches the rows again.  A round of it
// takes about 25 us and 24 a tile, so the tiles are dealt evenly to the token groups that fill its rounds.  QKV projection
// (96 tasks, K = 2048), smaller forms -> this one: 641 tokens (the line) 64 -> 46 us, 704 67 -> 61, 1024 68 -> 63, 1300 75 -> 66, 1811
// 107 -> 87, 2048 112 -> 108, 2500 143 -> 113, 3072 174 -> 165, 4000 211 -> 178; output projection (32 tasks): 2049 66 -> 64, 2500 76 ->
// 69, 3072 80 -> 82, 4000 93 -> 85, but up to 2048, one round of the smaller form, 32 -> 48 to 52 -> 66.  Over 48 to 384 tasks, K of
// 256 to 4096 and 129 to 4000 tokens it gains 3 to 30 % but where the smaller form just fills its rounds: 192 tasks of K = 4096 352
// tokens 97 -> 100, 1024 tokens 184 -> 185.  Task groups with more than a tenth of their waves idle stay with the smaller forms.
constexpr int DENSE_WIDE_TASKS = 8, DENSE_WIDE_TILES = 4;
inline DenseForm dense_form(bool bf16, int n_tasks, int T) {
  const int groups = (n_tasks + 3) / 4, tiles = (T + DENSE_TILE - 1) / DENSE_TILE;
  const int wide = (n_tasks + DENSE_WIDE_TASKS - 1) / DENSE_WIDE_TASKS;
  if (bf16 && (long long)groups * ((tiles + 1) / 2) > DENSE_CUS && 10 * n_tasks >= 9 * DENSE_WIDE_TASKS * wide) {
    const long long least = (tiles + DENSE_WIDE_TILES - 1) / DENSE_WIDE_TILES, rounds = (wide * least + DENSE_CUS - 1) / DENSE_CUS;
    const long long fill = rounds * DENSE_CUS / wide, g = fill < least ? least : fill < tiles ? fill : tiles;
    return DenseForm{DENSE_WIDE_TASKS, DENSE_WIDE_TILES, (int)g};
  }
  const bool two = bf16 ? groups * tiles > DENSE_CUS : groups * ((tiles + 1) / 2) >= 160;
  return two ? DenseForm{4, 2, (tiles + 1) / 2} : groups * tiles >= DENSE_FILL ? DenseForm{4, 1, tiles} : DenseForm{2, 1, tiles};
}

// Up to 64 tokens: split-K.  K slices (workgroups) per task: as many as leave every wave exactly one burst of k-steps (8 with
// one token tile, 4 with two), when K divides that way; one otherwise and whenever there are several token groups.
inline int gemm_slices(bool bf16, int K, int T) {
  if (T > 2 * DENSE_TILE) return 1;
  const int ksteps = K / (bf16 ? 16 : 8);
  const int burst = 4 * (T <= DENSE_TILE ? 8 : 4);   // of a workgroup's four waves
  return ksteps % burst == 0 ? ksteps / burst : 1;
}
// Slices a launch uses of those gemm_slices() allows (the workspace is sized for the latter): a hand-off among
// fewer workgroups is cheaper, so a projection with many tasks takes only as many slices as bring the launch to
// about half a workgroup per compute unit (measured at 32 tokens, K = 2048: the QKV projection, 96 tasks, 12.3 us
// with 2 slices against 13.1 with 4 and 14.9 with 1; the output projection, 32 tasks, 8.1 us with 4 slices, 10.0
// with 2, 13.4 with 1).
inline int ksplit_slices(bool bf16, int K, int T, int n_tasks) {
  const int most = gemm_slices(bf16, K, T);
  int s = 1;
  while (s < most && s * n_tasks < DENSE_CUS / 2) s *= 2;
  return most % s == 0 ? s : most;
}
// bf16, up to 32 tokens: half a task per workgroup of HALF_KW waves instead of two slices of a task, where two slices are what
// split-K would take (the order of the sums is theirs), half tasks are half a round of the chip to a whole one, and a wave's
// share of K fits its registers (HALF_PF k-steps, or half as many: K of 2048 or 1024; 1536 takes three slices, and other
// multiples of 128 below 2048 one).  QKV projection, split-K -> half tasks in us at 1 / 11 / 32 tokens (with the events around a
// launch): 66 tasks of K = 1024 11.7 -> 9.3 / 10.8 -> 9.2 / 11.1 -> 9.7, 126 tasks 13.2 -> 10.4 / 12.3 -> 9.9 / 12.7 -> 10.7; 66 tasks of K = 2048
// 13.4 -> 11.9 / 12.9 -> 11.8 / 13.6 -> 13.0, 96 tasks 14.4 -> 13.1 / 13.7 -> 12.9 / 14.8 -> 14.1, 126 tasks 15.8 -> 14.1 / 14.9 -> 13.9 / 15.8 -> 15.2.
constexpr int HALF_KW = 8, HALF_PF = 16;   // waves; most k-steps of a wave
inline bool half_applies(bool bf16, int K, int T, int n_tasks) {
  if (!bf16 || T > DENSE_TILE || 4 * n_tasks < DENSE_CUS || 2 * n_tasks > DENSE_CUS) return false;
  return ksplit_slices(bf16, K, T, n_tasks) == 2 && K / 16 <= HALF_KW * HALF_PF;
}

}  // namespace dinfer
