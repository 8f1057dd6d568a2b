// Which form the dense projections (QKV and output) of more than 64 tokens take.  Plain host C++.
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
// (96 tasks), before -> now: 800 tokens 74 -> 73 us, 1300 82 -> 75, 1811 122 -> 101, 2500 157 -> 128, 3072 191 -> 181, 4000
// 234 -> 195; output projection (32 tasks): 2500 79 -> 73, 4000 95 -> 90, 4287 121 -> 103, but up to 2048, one round of the
// smaller form, 32 -> 48 to 52 -> 66.  Task groups with more than a tenth of their waves idle stay with the smaller forms.
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

}  // namespace dinfer
