// Which form the dense projections (QKV and output) of more than 64 tokens take.  Plain host C++.
#pragma once

namespace dinfer {

constexpr int DENSE_TILE = 32;    // token rows of a tile
constexpr int DENSE_CUS = 256;    // compute units: a workgroup fills one
constexpr int DENSE_FILL = 140;   // workgroups a launch of four tasks and one tile each must keep

struct DenseForm {
  int tasks, tiles;               // per workgroup: 4 and 2, 4 and 1, 2 and 1
};
// bf16: one round of the chip takes 41 us (QKV of the 2048-wide model, four tasks and two tiles), 25 (four tasks, one tile)
// or 20 (two tasks, one tile): four tasks and one tile while their workgroups are one round (352 tokens: 264 of them, two
// rounds, 46 us; with two tiles 39; output projection at 1100 tokens 46 and 38), two tasks where four would leave nearly
// half the chip idle (192 tokens: 288 workgroups of two tasks, two rounds, 28 us; 144 of four, 26.7).
// float32: the matrix instructions bound a workgroup, so that one with two tiles takes twice as long as one with one, and
// a few workgroups beyond a round cost no more than two tiles each (hidden 1024, QKV: 704 tokens 80.6 us with one tile,
// 264 workgroups, 87.8 with two; 256 tokens of 3072 features 81.4 and 89.2): two tiles from 160 workgroups of them on.
inline DenseForm dense_form(bool bf16, int n_tasks, int T) {
  const int groups = (n_tasks + 3) / 4, tiles = (T + DENSE_TILE - 1) / DENSE_TILE;
  const bool two = bf16 ? groups * tiles > DENSE_CUS : groups * ((tiles + 1) / 2) >= 160;
  return two ? DenseForm{4, 2} : groups * tiles >= DENSE_FILL ? DenseForm{4, 1} : DenseForm{2, 1};
}

}  // namespace dinfer
