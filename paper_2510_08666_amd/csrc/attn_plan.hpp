// Which form of attention a forward takes.  Plain host C++.
#pragma once

namespace dinfer {

constexpr int ROWS_TILE = 32, ROWS_WAVES = 4, ROWS_MIN_WGS = 256;

// Groups of ROWS_WAVES query tiles if the rows form (attention_rows_kernel: one query tile per wave, which walks all keys
// of its sequence) takes the forward, else 0: the splitting form.  off[0 .. n_seq]: first token of every sequence;
// from_zero: all of them start at position 0 (prompts).
//  - A wave walks all keys alone, so the launch must fill the chip without splitting them (one prompt, 16 heads, rows /
//    splitting form in microseconds: 1024 tokens, 128 workgroups, 45 / 37; 2048 tokens, 256 workgroups, 89 / 103; 4096
//    tokens 266 / 345; prompts of 1811 + 333 + 825 + 1318, 576 workgroups, 136 / 169), with queries for three of four
//    waves.
//  - Behind cached prefixes, whose lengths the host does not know, the launch lasts as long as the longest one, walked by
//    one wave where the splitting form has eight (16 sequences of 64 + 32 positions, one layer of a vicinity step, rows /
//    splitting form: prefixes of 512 1629 / 1642 us, of 4096 1783 / 1780, of 100 to 8000 1886 / 1793; 64 + 16 positions
//    behind 1000 to 4096 1539 / 1511).
inline int attn_rows_groups(const int* off, int n_seq, int n_heads, bool from_zero) {
  int groups = 0, tiles = 0;
  for (int s = 0; s < n_seq; ++s) {
    const int n = (off[s + 1] - off[s] + ROWS_TILE - 1) / ROWS_TILE;
    tiles += n;
    groups += (n + ROWS_WAVES - 1) / ROWS_WAVES;
  }
  return from_zero && groups * n_heads >= ROWS_MIN_WGS && 4 * tiles >= 3 * ROWS_WAVES * groups ? groups : 0;
}

}  // namespace dinfer
