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
//  - Prompts of one length all end together: workgroups a little beyond a round of the chip share some compute units and
//    leave the others idle for the second half of the launch (one prompt, bf16, rows / splitting form, gain of the whole
//    layer in per cent; 8 heads: 256 workgroups +6, 264 to 312 -11 to -14, 328 to 376 -2, 392 +6, 520 and 544 -8; 16
//    heads: 256 +6, 272 to 320 -4 to -6, 336 +2, 512 +12, 544 -4, 592 +2; 24 heads: 264 to 312 -1 to -3, 336 +3).  The
//    shorter the walk the less that weighs (32 heads, 1132 and 1260 keys: -1 to +1; 4 prompts of 640: +4), and prompts
//    of different lengths fill each other's gaps (384 workgroups of 1536, 1024 and 512 keys: +6).
//  - Behind cached prefixes, whose lengths the host does not know, the launch lasts as long as the longest one, walked by
//    one wave where the splitting form has eight (16 sequences of 64 + 32 positions, one layer of a vicinity step, rows /
//    splitting form: prefixes of 512 1629 / 1642 us, of 4096 1783 / 1780, of 100 to 8000 1886 / 1793; 64 + 16 positions
//    behind 1000 to 4096 1539 / 1511).
inline int attn_rows_groups(const int* off, int n_seq, int n_heads, bool from_zero) {
  int groups = 0, tiles = 0, longest = 0;
  long long work = 0;      // keys times workgroups
  for (int s = 0; s < n_seq; ++s) {
    const int keys = off[s + 1] - off[s], n = (keys + ROWS_TILE - 1) / ROWS_TILE, g = (n + ROWS_WAVES - 1) / ROWS_WAVES;
    tiles += n;
    groups += g;
    work += (long long)keys * g;
    longest = keys > longest ? keys : longest;
  }
  const int wgs = groups * n_heads;
  if (!from_zero || wgs < ROWS_MIN_WGS || 4 * tiles < 3 * ROWS_WAVES * groups) return 0;
  const bool alike = 10 * work >= 9ll * groups * longest, beyond = wgs > 256 && wgs <= 320;
  const bool far_beyond = wgs > 256 && (wgs <= 384 || (wgs > 512 && wgs <= 576));
  return alike && ((longest > 1280 && beyond) || (longest > 4096 && far_beyond)) ? 0 : groups;
}

}  // namespace dinfer
