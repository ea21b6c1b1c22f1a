// How a transform is cut into passes and register rounds, and the bounds that its
// lazy words are held to.  Plain constants and functions: the kernels are built
// from them, and a CPU test follows the bounds through every schedule with them.
#pragma once
#include <stdint.h>

namespace hentt {

// Round geometry, for the block pass's stage count.
template <int B, int E> struct FwdFirst {   // forward: first round is the short one
  static constexpr int R = (B % E) ? (B % E) : E;
  static constexpr int LO = B - R;
};
template <int B, int E> struct InvLast {    // inverse: last round is the short one
  static constexpr int R = (B % E) ? (B % E) : E;
  static constexpr int LO = B - R;
};

// Words per lane (log2) of the kernels that hold a whole transform, product, or
// rescale in one workgroup.  Measured over 2, 3 and 4 at 1 to 4096 units: more
// lanes with fewer words win at every batch size, by latency at few units (the
// product of one pair of 2^12: 13.0 us with 8 words, 16.2 with 16) and by
// occupancy at many (2^12 forward, 4096 units: 68.6 against 72.9 us; 2^10
// product, 512 units: 9.8 us with 4 words, 12.4 with 8, 14.9 with 16).  At 2^13, where a
// workgroup of 8 words per lane fills a CU, the forward transform keeps 16 for calls of
// more than two generations (launch_whole).
constexpr int whole_e(int log_n) { return log_n <= 10 ? 2 : log_n <= 13 ? 3 : 4; }

// Column stages of a two-pass transform or product at N = 2^log_n (measured over
// 6 to 8 stages and, through registers alone, 1 to 5): the blocks behind it are
// of 2^7 to 2^9 words, so that one wave holds a block (three radix-8 rounds and
// no barrier).
constexpr int two_pass_cols(int log_n) { return log_n <= 15 ? 6 : log_n - 9; }

// Words of a workgroup of a two-pass transform's block pass of ST stages, 2^E
// words per lane: at least one wave.
constexpr int block_words(int st, int e) { return st > e + 6 ? st : e + 6; }

// ------------------------------------------------------------- bounds ----
// Every product by a root power is below 12q.  Three classes of moduli by their bit
// length k, uniform per workgroup:
//
// Forward stages (X' = X + WY, Y' = X - WY + 12q: both below X + 12q).
//   34..55 bits  no corrections: 17 stages add at most 204q to the input, a few q or a
//                60-bit word (the rescale's and the key switch's lifted words), below
//                2^63 in all;
//   56..60 bits  X, any 64-bit word, is brought below 3q (est3) before every stage
//                (3 + 12 < 16);
//   33 or fewer  no corrections (est3 leaves the words as they are): below 207q.
//
// Inverse stages (X' = X + Y doubles the bound of the words that stay on the X
// side), in rounds of R stages.  Words enter a round below 2^LBIN q and leave it below
// 2^LBOUT q:
//   34..55 bits  none inside a round: words stay below 512q (LBIN + R <= 9); at its end
//                the words that could exceed 2^LBOUT q are corrected (inv_over: the
//                few with a long run of X sides behind them);
//   56..60 bits  words below 4q on entry, or products below 7q: the product corrected
//                after every stage, X' after every second one and after the round's
//                last (8 + 8 <= 16);
//   33 or fewer  none in the whole transform: at stage v words are below
//                16q 2^v < 2^54.
// The last stage of a transform multiplies both of its outputs, which leaves 12q.
constexpr bool uncorrected(uint32_t k) { return k - 34u <= 21u; }

// Words between passes (in memory), and between rounds of one kernel: below 2^LB q.
constexpr int LB_PASS = 4, LB_ROUND = 5;

// 34..55 bits: whether word k of a round of R stages is corrected at its end.
template <int R, int LBIN, int LBOUT> constexpr bool inv_over(int k) {
  int h = -1;
  for (int b = 0; b < R; ++b)
    if ((k >> b) & 1) h = b;
  const int bound = h < 0 ? 1 << (LBIN + R) : 12 << (R - 1 - h);
  return bound > (1 << LBOUT);
}
// The others: whether a word is corrected after stage u of a round (y: a product).
constexpr bool inv_fix(int R, int u, bool y) { return y || (u & 1) || u == R - 1; }
// log2 of the multiple of q that keeps X - Y positive at stage u of a round, stage v
// of the transform.
constexpr uint32_t inv_off_log(uint32_t k, bool fix, int lbin, int u, int v) {
  return !fix ? (uint32_t)(lbin + u) : k < 34 ? 4u + v : 3u;
}

}  // namespace hentt
