// Which results go through the XCDs' L2s to memory as they are stored (store_through), and which stay there until the launch ends.  Plain
// arithmetic of the host, also compiled by the test of the lines below (tests/test_store_rule.py).
//
// A launch that leaves megabytes of changed lines in the L2s ends with their write-back, for which the next one waits: through the L2 wins while
// that is a good part of the launch.  Where a row does not start on a cache line, workgroups next to each other write half a line each; stores
// that stay in the L2 are put together there, others reach memory as two pieces, which costs more the more of them there are.
//   Time left in the L2 against through it, geometric mean and range over passes of 8000 to 60000 tokens, H from 32 to 1000, P 30 to 900:
//     MiB of the array                  up to 16              16 .. 32              32 .. 64              more
//     states, rows of whole lines       1.02  (0.99 .. 1.09)  1.02  (1.00 .. 1.07)  1.01  (1.00 .. 1.02)  1.001 (0.97 .. 1.07)
//     states, other rows                1.02  (0.99 .. 1.12)  1.01  (0.99 .. 1.05)  0.999 (0.98 .. 1.01)  0.991 (0.97 .. 1.01)
//     outputs, rows of whole lines      1.004 (0.97 .. 1.16)  1.01  (0.98 .. 1.07)  1.002 (0.98 .. 1.03)  0.997 (0.98 .. 1.01)
//     outputs, other rows               1.01  (0.99 .. 1.10)  1.004 (0.99 .. 1.04)  0.986 (0.92 .. 1.004) 0.94  (0.81 .. 0.996)
//   (Outputs of sequences of 256, on two planes and 128-row tiles mostly: 0.995 to 1.000 in every column.)  With all of them through the L2 the forward pass of
// 300 x 200 tokens, H = 500, P = 64 took 144 us instead of 131, of 160 x 200, 900, 30 118 instead of 95.
//   Scan kernels (scan and its reverse), rows of no whole lines: 11 MiB 1.10, 23 1.05, 46 to 62 0.997 to 1.016, 64 to 192 with P = 900, 935 or 100 0.97 to 1.00,
// with 250, 300 or 530 0.998 to 1.03.  Rows of whole lines, 128 to 384 MiB: 0.997 to 1.016.
//   All of the above repeats a pass on the same arrays.  Over four sets of arrays in turn, what the rule leaves in the L2 would take 1.025 (states, forward), 1.014
// (forward and gradient pass) and 1.039, 1.015 (outputs) times as long through it, 0.995 at the least (120 passes).  Not kept: left in the L2 as well where a row
// scan of at most 128 input columns has more than one round of workgroups (513 tiles of 64 x 128 and more).  Repeated on the same arrays the forward pass alone gains 2 to 5 %
// (6981 tokens, H = 38, P = 553: 49.5 -> 46.1 us) and forward and gradient pass lose 0.7 %; over four sets in turn the forward pass loses 1 to 3 % up to 1500 tiles.
#pragma once

#include <stdint.h>

namespace ssm {

constexpr int64_t CACHE_LINE = 128;
inline bool whole_lines(uintptr_t base, int64_t pitch) { return ((base | (uintptr_t)pitch) & (CACHE_LINE - 1)) == 0; }

// C and, where the store function has a second result, C2 (0: none): `rows` rows each, `pitch` bytes apart.  (A lane stores 16 bytes.  Where these
// are not aligned they are written in pieces that only the L2 puts together: forward pass of 208 x 64 tokens, H = 35, P = 72: 21.4 us, through
// the L2 24.0; forward and gradient pass of 200 x 64, 99, 33: 61.4 and 66.3, of 208 x 64, 64, 72: 65.1 and 62.5.)
inline bool output_through(uintptr_t C, uintptr_t C2, int64_t rows, int64_t pitch)
{
    if (((C | C2 | (uintptr_t)pitch) & 15) != 0) return false;
    return whole_lines(C | C2, pitch) || rows * pitch * (C2 ? 2 : 1) <= 32 << 20;
}

// `rows` tokens of P complex states each
inline bool states_through(uintptr_t x, int64_t rows, int64_t P) { return whole_lines(x, 8 * P) || rows * 8 * P <= 64 << 20; }

}  // namespace ssm
