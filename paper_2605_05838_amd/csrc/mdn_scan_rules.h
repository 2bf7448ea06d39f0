// Which instances of the 16-bit scans a call takes, by what it moves.  (Plain C++: sizes in, answers out.)
#pragma once
#include <stddef.h>

namespace mdn {

constexpr size_t kLastLevelCache = (size_t)256 << 20; // bytes

// Bytes that a 16-bit scan over `blocks` chunk blocks (64 tokens of a head) of d x d states moves between HBM and the caches at least: k, q, v
// (reverse: dO), T, Bm and the coefficients in, o (dv) out; with `vt` the V~ rows, with `states` the chunk states (their adjoints) out.
constexpr size_t scan_bytes(size_t blocks, int d, bool vt, bool states) {
    const size_t rows = 64 * (size_t)d * 2, operands = 3 * rows + 2 * 64 * 64 * 2 + 64 * 8 * 4;
    return blocks * (operands + rows + (vt ? rows : 0) + (states ? 2 * (size_t)d * d * 2 : 0));
}

// Whether the storing waves bring later chunks' operands into the L2 (LineTouch): only where a call moves about twice the last-level
// cache, whose latency the loads cover.  In us, without / with, forward with kept states: 16 heads of 128 with 14 336 tokens (595 MB) 277 / 270,
// 16 384 334 / 340, 20 000 528 / 461, 32 768 936 / 753; forward alone, 26 624 (559 MB) 622 / 524, 4 heads with 131 072 tokens 2 538 / 2 242.
// The reverse scan finds more in the caches behind a forward pass than its bytes say; forward and backward by it, 8 192 tokens of
// 16 heads of 128 (306 MB in the reverse scan) 433 / 439, 14 336 (536 MB) 750 / 753, 16 384 850 / 839, 32 768 1 663 / 1 608; 16 heads of 64 with 16 384
// (277 MB) 638 / 649, 28 672 (485 MB) 1 139 / 1 083, 65 536 2 608 / 2 446.
// And not with 32 columns, where every CU is at work and HBM itself is busy: 4 x 4 096 of 16 heads of 128 595 / 604 (every 128 bytes), forward of
// heads of 64 96 / 115.
// A call that is split into segments is asked for as a whole, not launch by launch: what a launch reads was last touched by the launches of
// another pass over all of it (32 768 tokens of 16 heads of 128, a reverse scan in eight segments of 153 MB: the 1 663 / 1 608 above).
constexpr bool touch_pays(size_t bytes, bool reverse) { return bytes > (reverse ? 9 : 10) * kLastLevelCache / 5; }

} // namespace mdn
