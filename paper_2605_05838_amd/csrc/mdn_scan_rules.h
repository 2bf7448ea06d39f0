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

// Whether a forward scan takes the q rows as a tile brought by the loading waves: no loads, and no waits for them, in the waves of the
// chain; but 16 (d = 64) or 32 KB more of LDS and four more of its reads in a step's last phase.  `pairs`: (sequence, head) pairs; `chunks`:
// of a sequence, on average.  Forward in us, q in registers / as a tile.
// 32 columns: where the kept states' stores hold up every load (d = 128; at d = 64 the chain is the longer part of a step then too).  The launch
// between those of a training step, 16 heads of 128: 4 x 1 500 tokens 64.8 / 62.9, 4 x 2 048 82.6 / 79.3, 4 x 2 500 105.4 / 98.7, of a whole layer's 4 x 2 048
// 65.8 / 64.0; calls of nothing but the forward, 4 x 2 048 83.2 / 83.9, 4 x 3 072 120 / 123, 8 x 2 048 213 / 205.  Without kept states 4 x 4 096 150 / 157,
// 8 x 2 048 of 8 heads 84 / 87, 4 x 4 096 of 24 heads of 64 100.8 / 105.5.
// 16 columns: where states are kept (16 heads of 128, 4 096 tokens 86.8 / 85.0; 4 heads 82.2 / 77.5) and where the start counts (up to 8 chunks: 64 tokens of
// 16 heads of 128 11.0 / 10.7, 512 19.2 / 19.1, 600 of 8 heads 20.7 / 20.8).  Else, with inputs out of HBM, heads of 128 where the caches don't hold what
// is moved, with V~ a little earlier (16 heads, 16 384 tokens (344 MB) 334 / 320, 22 000 508 / 452, 30 000 of 8 heads (315 MB) 548 / 546; V~ kept, 30 000 of 6
// (282 MB) 603 / 550); below it what the tile's reads add to the chain is more (777 25.2 / 25.9, 4 096 of 8 heads 78.8 / 81.3, 6 000 122 / 128, 30 000 of 4 502 /
// 536, V~ kept 510 / 533).  Heads of 64 except where a few pairs' loads have the memory to themselves (16 heads, 8 192 tokens 133 / 131, 22 000 395 / 367;
// 4 heads, 4 096 56.4 / 57.3, 30 000 386 / 370; 2 heads 53.5 / 56.1, 342 / 360, but V~ kept 53.9 / 54.5, 359 / 358).
constexpr bool q_tile_pays(int columns, int d, size_t pairs, size_t chunks, size_t bytes, bool vt, bool states) {
    if (columns == 32) return d == 128 && states;
    if (states || chunks <= 8) return true;
    return d == 64 ? vt || pairs >= 4 : bytes > (vt ? 4 : 5) * kLastLevelCache / 4;
}

} // namespace mdn
