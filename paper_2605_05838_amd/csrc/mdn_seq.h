// Where a workgroup's sequence or chunk lies: from the device tables of a packed batch, or by arithmetic for a
// fixed-length one.  Everything here is wave-uniform.
#pragma once
#include "mdn_kernels.h"

namespace mdn {

// Whether every chunk of a launch has 64 tokens and lies where arithmetic finds it.  The kernels' instances for that case
// (WHOLE) carry neither tables nor row limits, which cost registers that the kernels are short of: the 16-bit d = 128 gradient
// kernel spills 15 scalar registers with them and 4 without.  A pass in us, all launches by the general instances / by these:
// 8 x 2 048 tokens of 8 heads of 128 forward 92.5 / 91.4; forward and backward, 4 x 4 096 of 16 heads of 128 695 / 685, of 64
// 442 / 434.
inline bool whole_chunks(const Dims &d) { return !d.packed && d.T % 64 == 0; }

// one (sequence, head) pair of a scan
struct ScanSeq {
    size_t tok;   // its first token, as a row of the [tokens, H] tensors
    size_t blk;   // its first chunk block
    size_t state; // its index in the [sequences, H] state tensors
    int len;      // tokens
    int n0, n1;   // chunks of this launch
};
template <bool WHOLE> __device__ __forceinline__ ScanSeq scan_seq(const Dims &d, int bh) {
    const int b = bh / d.H, h = bh % d.H;
    ScanSeq q;
    if (!WHOLE && d.seqs) {
        // (from memory that the kernel also writes, the compiler loads the entry per lane, into vector registers)
        SeqEntry e = d.seqs[b];
        e.t0 = __builtin_amdgcn_readfirstlane(e.t0);
        e.len = __builtin_amdgcn_readfirstlane(e.len);
        e.cb = __builtin_amdgcn_readfirstlane(e.cb);
        e.idx = __builtin_amdgcn_readfirstlane(e.idx);
        const int N = (e.len + 63) >> 6;
        q.tok = (size_t)e.t0 * d.H + h;
        q.blk = (size_t)e.cb * d.H + (size_t)h * N;
        q.state = (size_t)e.idx * d.H + h;
        q.len = e.len;
        q.n0 = 0;
        q.n1 = N;
    } else {
        q.tok = (size_t)b * d.T * d.H + h;
        q.blk = (size_t)bh * d.N;
        q.state = bh;
        q.len = d.T;
        q.n0 = d.n0;
        q.n1 = d.n1;
    }
    return q;
}

// one chunk of a chunk-parallel kernel.  x runs over the chunks of a launch (those of all sequences for a packed
// batch, [n0, n1) of one (batch, head) pair otherwise), y over the heads or over the (batch, head) pairs.
struct ChunkPos {
    size_t tok; // its first token of this head, as a row of the [tokens, H] tensors
    size_t blk; // its chunk block
    int rows;   // tokens, 1..64
};
template <bool WHOLE> __device__ __forceinline__ ChunkPos chunk_pos(const Dims &d, int x, int y) {
    ChunkPos p;
    if (!WHOLE && d.chunks) {
        const ChunkEntry e = d.chunks[x];
        p.tok = (size_t)e.t0 * d.H + y;
        p.blk = (size_t)e.blk + (size_t)y * e.N;
        p.rows = e.rows;
    } else {
        const int n = d.n0 + x, b = y / d.H, h = y % d.H, left = d.T - n * 64;
        p.tok = ((size_t)b * d.T + (size_t)n * 64) * d.H + h;
        p.blk = (size_t)y * d.N + n;
        p.rows = WHOLE || left >= 64 ? 64 : left;
    }
    return p;
}
// the grid of such a launch
inline int chunk_grid_x(const Dims &d) { return d.chunks ? d.nchunks : d.n1 - d.n0; }
inline int chunk_grid_y(const Dims &d) { return d.chunks ? d.H : d.BH; }

} // namespace mdn
