// What the 16-bit scans (forward, reconstruction, reverse) have in common.  A workgroup of eight waves walks the chunks of one
// (sequence, head) pair for DVB dv columns, one barrier-separated phase after the other, and its waves have three jobs:
//   waves 0-3  the chain: every product of a step, the states in their accumulators.  They take all operands from LDS (in some
//              instances of the forward the q rows excepted) and leave all results there, so that nothing on the serial path waits for
//              memory;
//   waves 4-5  loads: the operands of chunks further on, HBM -> LDS without registers, into rings of 1 to 3 chunks;
//   waves 6-7  stores: results of the step before, LDS -> HBM (and at the start, with nothing to store, half of the first loads; with 16
//              columns also the operands of later chunks into the L2, see LineTouch).
// Loads and stores are apart because a wave's vector-memory operations are counted in order: a wave that does both waits for the
// acknowledgement of its stores whenever it waits for a load behind them.  With loads, stores and products in the same four waves
// a quarter to a half of a step was spent at the issue of memory instructions and in such waits (the forward scan of 4 x 4 096
// tokens, 16 heads of 128, in clocks of a step: 6 250, of them 3 400 in the products' phases).
#pragma once
#include "mdn_device.h"
#include "mdn_kernels.h"
#include "mdn_scan_rules.h"
#include "mdn_seq.h"

namespace mdn {

constexpr int kScanThreads = 512;

// Workgroups of a launch at most, a multiple of 8 (see xcd_map).  A launch of 2^32 threads or more reports no error and leaves
// workgroups out, and B * H = 2^24 pairs would reach that eight times over.  launch(number of the first workgroup, grid) for every part
// of `blocks` workgroups.
constexpr int kScanBlocks = 1 << 22;
template <typename F> hipError_t launch_in_parts(int blocks, F &&launch) {
    for (int first = 0; first < blocks; first += kScanBlocks) {
        launch(first, dim3(blocks - first < kScanBlocks ? blocks - first : kScanBlocks));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int DV, int DVB> int scan_blocks(const Dims &d) { return (d.BH + 7) / 8 * 8 * (DV / DVB); }
// see scan_bytes
inline size_t call_bytes(const Dims &d, bool vt, bool states) { return scan_bytes((size_t)d.nchunks * d.H, d.dk, vt, states); }

// LDS address of a __shared__ object, as M0 takes it
__device__ __forceinline__ unsigned lds_addr(const void *p) {
    return (unsigned)(size_t)((__attribute__((address_space(3))) const char *)p);
}

// vmcnt(N) alone
template <int N> __device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt immediate");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// 16 bytes per lane, HBM -> LDS: lane l's to dst + 16 l; base and dst are the same in all lanes.  (Inline assembly, and the waits by
// hand: see dma_token_tile.  The compiler does not see the hazard between a vector instruction that writes the base's scalar registers,
// such as the ones in front, and a vector-memory instruction that reads them: five wait states.)
__device__ __forceinline__ void dma16(const void *base, unsigned byte_off, unsigned dst) {
    const unsigned long long b = (unsigned long long)base;
    const unsigned long long ub = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32 |
                                  (unsigned)__builtin_amdgcn_readfirstlane((int)b);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(byte_off), "s"(ub), "s"(__builtin_amdgcn_readfirstlane((int)dst))
                 : "memory", "m0");
}

// 64 rows of LEN elements -> a tile of such rows in LDS, by two waves (w2 = 0, 1), COUNT instructions each.  SWIZZLE: the pieces of a
// row in the order of dma_token_tile.  The lanes' offsets are formed once per kernel.  `turn` (0..3): the quarter of the rows that
// comes first; the workgroups that want the same tile at the same time start with different quarters, so that most of
// their requests find the line already on its way (the forward's traffic without its products, 4 x 4 096 tokens of 16 heads of 128:
// 154 us, 168 us when all start with the same rows).
template <typename T, int LEN, bool SWIZZLE> struct TileLoad {
    static constexpr int E = 16 / (int)sizeof(T), CPR = LEN / E, XM = (CPR < 16 ? CPR : 16) - 1, P = 64 * CPR;
    static constexpr int COUNT = P / 128, QUARTER = P >= 256 ? P / 4 : 0;
    static_assert(P % 128 == 0 && QUARTER % 64 == 0, "whole waves");
    unsigned off[COUNT];
    // last: the last row that exists
    __device__ __forceinline__ void aim(unsigned rs, int w2, int lane, int turn, int last) {
#pragma unroll
        for (int u = 0; u < COUNT; ++u) {
            const int p = piece(u, w2, turn) + lane, row = p / CPR, pc = SWIZZLE ? (p % CPR) ^ (row & XM) : p % CPR;
            off[u] = ((unsigned)min(row, last) * rs + pc * E) * (unsigned)sizeof(T);
        }
    }
    static __device__ __forceinline__ int piece(int u, int w2, int turn) { return ((u * 2 + w2) * 64 + turn * QUARTER) & (P - 1); }
    __device__ __forceinline__ void request(const T *src, unsigned tile, int w2, int turn) const {
#pragma unroll
        for (int u = 0; u < COUNT; ++u) dma16(src, off[u], tile + piece(u, w2, turn) * 16);
    }
};

// The operands of chunks further on than the loads, brought into the L2 by the storing waves: four bytes of every 64, each workgroup of a
// (sequence, head) pair its share of the lanes.  A CU has only so many lines on their way at a time, so that what the loads bring per step is that
// over the latency of a line, which with the kept states' stores on the way to HBM grew until the loads were what a step waited for (16
// columns, d = 128: 3 700 clocks a step with kept states, 3 300 of them in the loading waves, 2 300 without the stores); out of the L2 they keep up.
// Every 64 bytes: of a line of 128 asked for once only half is fetched.  32 768 tokens of 16 heads of 128 in us, without / every 128 bytes
// / every 64 / every 32: forward 675 / 662 / 648 / 665, with kept states 924 / 797 / 772 / 803, forward and backward 1 846 / 1 675 / 1 646 / 1 677; three,
// four and six chunks ahead 1 661, 1 646 and 1 657.  Those in front of a step's last stores; behind them, as now, with kept states 750, forward
// and backward 1 614 (65 536 tokens of 16 heads of 64 2 466, 2 478 in front of them, 2 838 without); in the phase before 1 622, but 2 767 with heads of 64.
constexpr int kTouchAhead = 4;
// Where it is used: see touch_pays.
template <int DK, int DV, int G> struct LineTouch {
    static constexpr int LINE = 64, RK = DK * 2 / LINE, RV = DV * 2 / LINE;                              // lines of a row
    static constexpr int K = 64 * RK, V = 64 * RV, M = 4096 * 2 / LINE, C = 64 * kCoefRows * 4 / LINE; // of a tensor's chunk
    static constexpr int LINES = 2 * K + V + 2 * M + C, N = (LINES + G * 128 - 1) / (G * 128);
    const char *at[N];
    ptrdiff_t step[N];
    int end[N]; // a lane's line is in the chunks before this one
    // part: this wave's number among those of the pair's workgroups; n: the first chunk touched; rows behind `last` are not in chunk `ragged`
    __device__ __forceinline__ void aim(const void *k, const void *q, const void *v, const void *Tm, const void *Bm, const float *coef, const ScanSeq &sq, int H,
                                        int part, int lane, int n, int ragged, int last) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            int p = (u * G * 2 + part) * 64 + lane;
            end[u] = p < LINES ? sq.n1 : 0;
            if (p < 2 * K + V) { // [tokens, H, D]
                const void *t = p < K ? k : p < 2 * K ? q : v;
                const int per_row = p < 2 * K ? RK : RV, bytes = per_row * LINE;
                p = p < K ? p : p < 2 * K ? p - K : p - 2 * K;
                const int row = p / per_row;
                step[u] = (ptrdiff_t)64 * H * bytes;
                at[u] = static_cast<const char *>(t) + (sq.tok + (size_t)row * H) * bytes + p % per_row * LINE;
                if (ragged >= 0 && row > last) end[u] = ragged;
            } else { // chunk blocks
                p = min(p, LINES - 1) - (2 * K + V);
                const void *t = p < M ? Tm : p < 2 * M ? Bm : coef;
                step[u] = (p < 2 * M ? M : C) * LINE;
                p = p < M ? p : p < 2 * M ? p - M : p - 2 * M;
                at[u] = static_cast<const char *>(t) + sq.blk * step[u] + p * LINE;
            }
            at[u] += n * step[u];
        }
    }
    // chunk n: that of aim(), then the one after (DIR 1) or before it (-1) at every call.  (As LDS transfers, which nothing has to wait
    // for: dst is 256 bytes that nobody reads.)
    template <int DIR> __device__ __forceinline__ void chunk(int n, unsigned dst) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            if (n < end[u])
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 4\n\tglobal_load_lds_dword %0, off"
                             :
                             : "v"(at[u]), "s"(__builtin_amdgcn_readfirstlane((int)dst))
                             : "memory", "m0");
            at[u] += DIR * step[u];
        }
    }
};

// A tile kept [k][m] (ATile<bf16_t, 16 MV, ..>) as the rows of a tensor: 16 bytes, columns 8 pc .. 8 pc + 7 of the workgroup's
// (the columns that MFMA row 4 kg + x of tile mv stands for: 4 MV kg + 4 mv + x)
template <int MV> __device__ __forceinline__ bf16x8 tile_piece(const bf16_t *t, int ld, int row, int pc) {
    if constexpr (MV == 2) {
        const bf16x4 lo = load4_raw(t + row * ld + pc * 4), hi = load4_raw(t + row * ld + 16 + pc * 4);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
        return Op<bf16_t>::load(t + row * ld + pc * 8);
    }
}

// The storing waves' work (w2 = 0, 1).  Everything goes out non-temporal: stores that stay in the L2 until a load pushes them out
// stand in the way of the loads (traffic of a 16-column scan without its products, 2 048 tokens of 16 heads: 1.6 us a step, 0.95
// with non-temporal stores; 16 384 tokens 1.5 / 1.2).
template <int DK, int DV, int MV> struct StateStore { // a [2][DK][16 MV] copy (S | M) -> this workgroup's columns of a chunk block
    typedef ATile<bf16_t, MV * 16, 2 * DK> TS;
    static constexpr int N = 2 * DK * MV * 16 / 8 / 128; // 16-byte stores per lane
    bf16x8 v[N];
    static __device__ __forceinline__ int piece(int u, int w2, int lane) { return (u * 2 + w2) * 64 + lane; }
    __device__ __forceinline__ void read(const bf16_t *copy, int w2, int lane) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int p = piece(u, w2, lane), block = p / (4 * DK), row = p / 2 % (2 * DK);
            v[u] = tile_piece<MV>(copy, TS::LD, row, block * 2 + (p & 1));
        }
    }
    template <int U0, int U1> __device__ __forceinline__ void put(bf16_t *states, int dv0, int w2, int lane) const {
#pragma unroll
        for (int u = U0; u < U1; ++u) {
            const int p = piece(u, w2, lane), block = p / (4 * DK), row = p / 2 % (2 * DK);
            bf16_t *to = states + (row >= DK ? DK * DV : 0) + vblk(DK, row & (DK - 1), dv0 + block * 16 + (p & 1) * 8);
            __builtin_nontemporal_store(v[u], reinterpret_cast<bf16x8 *>(to));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
};
// a [64 tokens][16 MV] copy -> rows of a [tokens, H, DV] tensor from `base` on
template <int DV, int MV, bool WHOLE>
__device__ __forceinline__ void store_token_rows(bf16_t *base, const bf16_t *copy, int rows, int H, int w2, int lane) {
    constexpr int PPT = MV * 2, LD = ATile<bf16_t, MV * 16, 64>::LD; // 16-byte pieces per row
    const RowStore<bf16_t, WHOLE> out(base, rows, H * DV, MV * 16);
#pragma unroll
    for (int u = 0; u < MV; ++u) {
        const int p = (u * 2 + w2) * 64 + lane;
        out.put_nt((unsigned)(p / PPT * H) * DV + p % PPT * 8, tile_piece<MV>(copy, LD, p / PPT, p % PPT));
    }
    __builtin_amdgcn_sched_barrier(0);
}

// The chain's states: element x of tile (mv, nd) of wave w is S[dk = (w ND + nd) 16 + r][dv = dv0 + 4 MV kg + 4 mv + x].
template <int DK, int DV, int MV> struct ChainStates {
    static constexpr int ND = DK / 64;
    typedef ATile<bf16_t, MV * 16, 2 * DK> TS;
    f32x4 S[MV][ND], M[MV][ND];
    static __device__ __forceinline__ size_t at(size_t state, int w, int nd, int mv, int dv0, int r, int kg) {
        return (state * DK + (w * ND + nd) * 16 + r) * DV + dv0 + kg * (4 * MV) + mv * 4;
    }
    // from fp32 tensors (null: zeros)
    __device__ __forceinline__ void load(const float *s, const float *m, size_t state, int w, int dv0, int r, int kg) {
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
            for (int nd = 0; nd < ND; ++nd) {
                const size_t g = at(state, w, nd, mv, dv0, r, kg);
                S[mv][nd] = s ? *reinterpret_cast<const f32x4 *>(s + g) : f32x4{0.f, 0.f, 0.f, 0.f};
                M[mv][nd] = m ? *reinterpret_cast<const f32x4 *>(m + g) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
    }
    __device__ __forceinline__ void store(float *s, float *m, size_t state, int w, int dv0, int r, int kg) const {
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
            for (int nd = 0; nd < ND; ++nd) {
                const size_t g = at(state, w, nd, mv, dv0, r, kg);
                if (s) *reinterpret_cast<f32x4 *>(s + g) = S[mv][nd];
                if (m) *reinterpret_cast<f32x4 *>(m + g) = M[mv][nd];
            }
    }
    // the 16-bit copy in LDS
    __device__ __forceinline__ void publish(bf16_t *copy, int w, int r, int kg) const {
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
            for (int nd = 0; nd < ND; ++nd) {
                const int dk = (w * ND + nd) * 16 + r;
                TS::put4(copy, mv * 16 + kg * 4, dk, S[mv][nd]);
                TS::put4(copy, mv * 16 + kg * 4, DK + dk, M[mv][nd]);
            }
    }
    // what that rounding dropped, rounded again, -> a chunk block in HBM (calls that bring state adjoints in: see GradArgs)
    __device__ __forceinline__ void store_lo(bf16_t *block, int w, int dv0, int r, int kg) const {
#pragma unroll
        for (int nd = 0; nd < ND; ++nd) {
            bf16x4 ls[MV], lm[MV];
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                ls[mv] = narrow4<bf16_t>(S[mv][nd] - widen4_packed(narrow4<bf16_t>(S[mv][nd])));
                lm[mv] = narrow4<bf16_t>(M[mv][nd] - widen4_packed(narrow4<bf16_t>(M[mv][nd])));
            }
            bf16_t *to = block + vblk(DK, (w * ND + nd) * 16 + r, dv0 + kg * (4 * MV));
            store_cols_raw<MV>(to, ls);
            store_cols_raw<MV>(to + DK * DV, lm);
        }
    }
};

} // namespace mdn
