// Host-side launch interface between the C ABI (mdn_api.hip) and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mdn {

// One sequence of a packed batch, and one 64-token chunk of it: device tables that packed calls build in their
// workspace (fixed-length batches need none: the same values follow from B, T, H).
struct SeqEntry {
    int t0, len; // first token (row of the [T_total, H, *] tensors), tokens
    int cb;      // chunks of the sequences before it in memory order
    int idx;     // its index in the caller's order (states are [n_seq, H, dk, dv] in that order)
};
struct ChunkEntry {
    int t0, rows; // first token, tokens (1..64)
    int blk, N;   // chunk block of head 0, and what each further head adds (the sequence's chunks)
};

struct Dims {
    int B, T, H, N, BH; // B sequences of T tokens, N = ceil(T / 64) chunks each, BH = B * H.  Packed batches: B
                        // sequences of their own lengths, N = the longest one's chunks, T = all tokens
    int n0, n1;         // chunks [n0, n1) handled by this launch (0, N unless the call is split into segments)
    int dk, dv;
    int dtype; // MDN_DTYPE_*
    float scale;
    int nchunks;              // chunks of all sequences together (B * N unless packed)
    const SeqEntry *seqs;     // packed batches: [B], longest first (the scans' order of dispatch); otherwise null
    const ChunkEntry *chunks; // packed batches: [nchunks], memory order; otherwise null
    bool packed;              // sizes of a packed batch (host side; the tables are set for its launches)
};

// Chunk-parallel precompute ("intra") kernel arguments.  Workspace tensors are chunk-blocked,
// [sequence][H][chunk of the sequence][tile] (written [BH][N] below: what it is for a fixed-length batch), in the storage
// dtype unless noted; inside a tile, a [rows][dv] tensor is in the vblk layout of mdn_device.h, and an MFMA operand [rows][k] in its
// kblk layout (32-bit storage) or row by row (16-bit storage, whose scans read tiles through LDS).
// 16-bit storage has one set of operands, coef, T and Bm, for the forward and the reverse pass: their transposes and those of k and
// q are transposing LDS reads there.
// A chunk of fewer than 64 tokens (the last one of a sequence) is filled up with identity steps of the recurrence:
// k = q = eta = 0, alpha = mu = 1, beta = 0.  The intra kernel writes its operands that way (rows of K^T, Q^T, Bm zero,
// rows of T those of the unit matrix, Gamma_C = Rho_C = 0), after which whatever finite values the scans read for V, k,
// dO in those rows meet zeros; the scans read the last real token's row there and store only real rows.
constexpr int kCoefBlockCols = 8; // floats per token in the coefficient block

struct IntraArgs {
    const void *q, *k;                      // [B,T,H,dk]
    const float *alpha, *beta, *mu, *eta;   // [B,T,H]; eta may be null
    float *coef;                            // [BH][N][64][kCoefBlockCols] fp32 (one row of coefficients per token)
    void *Tm;                               // [64][64]        T = (I + A)^-1: row i, contraction index j
    void *Bm;                               // [64][64]        (Q~ K~^T) .* Gamma
    // 32-bit storage
    void *KT;                               // kblk [dk][64]   raw k, transposed
    // 32-bit storage, backward mode
    void *QT;                               // kblk [dk][64]   raw q, transposed
    void *BmT;                              // kblk [64][64]   Bm transposed
    void *TmT;                              // kblk [64][64]   T transposed
};

struct ScanFwdArgs {
    const void *q, *k;                      // [B,T,H,dk]
    const void *v;                          // [B,T,H,dv]
    const float *coef;
    const void *KT, *Tm, *Bm;
    const float *S0, *M0;                   // [B,H,dk,dv] or null
    void *o;                                // [B,T,H,dv]
    void *vt_saved;                         // [B,T,H,dv] or null
    void *states_saved;                     // [BH][N][2] x vblk [dk][dv], or null
    void *states_lo;                        // reconstruction, same layout, or null: what the 16-bit rounding of
                                            // states_saved dropped (see GradArgs)
    float *S_final, *M_final;               // or null
};

// State reconstruction from saved V~ (backward, when the forward did not keep the states).
struct RebuildArgs {
    const float *coef;
    const void *k;                          // [B,T,H,dk]
    const void *KT;                         // 32-bit storage
    const void *vt_saved;                   // [B,T,H,dv]
    const float *S0, *M0;
    void *states;                           // [BH][N][2] x vblk [dk][dv]
    void *states_lo;                        // or null: the rounding remainders of `states` (16-bit storage)
};

struct ScanBwdArgs {
    const void *q, *k;                      // [B,T,H,dk]
    const void *dO;                         // [B,T,H,dv]
    const float *coef;
    const void *Tm, *Bm;                    // 16-bit storage
    const void *QT, *KT, *BmT, *TmT;        // 32-bit storage
    const float *dS_final, *dM_final;       // or null
    void *dv;                               // [B,T,H,dv]  dV = T^T dV~
    void *dstates;                          // [BH][N][2] x vblk [dk][dv]: adjoints of the chunk-END states
    void *dstates_lo;                       // or null: the rounding remainders of `dstates` (16-bit storage)
    float *dS0, *dM0;                       // or null
};

struct GradArgs {
    const void *q, *k;                      // [B,T,H,dk]
    const float *alpha, *beta, *mu, *eta;
    const void *vt_saved, *dO, *dv;         // [B,T,H,dv]; dv (= dR, from the reverse scan) is read
    const void *KT, *QT;
    const void *states, *dstates;           // [BH][N][2] x vblk [dk][dv]
    // 16-bit storage, calls that bring adjoints of the final states in (both or neither): x - bf16(x) of the two
    // tensors above, again in bf16.  Adjoints that enter from outside can be large against everything dO puts into
    // the states; <dS', S>, <dS', M>, <dM', M> and the products of dS', dM' with V~ are then sums of dk dv terms
    // whose storage rounding alone would reach the tolerance, so those sums take hi + lo of both factors.
    const void *states_lo, *dstates_lo;
    void *dq, *dk;
    float *dalpha, *dbeta, *dmu, *deta;     // deta may be null
};

struct RecurrentArgs {
    const void *q, *k, *v;
    const float *alpha, *beta, *mu, *eta;
    float *S, *M;
    void *o;
};

// compute units of the current device (256 if it cannot be asked)
int num_cus();
// dv columns per workgroup of the scans for this shape.  16-bit storage: 16 if the CUs hold all workgroups of 16, or 32.  32-bit
// storage: 32, unless that leaves a quarter of the CUs or more without a workgroup or (d = 128) the prefetched fragments of 32 columns
// do not fit the registers: then 16
int scan_dvb(const Dims &d);
// workgroups of one scan launch: (batch*head rounded up to 8) x dv / scan_dvb; packed batches: those it takes the longest
// sequence's time to run
int scan_workgroups(const Dims &d);
// Whether a scan launch keeps a second workgroup off every CU (see lds_bytes_for_one_workgroup_per_cu): where the workgroups
// of the longest sequence's length do not outnumber the CUs.  Elsewhere 16-bit storage takes the instances that fit twice.
bool scan_one_per_cu(const Dims &d);

// mode 0: forward operands, 1: reverse-pass operands, 2: both (16-bit storage: the same ones, always mode 0)
hipError_t launch_intra(const Dims &d, int mode, const IntraArgs &a, hipStream_t s);
hipError_t launch_scan_fwd(const Dims &d, const ScanFwdArgs &a, hipStream_t s);
// Dynamic LDS bytes that keep a second workgroup of `kernel` off a CU (0 if one workgroup fills more than half of the
// 160 KB already).  For launches with fewer workgroups than CUs: the dispatcher otherwise puts two of them on one CU
// and leaves other CUs empty, and two scan workgroups that share a CU take turns at everything.
size_t lds_bytes_for_one_workgroup_per_cu(const void *kernel);

// 16-bit storage (what launch_scan_fwd, launch_rebuild and launch_scan_bwd go on to)
hipError_t launch_scan_fwd16(const Dims &d, const ScanFwdArgs &a, bool rebuild, hipStream_t s);
hipError_t launch_scan_bwd16(const Dims &d, const ScanBwdArgs &a, hipStream_t s);
hipError_t launch_rebuild(const Dims &d, const RebuildArgs &a, hipStream_t s);
// the same as arguments of the forward scan's kernels
ScanFwdArgs rebuild_args(const RebuildArgs &a);
// 16-bit storage: both in one launch
hipError_t launch_rebuild_and_scan_bwd(const Dims &d, const RebuildArgs &r, const ScanBwdArgs &b, hipStream_t s);
hipError_t launch_scan_bwd(const Dims &d, const ScanBwdArgs &a, hipStream_t s);
hipError_t launch_grad(const Dims &d, const GradArgs &a, hipStream_t s);
hipError_t launch_recurrent(const Dims &d, const RecurrentArgs &a, hipStream_t s);

// One tensor of a copy between the caller's layout and padded 64-token tiles.
struct TileTensor {
    const void *full; // the caller's tensor
    void *padded;     // the padded copy
    int row_bytes;    // a multiple of 4
    uint32_t pad_word;
};

// Chunk sizes below 64 (Algorithm 1 lists C in {16, 32, 64}): every chunk of C tokens becomes one 64-token tile whose
// rows from C on are padding (TileTensor::pad_word).  expand: [B,T,H,row] -> [B, ceil(T/C) * 64, H, row];
// collect: the real rows back.
struct ChunkCopy {
    int B, T, H, C, NC, n; // NC = ceil(T / C) chunks, n tensors
    TileTensor t[12];
};
hipError_t launch_chunk_copy(const ChunkCopy &c, bool expand, hipStream_t s);

// Packed variable-length batches: writes the device tables of Dims from the entries, which travel in the kernel
// arguments, kSeqsPerLaunch at a time (seqs[first + i] = e[i], and the chunk entries of that sequence).
constexpr int kSeqsPerLaunch = 224;
struct SeqList {
    int n, first, H;
    SeqEntry e[kSeqsPerLaunch];
};
// first tokens of the sequences of a packed batch that follow another one in a merged piece, part of the list
constexpr int kStartsPerLaunch = 960; // (a kernel's arguments end at 4 KB)
struct StartList { int n, H; int t[kStartsPerLaunch]; };
// a = b = 0 at the tokens of the list, all heads ([T,H] tensors)
hipError_t launch_clear_at_starts(const StartList &l, float *a, float *b, hipStream_t s);
// dst_a = a, dst_b = b: n floats each, 16-byte aligned
hipError_t launch_copy_gates(const float *a, const float *b, float *dst_a, float *dst_b, long long n, hipStream_t s);
hipError_t launch_seq_tables(const SeqList &l, SeqEntry *seqs, ChunkEntry *chunks, hipStream_t s);

} // namespace mdn
