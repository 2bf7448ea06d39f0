// Forward scan and state reconstruction for 16-bit storage: the recurrence of mdn_scan_fwd.hip (Sec. 3.1 "Chunkwise Algorithm"),
//     V~ = T (V - a . (K S) + pb . (K M))        O  = diag(a) Q~ S - diag(b) Q~ M + Bm V~
//     S' = a_C S - b_C M + (diag(Gamma_C) K~)^T V~        M' = m_C M - (diag(Rho_C) K~)^T V~
// one workgroup per (sequence, head) and DVB dv columns, its waves' jobs as in mdn_scan_tiles.h.  Products are formed transposed,
// with the dv index as the MFMA row index; row 4 kg + x of tile mv stands for column dv0 + 4 MV kg + 4 mv + x.
//
// A step has three phases, each ended by a barrier:
//   A  wave w forms (K S)^T, (K M)^T, (Q S)^T, (Q M)^T for its 16 tokens in one pass over the states' copy, leaves R^T in LDS;
//   B  V~^T = R^T T^T over all tokens, left in LDS in three scalings (raw, Gamma_C eta, -Rho_C eta);
//   C  the states' update out of K^T (transposing reads of the k tile) and the scaled V~, Bm V~ for the output, the new copy.
// What a phase reads of the operands is read before the barrier in front of it.  The reconstruction (REBUILD) reads V~ and
// has the last two phases only, and stops at the last chunk's start states.
//
// What bounds it: with every CU busy (256 workgroups) the mixture of loads and stores itself; a program that only makes this
// kernel's requests takes 155-168 us at 4 x 4 096 tokens of 16 heads of 128.  With fewer workgroups or without kept states, the
// step's chain of LDS reads, products and barriers; with few workgroups, kept states and more data than the caches hold, the loads'
// latency beside the stores (LineTouch).
#pragma once
#include "mdn_scan_tiles.h"
#include "mdn_kernels.h"

namespace mdn {

// AHEAD: how many chunks in front of the chain the loads are, 2 or (two workgroups per CU: see scan_one_per_cu) 1
// QTILE: the q rows come as a tile too (two chunks of them; with 32 columns of d = 128 at the cost of the third k tile), else from HBM into
// the product waves' registers
// TOUCH: the operands are brought into the L2 first (LineTouch)
template <int DK, int DV, int DVB, bool REBUILD, int AHEAD, bool QTILE = false, bool TOUCH = false> struct ScanFwdLds {
    typedef bf16_t T;
    typedef ATile<T, DVB, 2 * DK> TS; // the states' copy, contraction over dk: S | M
    typedef ATile<T, DVB, 64> TV;     // contraction over the chunk's tokens
    // operands: AHEAD chunks, and the chain's own where a tile is read in the last phase
    static constexpr int SLOTS = AHEAD + 1;
    static constexpr int KSLOTS = QTILE && DK == 128 && DVB == 32 ? 2 : SLOTS;
    __align__(16) T rK[KSLOTS][64 * DK];
    __align__(16) T rQ[QTILE ? 2 : 1][QTILE ? 64 * DK : 8];
    __align__(16) T rT[REBUILD ? 1 : AHEAD][REBUILD ? 8 : 4096];
    __align__(16) T rB[REBUILD ? 1 : AHEAD][REBUILD ? 8 : 4096];
    __align__(16) T rV[SLOTS][64 * DVB];
    __align__(16) float rC[SLOTS][64 * kCoefRows];
    // what the chain leaves
    __align__(16) T sSt[TS::SIZE];
    __align__(16) T sRt[REBUILD ? 8 : TV::SIZE];
    __align__(16) T sV0[REBUILD ? 8 : TV::SIZE];
    __align__(16) T sVg[TV::SIZE];
    __align__(16) T sVr[TV::SIZE];
    __align__(16) T sO[REBUILD ? 8 : TV::SIZE];
    __align__(16) unsigned touched[TOUCH ? 128 : 4];
};

// workgroup `block` of ((BH + 7) / 8) * 8 * DV / DVB
template <int DK, int DV, int DVB, bool REBUILD, bool WHOLE, int AHEAD, bool QTILE, bool TOUCH>
__device__ __forceinline__ void scan_fwd16(const Dims &d, const ScanFwdArgs &a, int block, ScanFwdLds<DK, DV, DVB, REBUILD, AHEAD, QTILE, TOUCH> &lds) {
    static_assert(!(QTILE || TOUCH) || (!REBUILD && AHEAD == 2), "");
    typedef bf16_t T;
    typedef Op<T> O;
    typedef ScanFwdLds<DK, DV, DVB, REBUILD, AHEAD, QTILE, TOUCH> L;
    typedef typename L::TS TS;
    typedef typename L::TV TV;
    constexpr int MV = DVB / 16, ND = DK / 64, G = DV / DVB, KS = DK / 32, SLOTS = L::SLOTS, KSLOTS = L::KSLOTS;

    int bh, blkv;
    xcd_map(block, G, bh, blkv);
    if (bh >= d.BH) return;
    const ScanSeq sq = scan_seq<WHOLE>(d, bh);
    const int dv0 = blkv * DVB, n0 = sq.n0, n1 = sq.n1 - (REBUILD ? 1 : 0); // chunks [n0, n1) are walked
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id()), w = wv & 3, w2 = wv & 1;
    const int r = lane & 15, kg = lane >> 4, i = w * 16 + r;
    // a partial last chunk: its loads stop at the last real token
    const int ragged = !WHOLE && (sq.len & 63) ? sq.len >> 6 : -1, last = (sq.len & 63) - 1; // that chunk (or none), its last row
    auto first_token = [&](int n) { return sq.tok + (size_t)n * 64 * d.H; };
    const int turn = blkv & 3;
    TileLoad<T, 64, true> tm;
    constexpr int NM = REBUILD ? 0 : tm.COUNT;
    auto request_m = [&](const void *m, int n, const T *ring, int par) {
        if constexpr (!REBUILD) tm.request(static_cast<const T *>(m) + (sq.blk + n) * 4096, lds_addr(ring) + par * (4096 * (int)sizeof(T)), w2, turn);
    };

    if (wv >= 6) {
        // ---------------------------------------------------------------- stores
        auto rows_of = [&](int n) { return !WHOLE && n == ragged ? last + 1 : 64; };
        StateStore<DK, DV, MV> st;
        constexpr int NS = StateStore<DK, DV, MV>::N;
        // (at the start, with nothing to store yet, these waves bring T and Bm of the first chunks)
        tm.aim(64, w2, lane, turn, 63);
        for (int ahead = 0; ahead < AHEAD && n0 + ahead < n1; ++ahead) {
            request_m(a.Tm, n0 + ahead, lds.rT[0], ahead);
            request_m(a.Bm, n0 + ahead, lds.rB[0], ahead);
        }
        if (AHEAD == 2 && n0 + 1 < n1) wait_vm<2 * NM>();
        else wait_vm<0>();
        [[maybe_unused]] LineTouch<DK, DV, G> touch;
        [[maybe_unused]] int next = n0 + AHEAD; // the chunk it is at
        if constexpr (TOUCH) touch.aim(a.k, a.q, a.v, a.Tm, a.Bm, a.coef, sq, d.H, blkv * 2 + w2, lane, next, ragged, last);
        __syncthreads();
        if (QTILE) __syncthreads();
        for (int n = n0;; ++n) {
            if (!REBUILD && n == n1) break;
            T *states = static_cast<T *>(a.states_saved) + (sq.blk + n) * (2 * DK * DV); // this chunk's start states
            if (a.states_saved) st.read(lds.sSt, w2, lane);
            if (!REBUILD && n > n0) store_token_rows<DV, MV, WHOLE>(static_cast<T *>(a.o) + first_token(n - 1) * DV + dv0, lds.sO, 64, d.H, w2, lane);
            if (a.states_saved) st.template put<0, NS / 2>(states, dv0, w2, lane);
            if (REBUILD && n == n1) { // the start states of the last chunk
                st.template put<NS / 2, NS>(states, dv0, w2, lane);
                break;
            }
            if (!REBUILD) __syncthreads(); // A
            if (!REBUILD && AHEAD == 2 && n == n0) { // T and Bm of the second chunk are there
                if (a.states_saved) wait_vm<NS / 2>();
                else wait_vm<0>();
            }
            if (a.states_saved) st.template put<NS / 2, NS * 3 / 4>(states, dv0, w2, lane);
            __syncthreads(); // B
            if (!REBUILD && a.vt_saved)
                store_token_rows<DV, MV, WHOLE>(static_cast<T *>(a.vt_saved) + first_token(n) * DV + dv0, lds.sV0, rows_of(n), d.H, w2, lane);
            if (a.states_saved) st.template put<NS * 3 / 4, NS>(states, dv0, w2, lane);
            if constexpr (TOUCH)
                for (; next < n1 && next <= n + kTouchAhead; ++next) touch.template chunk<1>(next, lds_addr(lds.touched + w2 * 64));
            __syncthreads(); // C
        }
        if (!REBUILD) store_token_rows<DV, MV, WHOLE>(static_cast<T *>(a.o) + first_token(n1 - 1) * DV + dv0, lds.sO, rows_of(n1 - 1), d.H, w2, lane);
        if constexpr (TOUCH) wait_vm<0>(); // (no transfer outlives the workgroup)
    } else if (wv >= 4) {
        // ---------------------------------------------------------------- loads
        const unsigned rsk = (unsigned)(d.H * DK), rsv = (unsigned)(d.H * DV);
        TileLoad<T, DK, true> tk;
        TileLoad<T, DVB, false> tv;
        TileLoad<float, kCoefRows, false> tc;
        constexpr int NK = tk.COUNT, NQ = QTILE ? NK : 0, NV = tv.COUNT + tc.COUNT;
        tm.aim(64, w2, lane, turn, 63);
        tc.aim(kCoefRows, w2, lane, turn, 63);
        tk.aim(rsk, w2, lane, turn, 63);
        tv.aim(rsv, w2, lane, turn, 63);
        auto aim_at = [&](int n) {
            if (!WHOLE && n == ragged) {
                tk.aim(rsk, w2, lane, turn, last);
                tv.aim(rsv, w2, lane, turn, last);
            }
        };
        auto request_k = [&](int n, int slot) {
            tk.request(static_cast<const T *>(a.k) + first_token(n) * DK, lds_addr(lds.rK[0]) + slot * (64 * DK * (int)sizeof(T)), w2, turn);
        };
        auto request_q = [&](int n, int slot) { // (the rows of q lie as those of k)
            if constexpr (QTILE)
                tk.request(static_cast<const T *>(a.q) + first_token(n) * DK, lds_addr(lds.rQ[0]) + slot * (64 * DK * (int)sizeof(T)), w2, turn);
        };
        auto request_v = [&](int n, int slot) { // V (V~) and the coefficients
            tv.request(static_cast<const T *>(REBUILD ? a.vt_saved : a.v) + first_token(n) * DV + dv0,
                       lds_addr(lds.rV[0]) + slot * (64 * DVB * (int)sizeof(T)), w2, turn);
            tc.request(a.coef + (sq.blk + n) * (64 * kCoefRows), lds_addr(lds.rC[0]) + slot * (64 * kCoefRows * 4), w2, turn);
        };
        // (only chunks that exist: a chunk more than there are, requested again, is a third of a three-chunk call's traffic)
        for (int ahead = 0; ahead < AHEAD; ++ahead) {
            const int n = n0 + ahead;
            if (n >= n1) break;
            aim_at(n);
            request_k(n, ahead);
            request_q(n, ahead);
            request_v(n, ahead);
        }
        if constexpr (AHEAD == 2) {
            // With a q tile the k tile is requested in the last phase, the longest one, which with three slots is three chunks ahead:
            // 16 requests, k and q, at the start of a step kept its first barrier waiting (32 768 tokens of 16 heads of 128, forward
            // 721 us so, 662 now).
            constexpr int KAHEAD = QTILE ? KSLOTS : 2;
            if (KAHEAD == 3 && n0 + 2 < n1) {
                aim_at(n0 + 2);
                request_k(n0 + 2, 2);
            }
            if (KAHEAD == 3 && n0 + 2 < n1) wait_vm<2 * NK + NQ + NV>();
            else if (n0 + 1 < n1) wait_vm<NK + NQ + NV>();
            else wait_vm<0>();
            __syncthreads();
            if (QTILE) __syncthreads(); // the first chunk's q has been read
            int slot = 2, par = 0, kslot = 0;
            int n = n0;
            for (; n + 2 < n1; ++n) {
                const int nn = n + 2;
                aim_at(nn);
                if (!QTILE) request_k(nn, slot);
                request_q(nn, par); // (q of this chunk has been read)
                if (!REBUILD) __syncthreads(); // A: T of this chunk has been read
                request_m(a.Tm, nn, lds.rT[0], par);
                request_v(nn, slot);
                wait_vm<(KAHEAD == 3 || !QTILE ? NK : 0) + NQ + NM + NV>(); // everything of the next chunk is there
                __syncthreads(); // B: so have Bm and k
                request_m(a.Bm, nn, lds.rB[0], par);
                if (QTILE && n + KAHEAD < n1) {
                    if (KAHEAD == 3) aim_at(n + 3);
                    request_k(n + KAHEAD, KAHEAD == 3 ? kslot : par);
                }
                slot = slot == 2 ? 0 : slot + 1;
                kslot = kslot == 2 ? 0 : kslot + 1;
                par ^= 1;
                __syncthreads(); // C
            }
            for (; n < n1; ++n) {
                if (!REBUILD) __syncthreads(); // A
                wait_vm<0>();
                __syncthreads(); // B
                __syncthreads(); // C
            }
        } else {
            // (the chain reads the rows of a chunk at the end of the step before, T in phase A and Bm in phase B)
            auto request_rows = [&](int n) {
                if (n >= n1) return;
                aim_at(n);
                request_k(n, (n - n0) & 1);
                request_v(n, (n - n0) & 1);
            };
            wait_vm<0>();
            __syncthreads();
            request_rows(n0 + 1);
            for (int n = n0; n < n1; ++n) {
                const bool next = n + 1 < n1;
                if (!REBUILD) {
                    if (next) wait_vm<NK + NV>(); // Bm of this chunk is there
                    else wait_vm<0>();
                    __syncthreads(); // A: T of this chunk has been read
                    if (next) request_m(a.Tm, n + 1, lds.rT[0], 0);
                }
                wait_vm<NM>(); // the rows of the next chunk are there (nothing is outstanding if there is none)
                __syncthreads(); // B: this chunk's rows and Bm have been read
                if (next) request_m(a.Bm, n + 1, lds.rB[0], 0);
                request_rows(n + 2);
                if (!REBUILD) {
                    if (n + 2 < n1) wait_vm<NM + NK + NV>(); // T of the next chunk is there
                    else wait_vm<NM>();
                }
                __syncthreads(); // C
            }
        } // (no transfer outlives the workgroup: the last step has waited for all of them)
    } else {
        // ---------------------------------------------------------------- the chain
        __builtin_amdgcn_s_setprio(3);
        // the q rows: out of their tile with what a step needs first, or, without a place in LDS, from HBM into registers, requested when
        // those of the chunk before have been used
        struct QRows { O::Frag f[KS]; };
        auto load_q = [&](int n, QRows &q) {
            if constexpr (!REBUILD && !QTILE) {
                const T *Qg = static_cast<const T *>(a.q) + first_token(n) * DK;
                const unsigned it = (unsigned)((!WHOLE && n == ragged ? min(i, last) : i) * d.H);
#pragma unroll
                for (int s = 0; s < KS; ++s) q.f[s] = O::load(at32(Qg, it * DK + kg * 8 + s * 32));
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        QRows q;
        load_q(n0, q);
        ChainStates<DK, DV, MV> acc;
        acc.load(a.S0, a.M0, sq.state, w, dv0, r, kg);
        acc.publish(lds.sSt, w, r, kg);
        if (REBUILD && a.states_lo) acc.store_lo(static_cast<T *>(a.states_lo) + (sq.blk + n0) * (2 * DK * DV), w, dv0, r, kg);
        __syncthreads();
        // what a step needs first, read one barrier early
        O::Frag fk[KS];
        f32x4 c0, c1;
        bf16x4 u[MV];
        int slot = 0, par = 0;
        auto k_tile = [&]() -> const T * { return lds.rK[KSLOTS == SLOTS ? slot : par]; };
        auto first_reads = [&]() {
            if constexpr (!REBUILD) {
#pragma unroll
                for (int s = 0; s < KS; ++s) fk[s] = token_tile_row_frag<DK>(k_tile(), i, s, kg);
            }
            if constexpr (QTILE) {
#pragma unroll
                for (int s = 0; s < KS; ++s) q.f[s] = token_tile_row_frag<DK>(lds.rQ[par], i, s, kg);
            }
            c0 = *reinterpret_cast<const f32x4 *>(lds.rC[slot] + i * kCoefRows);
            c1 = *reinterpret_cast<const f32x4 *>(lds.rC[slot] + i * kCoefRows + 4);
            load_cols_raw<MV>(lds.rV[slot] + i * DVB + kg * (4 * MV), u);
        };
        first_reads();
        // (the tile of the first chunk's q is requested anew at the start of its step; later ones are read in front of a barrier anyway.
        //  The first of these requests behind A instead, by a branch in the loading waves: 88.8 instead of 86.2 us for 4 096 tokens of 16 heads
        //  of 128.)
        if (QTILE) __syncthreads();
        // (one copy of a step: two or three, for q registers two chunks ahead, took 92.0 instead of 89.2 us for 16 x 512 tokens of 16
        //  heads of 128 and 14.4 instead of 13.9 for 1 x 128)
        for (int n = n0; n < n1; ++n) {
            f32x4 o[MV];
            bf16x4 vb[MV]; // V~ in storage form
            O::Frag kt[2][ND], bm[2];
            auto read_kt = [&]() {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int nd = 0; nd < ND; ++nd) kt[s][nd] = token_tile_col_frag<DK>(k_tile(), w * ND + nd, s, r, kg);
            };
            if constexpr (!REBUILD) {
                f32x4 x1[MV], x2[MV], os[MV], om[MV], v[MV];
                zero_acc(x1);
                zero_acc(x2);
                zero_acc(os);
                zero_acc(om);
                zero_acc(v);
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int mv = 0; mv < MV; ++mv) {
                        const O::Frag fs = TS::frag(lds.sSt, mv, s * 32, r, kg), fm = TS::frag(lds.sSt, mv, DK + s * 32, r, kg);
                        x1[mv] = O::mma(fs, fk[s], x1[mv]);
                        x2[mv] = O::mma(fm, fk[s], x2[mv]);
                        os[mv] = O::mma(fs, q.f[s], os[mv]);
                        om[mv] = O::mma(fm, q.f[s], om[mv]);
                    }
                O::Frag tm[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) tm[s] = token_tile_row_frag<64>(lds.rT[par], i, s, kg);
#pragma unroll
                for (int mv = 0; mv < MV; ++mv)
                    TV::put4(lds.sRt, mv * 16 + kg * 4, i, widen4(u[mv]) - c0[COEF_A] * x1[mv] + c0[COEF_PB] * x2[mv]);
                if (n + 1 < n1) load_q(n + 1, q);
                __syncthreads(); // A
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int mv = 0; mv < MV; ++mv) v[mv] = O::mma(TV::frag(lds.sRt, mv, s * 32, r, kg), tm[s], v[mv]);
#pragma unroll
                for (int s = 0; s < 2; ++s) bm[s] = token_tile_row_frag<64>(lds.rB[par], i, s, kg);
                read_kt();
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    o[mv] = d.scale * (c0[COEF_A] * os[mv] - c0[COEF_B] * om[mv]);
                    vb[mv] = narrow4<T>(v[mv]);
                    TV::put4_raw(lds.sV0, mv * 16 + kg * 4, i, vb[mv]);
                }
            } else {
                read_kt();
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) vb[mv] = u[mv];
            }
            const float aC = c0[COEF_AC], bC = c1[COEF_BC - 4], mC = c1[COEF_MC - 4];
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                const f32x4 vt = widen4_packed(vb[mv]);
                TV::put4(lds.sVg, mv * 16 + kg * 4, i, c1[COEF_GC - 4] * vt);
                TV::put4(lds.sVr, mv * 16 + kg * 4, i, -c1[COEF_RC - 4] * vt);
#pragma unroll
                for (int nd = 0; nd < ND; ++nd) {
                    acc.S[mv][nd] = aC * acc.S[mv][nd] - bC * acc.M[mv][nd];
                    acc.M[mv][nd] = mC * acc.M[mv][nd];
                }
            }
            __syncthreads(); // B
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    const O::Frag fg = TV::frag(lds.sVg, mv, s * 32, r, kg), fr = TV::frag(lds.sVr, mv, s * 32, r, kg);
#pragma unroll
                    for (int nd = 0; nd < ND; ++nd) {
                        acc.S[mv][nd] = O::mma(fg, kt[s][nd], acc.S[mv][nd]);
                        acc.M[mv][nd] = O::mma(fr, kt[s][nd], acc.M[mv][nd]);
                    }
                }
            if constexpr (!REBUILD) {
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int mv = 0; mv < MV; ++mv) o[mv] = O::mma(TV::frag(lds.sV0, mv, s * 32, r, kg), bm[s], o[mv]);
            }
            slot = slot == SLOTS - 1 ? 0 : slot + 1;
            if (AHEAD == 2) par ^= 1;
            // (the branch keeps what the next step needs behind this one's products, also where it is always taken: 4 x 2 048 tokens of
            //  16 heads of 128, forward 83.9 us without it, 82.2 with it; d = 64 is faster with both interleaved, 1 x 2 048 of 16
            //  heads 40.3 us with it, 38.3 without)
            if (REBUILD || DK == 64 || n + 1 < n1) {
                first_reads();
                acc.publish(lds.sSt, w, r, kg);
            }
            if constexpr (!REBUILD) {
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) TV::put4(lds.sO, mv * 16 + kg * 4, i, o[mv]);
            } else if (a.states_lo) {
                acc.store_lo(static_cast<T *>(a.states_lo) + (sq.blk + n + 1) * (2 * DK * DV), w, dv0, r, kg);
            }
            __syncthreads(); // C
        }
        if (!REBUILD) acc.store(a.S_final, a.M_final, sq.state, w, dv0, r, kg);
    }
}

} // namespace mdn
