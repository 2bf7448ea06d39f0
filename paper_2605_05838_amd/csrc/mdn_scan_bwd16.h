// Reverse scan for 16-bit storage: the adjoint recurrence of mdn_scan_bwd.hip, chunks from last to first,
//     dV~ = Bm^T dO + (Gamma_C eta . K) dS' - (Rho_C eta . K) dM'        dV = T^T dV~
//     dS  = a_C dS' + (a . Q~)^T dO - K^T (a . dV)        dM = m_C dM' - b_C dS' - (b . Q~)^T dO + K^T (pb . dV)
// one workgroup per (sequence, head) and DVB dv columns, its waves' jobs as in mdn_scan_tiles.h, products transposed as in
// mdn_scan_fwd16.h.  K^T, Q^T, Bm^T and T^T are transposing reads of the same tiles that the forward uses: nothing is written
// to HBM a second time in another orientation for this kernel.
//
// A step has three phases, each ended by a barrier:
//   A  dV~^T of the wave's 16 tokens from the adjoints' copy, the k rows, Bm and dO, left in LDS; dO in the two scalings
//      with which it enters the states;
//   B  dV^T = dV~^T T over all tokens, left raw (the output) and in two scalings; (a . Q~)^T dO and (b . Q~)^T dO of the first 32
//      tokens into the states, whose products fill the waits of this short phase;
//   C  K^T (a . dV), K^T (pb . dV) of those tokens into the states, then both of the other 32, the new copy.
// The state adjoints thus sum in the order of mdn_scan_bwd.hip, 32 tokens of Q, then of K.  (All of Q in phase B, all of K in phase C
// is as fast, 4 x 4 096 tokens of 16 heads of 128 forward and backward 604 against 606 us, but every gradient then differs by 1e-3:
// roundings of the copies, dV~ and dV carry the last bits of a sum on from chunk to chunk.)
#pragma once
#include "mdn_scan_tiles.h"
#include "mdn_kernels.h"

namespace mdn {

// AHEAD: how many chunks in front of the chain the loads are, 2 or (two workgroups per CU: see scan_one_per_cu) 1, as far as one set
// of operands allows
// TOUCH: the operands are brought into the L2 first (LineTouch)
template <int DK, int DV, int DVB, int AHEAD, bool TOUCH = false> struct ScanBwdLds {
    typedef bf16_t T;
    typedef ATile<T, DVB, 2 * DK> TD; // the adjoints' copy, contraction over dk: dS' | dM'
    typedef ATile<T, DVB, 64> TV;     // contraction over the chunk's tokens
    // operands of AHEAD chunks; of two chunks the k tile, read from the first to the last phase, of three where there is room
    static constexpr int KSLOTS = AHEAD == 1 ? 1 : DVB == 16 || DK == 64 ? 3 : 2;
    __align__(16) T rK[KSLOTS][64 * DK];
    __align__(16) T rQ[AHEAD][64 * DK];
    __align__(16) T rT[AHEAD][4096];
    __align__(16) T rB[AHEAD][4096];
    __align__(16) T rO[AHEAD][64 * DVB];
    __align__(16) float rC[AHEAD][64 * kCoefRows];
    // what the chain leaves
    __align__(16) T sD[TD::SIZE];
    __align__(16) T sOa[TV::SIZE]; // (scale a . dO)^T
    __align__(16) T sOb[TV::SIZE]; // (-scale b . dO)^T
    __align__(16) T sDV[TV::SIZE]; // dV~^T
    __align__(16) T sR0[TV::SIZE]; // dV^T
    __align__(16) T sRa[TV::SIZE]; // (-a . dV)^T
    __align__(16) T sRb[TV::SIZE]; // (pb . dV)^T
    __align__(16) unsigned touched[TOUCH ? 128 : 4];
};

// workgroup `block` of ((BH + 7) / 8) * 8 * DV / DVB
template <int DK, int DV, int DVB, bool WHOLE, int AHEAD, bool TOUCH>
__device__ __forceinline__ void scan_bwd16(const Dims &d, const ScanBwdArgs &a, int block, ScanBwdLds<DK, DV, DVB, AHEAD, TOUCH> &lds) {
    typedef bf16_t T;
    typedef Op<T> O;
    typedef ScanBwdLds<DK, DV, DVB, AHEAD, TOUCH> L;
    typedef typename L::TD TD;
    typedef typename L::TV TV;
    constexpr int MV = DVB / 16, ND = DK / 64, G = DV / DVB, KS = DK / 32, KSLOTS = L::KSLOTS;

    int bh, blkv;
    xcd_map(block, G, bh, blkv);
    if (bh >= d.BH) return;
    const ScanSeq sq = scan_seq<WHOLE>(d, bh);
    const int dv0 = blkv * DVB, n0 = sq.n0, n1 = sq.n1;
    const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id()), w = wv & 3, w2 = wv & 1;
    const int r = lane & 15, kg = lane >> 4, i = w * 16 + r;
    // a partial last chunk (the first one here): its loads stop at the last real token
    const int ragged = !WHOLE && (sq.len & 63) ? sq.len >> 6 : -1, last = (sq.len & 63) - 1; // that chunk (or none), its last row
    auto first_token = [&](int n) { return sq.tok + (size_t)n * 64 * d.H; };
    const int turn = blkv & 3;
    TileLoad<T, 64, true> tm;
    auto request_m = [&](const void *m, int n, const T *ring, int par) {
        tm.request(static_cast<const T *>(m) + (sq.blk + n) * 4096, lds_addr(ring) + par * (4096 * (int)sizeof(T)), w2, turn);
    };

    if (wv >= 6) {
        // ---------------------------------------------------------------- stores
        StateStore<DK, DV, MV> st;
        constexpr int NS = StateStore<DK, DV, MV>::N;
        // (at the start, with nothing to store yet, these waves bring Bm and T of the first chunks)
        tm.aim(64, w2, lane, turn, 63);
        for (int ahead = 0; ahead < AHEAD && n1 - 1 - ahead >= n0; ++ahead) {
            request_m(a.Bm, n1 - 1 - ahead, lds.rB[0], ahead);
            request_m(a.Tm, n1 - 1 - ahead, lds.rT[0], ahead);
        }
        if (AHEAD == 2 && n0 + 1 < n1) wait_vm<2 * tm.COUNT>();
        else wait_vm<0>();
        [[maybe_unused]] LineTouch<DK, DV, G> touch; // (of what comes before the partial chunk)
        [[maybe_unused]] int next = n1 - 1 - AHEAD; // the chunk it is at
        if constexpr (TOUCH) touch.aim(a.k, a.q, a.dO, a.Tm, a.Bm, a.coef, sq, d.H, blkv * 2 + w2, lane, next, -1, 63);
        __syncthreads();
        for (int n = n1 - 1; n >= n0; --n) {
            T *states = static_cast<T *>(a.dstates) + (sq.blk + n) * (2 * DK * DV); // adjoints of this chunk's END states
            st.read(lds.sD, w2, lane);
            st.template put<0, NS / 2>(states, dv0, w2, lane);
            __syncthreads(); // A
            if (AHEAD == 2 && n == n1 - 1) wait_vm<NS / 2>(); // Bm and T of the second chunk are there
            st.template put<NS / 2, NS * 3 / 4>(states, dv0, w2, lane);
            __syncthreads(); // B
            store_token_rows<DV, MV, WHOLE>(static_cast<T *>(a.dv) + first_token(n) * DV + dv0, lds.sR0, !WHOLE && n == ragged ? last + 1 : 64, d.H, w2, lane);
            st.template put<NS * 3 / 4, NS>(states, dv0, w2, lane);
            if constexpr (TOUCH)
                for (; next >= n0 && next >= n - kTouchAhead; --next) touch.template chunk<-1>(next, lds_addr(lds.touched + w2 * 64));
            __syncthreads(); // C
        }
        if constexpr (TOUCH) wait_vm<0>(); // (no transfer outlives the workgroup)
    } else if (wv >= 4) {
        // ---------------------------------------------------------------- loads: two chunks ahead, as the slots become free
        const unsigned rsk = (unsigned)(d.H * DK), rsv = (unsigned)(d.H * DV);
        TileLoad<T, DK, true> tk; // (the rows of q lie as those of k)
        TileLoad<T, DVB, false> tv;
        TileLoad<float, kCoefRows, false> tc;
        tm.aim(64, w2, lane, turn, 63);
        tc.aim(kCoefRows, w2, lane, turn, 63);
        auto aim_at = [&](int rows) {
            tk.aim(rsk, w2, lane, turn, rows);
            tv.aim(rsv, w2, lane, turn, rows);
        };
        auto request_rows = [&](const void *x, int n, const T *ring, int slot) {
            tk.request(static_cast<const T *>(x) + first_token(n) * DK, lds_addr(ring) + slot * (64 * DK * (int)sizeof(T)), w2, turn);
        };
        auto request_o = [&](int n, int par) {
            tv.request(static_cast<const T *>(a.dO) + first_token(n) * DV + dv0, lds_addr(lds.rO[0]) + par * (64 * DVB * (int)sizeof(T)), w2, turn);
        };
        auto request_c = [&](int n, int par) {
            tc.request(a.coef + (sq.blk + n) * (64 * kCoefRows), lds_addr(lds.rC[0]) + par * (64 * kCoefRows * 4), w2, turn);
        };
        constexpr int NALL = 2 * tk.COUNT + 2 * tm.COUNT + tv.COUNT + tc.COUNT;
        // (only chunks that exist)
        for (int ahead = 0; ahead < AHEAD; ++ahead) {
            const int n = n1 - 1 - ahead;
            if (n < n0) break;
            aim_at(!WHOLE && n == ragged ? last : 63);
            request_rows(a.k, n, lds.rK[0], ahead);
            request_c(n, ahead);
            request_o(n, ahead);
            request_rows(a.q, n, lds.rQ[0], ahead);
        }
        if (AHEAD == 2 && n0 + 1 < n1) wait_vm<NALL - 2 * tm.COUNT>();
        else wait_vm<0>();
        __syncthreads();
        if (!WHOLE) aim_at(63); // (what is requested from here on is not the partial chunk)
        int slot = 2, par = 0;
        int n = n1 - 1;
        for (; n - AHEAD >= n0; --n) {
            const int nn = n - AHEAD;
            if (KSLOTS == 3) request_rows(a.k, nn, lds.rK[0], slot);
            if (AHEAD == 1) wait_vm<0>(); // q of this chunk is there
            __syncthreads(); // A: Bm, T, dO and the coefficients of this chunk have been read
            request_m(a.Bm, nn, lds.rB[0], par);
            request_m(a.Tm, nn, lds.rT[0], par);
            request_o(nn, par);
            request_c(nn, par);
            __syncthreads(); // B: so have k and q
            if (KSLOTS < 3) request_rows(a.k, nn, lds.rK[0], par);
            request_rows(a.q, nn, lds.rQ[0], par);
            wait_vm<AHEAD == 2 ? NALL : tk.COUNT>(); // everything of the next chunk is there (one chunk ahead: q not yet)
            slot = slot == 2 ? 0 : slot + 1;
            if (AHEAD == 2) par ^= 1;
            __syncthreads(); // C
        }
        for (; n >= n0; --n) {
            if (AHEAD == 1) wait_vm<0>();
            __syncthreads(); // A
            __syncthreads(); // B
            wait_vm<0>();
            __syncthreads(); // C
        } // (no transfer outlives the workgroup: the last step has waited for all of them)
    } else {
        // ---------------------------------------------------------------- the chain
        __builtin_amdgcn_s_setprio(3);
        ChainStates<DK, DV, MV> acc;
        acc.load(a.dS_final, a.dM_final, sq.state, w, dv0, r, kg);
        acc.publish(lds.sD, w, r, kg);
        __syncthreads();
        int slot = 0, par = 0;
        for (int n = n1 - 1; n >= n0; --n) {
            if (a.dstates_lo) acc.store_lo(static_cast<T *>(a.dstates_lo) + (sq.blk + n) * (2 * DK * DV), w, dv0, r, kg);
            const T *kc = lds.rK[slot], *qc = lds.rQ[par], *oc = lds.rO[par];
            const f32x4 c0 = *reinterpret_cast<const f32x4 *>(lds.rC[par] + i * kCoefRows);
            const f32x4 c1 = *reinterpret_cast<const f32x4 *>(lds.rC[par] + i * kCoefRows + 4);
            // ---- phase A
            f32x4 x1[MV], x2[MV], dv[MV];
            zero_acc(x1);
            zero_acc(x2);
            zero_acc(dv);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const O::Frag fk = token_tile_row_frag<DK>(kc, i, s, kg);
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    x1[mv] = O::mma(TD::frag(lds.sD, mv, s * 32, r, kg), fk, x1[mv]);
                    x2[mv] = O::mma(TD::frag(lds.sD, mv, DK + s * 32, r, kg), fk, x2[mv]);
                }
            }
            O::Frag tT[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const O::Frag bT = token_tile_col_frag<64>(lds.rB[par], w, s, r, kg);
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    // dO^T out of the rows as they are in HBM: lane 4e + c of a 16-lane group addresses the columns of MFMA rows 4c .. 4c+3
                    const T *p = oc + (s * 32 + kg * 8 + (r >> 2)) * DVB + (r & 3) * (4 * MV) + 4 * mv;
                    dv[mv] = O::mma(tr_pair(p, p + 4 * DVB), bT, dv[mv]);
                }
                tT[s] = token_tile_col_frag<64>(lds.rT[par], w, s, r, kg);
            }
            bf16x4 u[MV];
            load_cols_raw<MV>(oc + i * DVB + kg * (4 * MV), u);
            // (rows behind a partial chunk hold the last real row of q and dO: they must not reach the states.  In the other
            //  products Bm, Gamma_C and Rho_C are zero there.)
            const float real = WHOLE || n != ragged || i <= last ? d.scale : 0.f;
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                const f32x4 ow = widen4(u[mv]);
                TV::put4(lds.sOa, mv * 16 + kg * 4, i, (real * c0[COEF_A]) * ow);
                TV::put4(lds.sOb, mv * 16 + kg * 4, i, -(real * c0[COEF_B]) * ow);
                TV::put4(lds.sDV, mv * 16 + kg * 4, i, dv[mv] + c1[COEF_GC - 4] * x1[mv] - c1[COEF_RC - 4] * x2[mv]);
            }
            __syncthreads(); // A
            // ---- phase B
            f32x4 dR[MV];
            zero_acc(dR);
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) dR[mv] = O::mma(TV::frag(lds.sDV, mv, s * 32, r, kg), tT[s], dR[mv]);
            const float aC = c0[COEF_AC], bC = c1[COEF_BC - 4], mC = c1[COEF_MC - 4];
#pragma unroll
            for (int mv = 0; mv < MV; ++mv)
#pragma unroll
                for (int nd = 0; nd < ND; ++nd) {
                    const f32x4 s = acc.S[mv][nd], m = acc.M[mv][nd];
                    acc.S[mv][nd] = aC * s;
                    acc.M[mv][nd] = mC * m - bC * s;
                }
            O::Frag kT[2][ND], qT[2][ND];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int nd = 0; nd < ND; ++nd) {
                    qT[s][nd] = token_tile_col_frag<DK>(qc, w * ND + nd, s, r, kg);
                    kT[s][nd] = token_tile_col_frag<DK>(kc, w * ND + nd, s, r, kg);
                }
            auto q_into_states = [&](int s) {
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    const O::Frag fa = TV::frag(lds.sOa, mv, s * 32, r, kg), fb = TV::frag(lds.sOb, mv, s * 32, r, kg);
#pragma unroll
                    for (int nd = 0; nd < ND; ++nd) {
                        acc.S[mv][nd] = O::mma(fa, qT[s][nd], acc.S[mv][nd]);
                        acc.M[mv][nd] = O::mma(fb, qT[s][nd], acc.M[mv][nd]);
                    }
                }
            };
            q_into_states(0);
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                TV::put4(lds.sR0, mv * 16 + kg * 4, i, dR[mv]);
                TV::put4(lds.sRa, mv * 16 + kg * 4, i, -c0[COEF_A] * dR[mv]);
                TV::put4(lds.sRb, mv * 16 + kg * 4, i, c0[COEF_PB] * dR[mv]);
            }
            __syncthreads(); // B
            // ---- phase C
            auto k_into_states = [&](int s) {
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    const O::Frag fa = TV::frag(lds.sRa, mv, s * 32, r, kg), fb = TV::frag(lds.sRb, mv, s * 32, r, kg);
#pragma unroll
                    for (int nd = 0; nd < ND; ++nd) {
                        acc.S[mv][nd] = O::mma(fa, kT[s][nd], acc.S[mv][nd]);
                        acc.M[mv][nd] = O::mma(fb, kT[s][nd], acc.M[mv][nd]);
                    }
                }
            };
            k_into_states(0);
            q_into_states(1);
            k_into_states(1);
            acc.publish(lds.sD, w, r, kg);
            slot = slot == KSLOTS - 1 ? 0 : slot + 1;
            if (AHEAD == 2) par ^= 1;
            __syncthreads(); // C
        }
        acc.store(a.dS0, a.dM0, sq.state, w, dv0, r, kg);
    }
}

} // namespace mdn
