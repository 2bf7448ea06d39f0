// Sequential inter-chunk propagation of the state S and the momentum M (forward) for 32-bit storage (16-bit: mdn_scan_fwd16.h), Sec. 3.1
// "Chunkwise Algorithm":
//     V~  = U - Y S + Z M                      with U = T V, Y = T diag(a^-) P, Z = T diag(b^-) P, P = alpha K
//         = T (V - a . (K S) + pb . (K M))     alpha_i a_{i-1} = a_i, pb_i = alpha_i b_{i-1}  (T pulled out:
//                                              U, Y, Z are never formed, the scan applies T itself)
//     O   = diag(a) Q~ S - diag(b) Q~ M + Bm V~
//     S'  = a_C S - b_C M + (diag(Gamma_C) K~)^T V~
//     M'  = m_C M - (diag(Rho_C) K~)^T V~
// Every dv column of S, M, V~, O evolves independently, so one workgroup owns DVB columns of one
// (batch, head) and walks the chunks in order: grid = batch*head x dv/DVB, all workgroups of one
// (batch, head) on the same XCD so that the chunk operands they share are served by one L2.
//
// Inside a workgroup (4 waves) every product is formed TRANSPOSED, with the dv index as the MFMA
// row index: an accumulator lane then holds 4 consecutive dv of one token (or of one dk row), which
// is 8 contiguous bytes of V, V~, O and of the saved states in HBM.  Row m = 4 kg + x of MFMA tile mv stands
// for column dv0 + kg*4*MV + 4 mv + x of the workgroup's DVB = 16 MV columns, so that the MV tiles of a lane
// are neighbours in HBM; inside LDS the tiles keep
// their own order (row mv*16 + m), which no one outside the workgroup sees.
//   S^T, M^T live in fp32 accumulators (wave w owns dk columns [w*dk/4, (w+1)*dk/4)); a storage-type
//   copy sits in LDS (rows dv, contraction index dk | dk: see ATile) and is the A operand of the dk-contractions of stage 1a
//   (wave w owns tokens 16w..16w+15): (K S)^T, (K M)^T and the two inter-chunk read-outs.
//   R^T = (V - a.(K S) + pb.(K M))^T goes to LDS (rows dv, contraction index token); stage 1b contracts it over ALL
//   tokens with the wave's rows of T: V~^T, which goes to LDS the same way in three scalings (raw, Gamma_C eta,
//   -Rho_C eta): the A operand of the token-contractions of stage 2 (intra-chunk output, state update).
//   Scalings along a contraction index are folded into those copies, so the B operands are raw rows of
//   K, Q, T, Bm, K^T straight from HBM.
// Three barriers per chunk.  Nothing a chunk reads from HBM depends on the state, so all of a chunk's
// fragments, its V tile and its coefficients are requested one whole chunk ahead; the serial chain then
// only waits on LDS and MFMA latency.
#include "mdn_device.h"
#include "mdn_kernels.h"
#include "mdn_seq.h"

namespace mdn {

namespace {

static_assert(kCoefRows == kCoefBlockCols, "device-side and host-side view of the coefficient block");

// Operands of one chunk held by one lane.
template <typename T, int DK, int MV> struct ChunkOps {
    typedef Op<T> O;
    static constexpr int KS = DK / O::KSTEP, KS2 = 64 / O::KSTEP, ND = DK / 64;
    typename O::Frag kr[KS];              // stage 1: rows (token i0 + r) of K
    typename O::Frag q[KS];               // stage 1: rows of Q
    typename O::Frag tm[KS2];             // stage 1: row i0 + r of T = (I + A)^-1
    typename O::Frag bm[KS2];             // stage 2: Bm row i0 + r
    typename O::Frag kt[ND][KS2];         // stage 2: K^T rows (dk) of this wave's state columns
    // (everything here is kept exactly as loaded: arithmetic on a freshly loaded value would make the wave wait
    //  for it, and for every load issued before it, at fetch time instead of one chunk later)
    typename Raw4<T>::type u[MV];         // V[token i0 + r][4 MV consecutive dv] (V~ in reconstruction), storage form
    f32x4 c0, c1;                         // the token's coefficient row (COEF_*)
};

// The operands of one chunk are requested in portions (P = 0..4) spread over the work on the previous
// chunk: a wave that issues them all at once sits at the issue until the memory pipeline has taken them
// (the time to move a chunk's operands into the CU), with its matrix work waiting behind.
// itok: this lane's token of a chunk, in token rows (i * H; in a partial chunk no further than the last real token).
template <typename T, int DK, int DV, int DVB, bool REBUILD, int P>
__device__ __forceinline__ void fetch_part(ChunkOps<T, DK, DVB / 16> &c, const Dims &d, const ScanFwdArgs &a, const ScanSeq &sq,
                                           int n, int dv0, unsigned itok) {
    typedef Op<T> O;
    typedef ChunkOps<T, DK, DVB / 16> CO;
    const int lane = lane_id(), w = wave_id() & 3, r = lane & 15, kg = lane >> 4, i = w * 16 + r;
    // every address is a wave-uniform 64-bit base (chunk, batch, head: scalar arithmetic) plus a 32-bit lane offset that
    // does not change from chunk to chunk (at32: one address register per access, no vector 64-bit adds)
    const size_t blk = sq.blk + n;
    const size_t tok0 = sq.tok + (size_t)n * 64 * d.H; // the chunk's first token of this head
    if (P == 0) {
        // (through the vector path on purpose: a scalar load would share its wait counter with the LDS reads and
        //  make the first of those wait for memory)
        const float *coef = a.coef + blk * (kCoefRows * 64);
        c.c0 = *reinterpret_cast<const f32x4 *>(at32(coef, (unsigned)(i * kCoefRows)));
        c.c1 = *reinterpret_cast<const f32x4 *>(at32(coef, (unsigned)(i * kCoefRows + 4)));
        // the forward reads V, the reconstruction the saved V~
        const T *vs = static_cast<const T *>(REBUILD ? a.vt_saved : a.v) + tok0 * DV + dv0;
        load_cols_raw<DVB / 16>(at32(vs, itok * DV + kg * (DVB / 4)), c.u);
    }
    if (P == 1 && !REBUILD) {
        const T *Qg = static_cast<const T *>(a.q) + tok0 * DK;
#pragma unroll
        for (int s = 0; s < CO::KS; ++s) c.q[s] = O::load(at32(Qg, itok * DK + kg * O::EPL + s * O::KSTEP));
    }
    if (P == 2) {
        const T *KTg = static_cast<const T *>(a.KT) + blk * (DK * 64);
#pragma unroll
        for (int nd = 0; nd < CO::ND; ++nd)
#pragma unroll
            for (int s = 0; s < CO::KS2; ++s)
                c.kt[nd][s] = O::load(at32(KTg, (unsigned)kblk<T>(DK, (w * CO::ND + nd) * 16 + r, s * O::KSTEP + kg * O::EPL)));
    }
    if (P == 3 && !REBUILD) {
        const T *Bg = static_cast<const T *>(a.Bm) + blk * 4096, *Tg = static_cast<const T *>(a.Tm) + blk * 4096;
#pragma unroll
        for (int s = 0; s < CO::KS2; ++s) {
            c.tm[s] = O::load(at32(Tg, (unsigned)kblk<T>(64, i, s * O::KSTEP + kg * O::EPL)));
            c.bm[s] = O::load(at32(Bg, (unsigned)kblk<T>(64, i, s * O::KSTEP + kg * O::EPL)));
        }
    }
    if (P == 4 && !REBUILD) {
        const T *Kg = static_cast<const T *>(a.k) + tok0 * DK;
#pragma unroll
        for (int s = 0; s < CO::KS; ++s) c.kr[s] = O::load(at32(Kg, itok * DK + kg * O::EPL + s * O::KSTEP));
    }
    __builtin_amdgcn_sched_barrier(0); // the portion leaves here, not where the scheduler would gather the loads
}

template <typename T, int DK, int DV, int DVB, bool REBUILD>
__device__ __forceinline__ void fetch_chunk(ChunkOps<T, DK, DVB / 16> &c, const Dims &d, const ScanFwdArgs &a,
                                            const ScanSeq &sq, int n, int dv0, unsigned itok) {
    fetch_part<T, DK, DV, DVB, REBUILD, 0>(c, d, a, sq, n, dv0, itok);
    fetch_part<T, DK, DV, DVB, REBUILD, 4>(c, d, a, sq, n, dv0, itok);
    fetch_part<T, DK, DV, DVB, REBUILD, 1>(c, d, a, sq, n, dv0, itok);
    fetch_part<T, DK, DV, DVB, REBUILD, 3>(c, d, a, sq, n, dv0, itok);
    fetch_part<T, DK, DV, DVB, REBUILD, 2>(c, d, a, sq, n, dv0, itok);
}

// accumulator element x of tile (mv, nd) of wave w is S[dk = (w*ND + nd)*16 + r][dv = mv*16 + kg*4 + x]
template <typename T, int DK, int MV>
__device__ __forceinline__ void publish_state(T *sSt, const f32x4 (&accS)[MV][DK / 64], const f32x4 (&accM)[MV][DK / 64]) {
    typedef ATile<T, MV * 16, 2 * DK> TS;
    const int r = lane_id() & 15, kg = lane_id() >> 4, w = wave_id();
#pragma unroll
    for (int mv = 0; mv < MV; ++mv)
#pragma unroll
        for (int nd = 0; nd < DK / 64; ++nd) {
            const int dk = (w * (DK / 64) + nd) * 16 + r;
            TS::put4(sSt, mv * 16 + kg * 4, dk, accS[mv][nd]);
            TS::put4(sSt, mv * 16 + kg * 4, DK + dk, accM[mv][nd]);
        }
}

// REBUILD = false: full forward scan.  REBUILD = true: state reconstruction from saved V~ only
// (the update lines), writing the chunk-start states.
// WHOLE: see whole_chunks.
template <typename T, int DK, int DV, int DVB, bool REBUILD, bool WHOLE>
__global__ __launch_bounds__(kThreads) void scan_fwd_kernel(Dims d, ScanFwdArgs a) {
    typedef Op<T> O;
    typedef ChunkOps<T, DK, DVB / 16> CO;
    constexpr int MV = DVB / 16, ND = DK / 64, G = DV / DVB;
    // the A operands that the workgroup builds itself (rows = dv; see ATile for how they sit in LDS)
    typedef ATile<T, DVB, 2 * DK> TS; // state copy, contraction over dk: S | M
    typedef ATile<T, DVB, 64> TV;     // contraction over the chunk's tokens
    __shared__ __align__(16) T sSt[TS::SIZE];
    __shared__ __align__(16) T sRt[REBUILD ? 8 : TV::SIZE]; // R^T = (V - a.(K S) + pb.(K M))^T, all 64 tokens
    __shared__ __align__(16) T sV0[TV::SIZE];
    __shared__ __align__(16) T sVg[TV::SIZE];
    __shared__ __align__(16) T sVr[TV::SIZE];

    int bh, blkv;
    xcd_map(blockIdx.x, G, bh, blkv);
    if (bh >= d.BH) return;
    const ScanSeq sq = scan_seq<WHOLE>(d, bh);
    const int dv0 = blkv * DVB;
    const int lane = lane_id(), w = wave_id(), r = lane & 15, kg = lane >> 4, i = w * 16 + r;
    // a partial last chunk: its loads stop at the last real token
    const int ragged = !WHOLE && (sq.len & 63) ? sq.len >> 6 : -1, last = (sq.len & 63) - 1; // that chunk (or none), its last row
    const unsigned iH = (unsigned)(i * d.H);
    unsigned itok = iH;

    if (!WHOLE && sq.n0 == ragged) itok = (unsigned)(min(i, last) * d.H);

    f32x4 accS[MV][ND], accM[MV][ND];
#pragma unroll
    for (int mv = 0; mv < MV; ++mv)
#pragma unroll
        for (int nd = 0; nd < ND; ++nd) {
            const size_t g = (sq.state * DK + (w * ND + nd) * 16 + r) * DV + dv0 + kg * (4 * MV) + mv * 4;
            accS[mv][nd] = a.S0 ? *reinterpret_cast<const f32x4 *>(a.S0 + g) : f32x4{0.f, 0.f, 0.f, 0.f};
            accM[mv][nd] = a.M0 ? *reinterpret_cast<const f32x4 *>(a.M0 + g) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    if (!REBUILD) publish_state<T, DK, MV>(sSt, accS, accM);
    __syncthreads();

    // The chunk-start states leave for HBM out of a copy in registers.  Forward scan: made at the end of the step that produced
    // them, for the LDS copy and for HBM alike, stored in one burst.  Reconstruction, which does little else than store: in 8
    // portions spread over the step.
    constexpr int NS = 2 * ND; // vector stores per lane: S and M, ND rows, MV * 4 consecutive columns each
    typename Raw4<T>::type sv[NS][MV];
    // sv: the states in storage form
    auto narrow_states = [&]() {
#pragma unroll
        for (int nd = 0; nd < ND; ++nd)
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                sv[2 * nd][mv] = narrow4<T>(accS[mv][nd]);
                sv[2 * nd + 1][mv] = narrow4<T>(accM[mv][nd]);
            }
    };
    // portion PORTION of the stores of sv as the start states of chunk block sblk
    size_t sblk = 0;
    auto emit_states = [&](auto PORTION) {
        if (!a.states_saved) return;
        T *st = static_cast<T *>(a.states_saved) + sblk * (2 * DK * DV);
        static_for<NS>([&](auto IDX) {
            constexpr int idx = decltype(IDX)::value, nd = idx >> 1;
            if ((REBUILD ? idx * 8 / NS : 0) == decltype(PORTION)::value) {
                // (dv0 is a multiple of 16: the workgroup's first column block is part of the uniform base)
                const unsigned off = (unsigned)vblk(DK, (w * ND + nd) * 16 + r, kg * (4 * MV));
                const size_t base = ((idx & 1) ? DK * DV : 0) + vblk(DK, 0, dv0);
                store_cols_raw<MV>(at32(st + base, off), sv[idx]);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    // one chunk: its operands are in `cur`; those of the next chunk go on their way into `nxt`, portion by portion.
    if constexpr (!REBUILD) {
        if (a.states_saved) { // the start states of the first chunk: what came in
            narrow_states();
            sblk = sq.blk + sq.n0;
            emit_states(std::integral_constant<int, 0>{});
        }
    }
    auto step = [&](int n, const CO &cur, CO &nxt) {
        const size_t blk = sq.blk + n;
        const size_t tok0 = sq.tok + (size_t)n * 64 * d.H; // (uniform base + 32-bit lane offset, as in fetch_part)
        const int nn = (n + 1 < sq.n1) ? n + 1 : n;
        const int rows = !WHOLE && n == ragged ? last + 1 : 64; // tokens of this chunk: their outputs are stored
        if (!WHOLE && nn == ragged) itok = (unsigned)(min(i, last) * d.H); // (the chunk requested from here on is the partial one)
        fetch_part<T, DK, DV, DVB, REBUILD, 0>(nxt, d, a, sq, nn, dv0, itok);

        sblk = blk;
        auto emit_in_step = [&](auto PORTION) {
            if constexpr (REBUILD) emit_states(PORTION);
        };
        if constexpr (REBUILD) {
            if (a.states_saved) narrow_states();
        }
        emit_in_step(std::integral_constant<int, 0>{});

        fetch_part<T, DK, DV, DVB, REBUILD, 4>(nxt, d, a, sq, nn, dv0, itok);
        emit_in_step(std::integral_constant<int, 1>{});
        // ---------------- stage 1: R^T = (V - a.(K S) + pb.(K M))^T and the inter-chunk read-outs for token i,
        //                  then V~^T = R^T T^T over all 64 tokens
        f32x4 accO[MV], vt[MV]; // vt = V~ rounded to the storage type
        typename Raw4<T>::type vb[MV]; // (the same in storage form: narrowed once, for HBM, for LDS and for vt)
        if (!REBUILD) {
            f32x4 x1[MV], x2[MV], accOS[MV], accOM[MV];
            zero_acc(x1);
            zero_acc(x2);
            zero_acc(accOS);
            zero_acc(accOM);
#pragma unroll
            for (int s = 0; s < CO::KS; ++s) {
                const typename O::Frag fk = cur.kr[s];
#pragma unroll
                for (int mv = 0; mv < MV; ++mv) {
                    const typename O::Frag fs = TS::frag(sSt, mv, s * O::KSTEP, r, kg);
                    const typename O::Frag fm = TS::frag(sSt, mv, DK + s * O::KSTEP, r, kg);
                    x1[mv] = O::mma(fs, fk, x1[mv]);
                    accOS[mv] = O::mma(fs, cur.q[s], accOS[mv]);
                    x2[mv] = O::mma(fm, fk, x2[mv]);
                    accOM[mv] = O::mma(fm, cur.q[s], accOM[mv]);
                }
            }
            fetch_part<T, DK, DV, DVB, REBUILD, 1>(nxt, d, a, sq, nn, dv0, itok);
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                accO[mv] = d.scale * (cur.c0[COEF_A] * accOS[mv] - cur.c0[COEF_B] * accOM[mv]);
                TV::put4(sRt, mv * 16 + kg * 4, i, widen4(cur.u[mv]) - cur.c0[COEF_A] * x1[mv] + cur.c0[COEF_PB] * x2[mv]);
            }
            __syncthreads();
            f32x4 accV[MV];
            zero_acc(accV);
#pragma unroll
            for (int s = 0; s < CO::KS2; ++s)
#pragma unroll
                for (int mv = 0; mv < MV; ++mv)
                    accV[mv] = O::mma(TV::frag(sRt, mv, s * O::KSTEP, r, kg), cur.tm[s], accV[mv]);
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                vb[mv] = narrow4<T>(accV[mv]);
                vt[mv] = widen4_packed(vb[mv]);
            }
            if (a.vt_saved) {
                RowStore<T, WHOLE>(static_cast<T *>(a.vt_saved) + tok0 * DV + dv0, rows, d.H * DV, DVB).template put_cols<MV>(iH * DV + kg * (4 * MV), vb);
            }
        } else {
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                vb[mv] = cur.u[mv];
                vt[mv] = widen4(cur.u[mv]);
            }
        }
        emit_in_step(std::integral_constant<int, 2>{});
        // V~^T to LDS in the three scalings of stage 2
#pragma unroll
        for (int mv = 0; mv < MV; ++mv) {
            if (!REBUILD) TV::put4_raw(sV0, mv * 16 + kg * 4, i, vb[mv]);
            TV::put4(sVg, mv * 16 + kg * 4, i, cur.c1[COEF_GC - 4] * vt[mv]);
            TV::put4(sVr, mv * 16 + kg * 4, i, -cur.c1[COEF_RC - 4] * vt[mv]);
        }
        emit_in_step(std::integral_constant<int, 3>{});
        __syncthreads();

        // ---------------- stage 2: intra-chunk output and the state update
        fetch_part<T, DK, DV, DVB, REBUILD, 2>(nxt, d, a, sq, nn, dv0, itok);
        emit_in_step(std::integral_constant<int, 4>{});
        const float aC = cur.c0[COEF_AC], bC = cur.c1[COEF_BC - 4], mC = cur.c1[COEF_MC - 4];
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
            for (int nd = 0; nd < ND; ++nd) {
                accS[mv][nd] = aC * accS[mv][nd] - bC * accM[mv][nd];
                accM[mv][nd] = mC * accM[mv][nd];
            }
#pragma unroll
        for (int s = 0; s < CO::KS2; ++s) {
#pragma unroll
            for (int mv = 0; mv < MV; ++mv) {
                const typename O::Frag fg = TV::frag(sVg, mv, s * O::KSTEP, r, kg);
                const typename O::Frag fr = TV::frag(sVr, mv, s * O::KSTEP, r, kg);
#pragma unroll
                for (int nd = 0; nd < ND; ++nd) {
                    accS[mv][nd] = O::mma(fg, cur.kt[nd][s], accS[mv][nd]);
                    accM[mv][nd] = O::mma(fr, cur.kt[nd][s], accM[mv][nd]);
                }
                if (!REBUILD) {
                    accO[mv] = O::mma(TV::frag(sV0, mv, s * O::KSTEP, r, kg), cur.bm[s], accO[mv]);
                }
            }
        }
        emit_in_step(std::integral_constant<int, 5>{});
        fetch_part<T, DK, DV, DVB, REBUILD, 3>(nxt, d, a, sq, nn, dv0, itok);
        emit_in_step(std::integral_constant<int, 6>{});
        if constexpr (!REBUILD) {
            // the states after this chunk, narrowed once: the LDS copy for the next chunk's stage 1 and, in HBM, that
            // chunk's start states
            narrow_states();
#pragma unroll
            for (int mv = 0; mv < MV; ++mv)
#pragma unroll
                for (int nd = 0; nd < ND; ++nd) {
                    const int dk = (w * ND + nd) * 16 + r;
                    TS::put4_raw(sSt, mv * 16 + kg * 4, dk, sv[2 * nd][mv]);
                    TS::put4_raw(sSt, mv * 16 + kg * 4, DK + dk, sv[2 * nd + 1][mv]);
                }
            if (n + 1 < sq.n1) {
                sblk = blk + 1;
                emit_states(std::integral_constant<int, 0>{});
            }
            RowStore<T, WHOLE>(static_cast<T *>(a.o) + tok0 * DV + dv0, rows, d.H * DV, DVB).template put_narrowed<MV>(iH * DV + kg * (4 * MV), accO);
        }
        emit_in_step(std::integral_constant<int, 7>{});
        __syncthreads();
    };
    // two operand sets used alternately: handing one set over to the other by assignment would touch every
    // register of the set that was just requested, i.e. wait for all of its loads
    {
        CO opsA, opsB;
        fetch_chunk<T, DK, DV, DVB, REBUILD>(opsA, d, a, sq, sq.n0, dv0, itok);
        int n = sq.n0;
        for (; n + 1 < sq.n1; n += 2) {
            step(n, opsA, opsB);
            step(n + 1, opsB, opsA);
        }
        if (n < sq.n1) step(n, opsA, opsB);
    }

#pragma unroll
    for (int mv = 0; mv < MV; ++mv)
#pragma unroll
        for (int nd = 0; nd < ND; ++nd) {
            const size_t g = (sq.state * DK + (w * ND + nd) * 16 + r) * DV + dv0 + kg * (4 * MV) + mv * 4;
            if (a.S_final) *reinterpret_cast<f32x4 *>(a.S_final + g) = accS[mv][nd];
            if (a.M_final) *reinterpret_cast<f32x4 *>(a.M_final + g) = accM[mv][nd];
        }
}


template <typename T, int DK, int DV, int DVB, bool REBUILD, bool WHOLE>
hipError_t launch_scan_w(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    constexpr int G = DV / DVB;
    dim3 grid(((d.BH + 7) / 8) * 8 * G), block(kThreads);
    static const size_t spread = lds_bytes_for_one_workgroup_per_cu(
        reinterpret_cast<const void *>(&scan_fwd_kernel<T, DK, DV, DVB, REBUILD, WHOLE>));
    const size_t dyn = scan_one_per_cu(d) ? spread : 0;
    hipLaunchKernelGGL((scan_fwd_kernel<T, DK, DV, DVB, REBUILD, WHOLE>), grid, block, dyn, s, d, a);
    return hipGetLastError();
}

template <typename T, int DK, int DV, int DVB, bool REBUILD>
hipError_t launch_scan_t(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    return whole_chunks(d) ? launch_scan_w<T, DK, DV, DVB, REBUILD, true>(d, a, s) : launch_scan_w<T, DK, DV, DVB, REBUILD, false>(d, a, s);
}

template <typename T, int DK, int DV, bool REBUILD>
hipError_t pick_dvb(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    if (scan_dvb(d) == 16) return launch_scan_t<T, DK, DV, 16, REBUILD>(d, a, s);
    return launch_scan_t<T, DK, DV, 32, REBUILD>(d, a, s);
}

template <bool REBUILD> hipError_t dispatch_scan(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    if (d.dtype == 0) return launch_scan_fwd16(d, a, REBUILD, s);
    if (!a.coef || !a.k || !a.KT) return hipErrorInvalidValue;
    if (d.dk == 64 && d.dv == 64) return pick_dvb<float, 64, 64, REBUILD>(d, a, s);
    if (d.dk == 128 && d.dv == 128) return pick_dvb<float, 128, 128, REBUILD>(d, a, s);
    return hipErrorInvalidValue;
}

} // namespace

int num_cus() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
            v = 256;
        return v;
    }();
    return n;
}

// (batch, head) pairs of a launch; packed batches: as many as sequences of the longest one's length would make up the batch,
// every sequence counted with the ~4 steps that its states' way in and out takes.  The launch lasts at least the longest sequence's
// chain of steps, which is shorter with 16 columns per workgroup and with a CU for each of its workgroups, however many short
// sequences run beside it.  Forward and backward in us by the number of sequences / by this, d = 128: 29 500 tokens and 16 of 205,
// 16 heads 798 + 1 289 / 729 + 1 289, 4 heads 702 + 981 / 501 + 663; 16 384 and 32 of 512, 8 heads 432 + 987 / 335 + 637.
static long long scan_pairs(const Dims &d) {
    return d.packed ? ((long long)d.nchunks + 4LL * d.B) * d.H / (d.N + 4) : d.BH;
}

// 16-bit storage: 16 columns as long as their workgroups fit the CUs (they hold one each: a second round costs more than the wider
// step).  16 / 32 columns in us, forward and forward with kept states and backward: 32 pairs of heads of 128, 1 024 tokens 32.7 / 39.4
// and 85.7 / 102.0; 40 pairs 51.7 / 41.2 and 133.7 / 115.1, 64 tokens 15.7 / 13.6 and 36.5 / 33.0; heads of 64, 64 pairs, 1 024 tokens
// 29.6 / 35.3 and 82.0 / 93.2; 72 pairs 41.8 / 38.7 and 112.1 / 103.9.
int scan_dvb(const Dims &d) {
    if (d.dtype != 1) return scan_pairs(d) * (d.dv / 16) <= num_cus() ? 16 : 32;
    return 4 * scan_pairs(d) * (d.dv / 32) < 3 * num_cus() || d.dk == 128 ? 16 : 32;
}

bool scan_one_per_cu(const Dims &d) {
    const int wgs = scan_workgroups(d);
    return wgs <= num_cus() || (d.packed && d.BH >= 2 * scan_pairs(d) && 4 * wgs <= 5 * num_cus());
}

int scan_workgroups(const Dims &d) { return (int)((scan_pairs(d) + 7) / 8 * 8 * (d.dv / scan_dvb(d))); }

size_t lds_bytes_for_one_workgroup_per_cu(const void *kernel) {
    hipFuncAttributes fa;
    if (hipFuncGetAttributes(&fa, kernel) != hipSuccess) return 0;
    const size_t half = 80 * 1024, want = half + 1024; // two workgroups of more than 80 KB do not fit the 160 KB of a CU
    return fa.sharedSizeBytes > half ? 0 : want - fa.sharedSizeBytes;
}

hipError_t launch_scan_fwd(const Dims &d, const ScanFwdArgs &a, hipStream_t s) { return dispatch_scan<false>(d, a, s); }

ScanFwdArgs rebuild_args(const RebuildArgs &r) {
    ScanFwdArgs a = {};
    a.coef = r.coef;
    a.k = r.k;
    a.KT = r.KT;
    a.vt_saved = const_cast<void *>(r.vt_saved);
    a.S0 = r.S0;
    a.M0 = r.M0;
    a.states_saved = r.states;
    a.states_lo = r.states_lo;
    return a;
}

hipError_t launch_rebuild(const Dims &d, const RebuildArgs &r, hipStream_t s) { return dispatch_scan<true>(d, rebuild_args(r), s); }

} // namespace mdn
