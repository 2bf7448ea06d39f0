// Chunk-parallel precompute kernel ("intra"): everything of one 64-token chunk that does not
// depend on the incoming states S, M.
//
//   coefficients (Sec. 3.1 Eq. "coefficients", Appendix D), computed WITHOUT the log domain:
//       a_i = prod alpha,  m_i = prod mu,  b_i = alpha_i b_{i-1} + beta_i m_i,
//       Rho_jj = 1, Rho_ij = mu_i Rho_{i-1,j},  Gamma_ij = alpha_i Gamma_{i-1,j} + beta_i Rho_ij
//     (equal to (a_i/m_j)(c_i - c_{j-1}); only positive terms, no division, valid at mu = 0)
//   masked products (Sec. 3.1 "Chunkwise Algorithm"):
//       A  = (P K~^T) .* Gamma^-   (strictly lower; Gamma^-_ij = Gamma_{i-1,j}),  P = alpha k, K~ = eta k
//       Bm = (Q~ K~^T) .* Gamma    (lower incl. diagonal),                         Q~ = scale q
//   triangular solve  T = (I + A)^{-1}
//
// The WY-style factors U = T V, Y = T diag(a^-) P, Z = T diag(b^-) P of Sec. 3.1 are NOT formed: the scans
// apply T themselves,  V~ = T (V - a.(K S) + pb.(K M))  with  alpha_i a_{i-1} = a_i,  pb_i = alpha_i b_{i-1}
// (the same expression with T pulled out; Appendix C, Eq. "apx.v.before" solved for V~), and the reverse scan
// uses Y^T dV~ = K^T (a . T^T dV~).  That trades three 64 x d products and their 1.3 KB per token of HBM
// round trips for one 64 x 64 x dv product inside the scan.
//
// What bounds it: up to a workgroup per CU the chain of one chunk (5.1 us, of which 1.8 until the gates and tiles have arrived; 13 chunks of
// 16 heads of 128, 7.1 -> 5.7 us for the launch); with more, instruction issue and HBM together (8 x 2 048 tokens of 8 heads 30.8 ->
// 25.5 us, 107 MB: 4.2 TB/s where a large copy reaches 4.8).
//
// One workgroup (4 waves) per (chunk, batch*head).  16-bit storage: T, Bm and the coefficients, row by row, for both scans.
// 32-bit storage: forward mode writes T, Bm and K^T; backward mode the transposed operands of the reverse scan (Bm^T, T^T, K^T,
// Q^T); a training forward writes both sets at once, so that the backward need not recompute them; all of them in the blocked
// layout of mdn_device.h (kblk), in which the serial scans' fragment loads are contiguous.
#include "mdn_coef.h"
#include "mdn_device.h"
#include "mdn_kernels.h"
#include "mdn_seq.h"

namespace mdn {

namespace {

// Row strides (floats) of the fp32 A / T matrix and of Gamma in LDS: 16-byte reads of 16 rows take 4.4 clocks of the LDS with 288-byte
// rows, 8 with 272.
constexpr int LDA = 72, LDG = 72;

// LDS [R][ld] (first 64 columns) -> global, kblk layout of an [R][64] operand.  Consecutive lanes write
// consecutive 16-byte pieces of the destination (the pieces of one row's contraction step, then the next
// row's): every store instruction covers whole cache lines.
template <typename T>
__device__ __forceinline__ void store_tile_64cols(T *dst, const T *src, int ld, int rows, int tid) {
    constexpr int E = Op<T>::EPL, PPS = Op<T>::KSTEP / E, CPR = 64 / E; // pieces per contraction step, per row
    for (int c = tid; c < rows * CPR; c += kThreads) {
        const int p = c % PPS, row = (c / PPS) % rows, ks = c / (PPS * rows), cc = ks * PPS + p;
        *reinterpret_cast<Vec16<T> *>(dst + kblk<T>(rows, row, cc * E)) =
            *reinterpret_cast<const Vec16<T> *>(src + row * ld + cc * E);
    }
}

// MODE 0: forward operands; 1: operands of the reverse pass; 2: both (training forward that keeps the
// reverse pass's operands instead of recomputing them)
// WHOLE: see whole_chunks.
template <typename T, int DK, int DV, int MODE, bool WHOLE>
__global__ __launch_bounds__(kThreads, sizeof(T) == 2 ? 3 : 1) void intra_kernel(Dims d, IntraArgs a) {
    constexpr bool FWD = MODE != 1, BWD = MODE != 0, HALF = sizeof(T) == 2;
    static_assert(!HALF || MODE == 0, "16-bit storage: one set of operands");
    typedef Op<T> O;
    constexpr int E = O::EPL;
    constexpr int LDN = HALF ? DK : DK + O::PAD; // natural tiles (16-bit storage: pieces permuted, see token_tile_row_frag)
    constexpr int LDT = 64 + O::PAD; // transposed tiles (32-bit storage)
    constexpr int DX = BWD ? DK : 0; // second transposed tile: Q^T (reverse-pass operands only)
    constexpr int REG_NAT = 2 * 64 * LDN, REG_TR = HALF ? 0 : (DK + DX) * LDT;
    constexpr int REG_A = 64 * LDA * 4 / (int)sizeof(T), REG_KQ = REG_NAT > REG_TR ? REG_NAT : REG_TR;
    constexpr int REGION = REG_KQ > REG_A ? REG_KQ : REG_A;
    constexpr int NVK = 64 * DK / E / kThreads, NVX = BWD ? NVK : 1; // 16-byte vectors per thread

    __shared__ __align__(16) T sR[REGION];
    // Gamma (row stride LDG)
    __shared__ __align__(16) float sG[64 * LDG];
    // A, then T: in the space of the K, Q tiles, once every wave is done with those (70 -> 52 KB of LDS for 16-bit
    // storage at d = 128: three workgroups per CU instead of two)
    float *sA = reinterpret_cast<float *>(sR);
    __shared__ __align__(16) float s_al[64], s_et[64];

    T *sK = sR, *sQ = sR + 64 * LDN;      // phase A
    T *sKT = sR, *sXT = sR + DK * LDT;    // phase B (aliases phase A)

    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const ChunkPos cp = chunk_pos<WHOLE>(d, blockIdx.x, blockIdx.y);
    const size_t tok0 = cp.tok, blk = cp.blk; // (blk: chunk-block index into the workspace tensors)
    // rows from `rows` on are identity steps: their loads go to the last real row and are replaced
    const int rows = WHOLE ? 64 : cp.rows;
    const T *qg = static_cast<const T *>(a.q) + tok0 * DK;
    const T *kg_ = static_cast<const T *>(a.k) + tok0 * DK;
    const size_t rsk = (size_t)d.H * DK;
    float *coef = a.coef + blk * (kCoefRows * 64);

    // ---- the gates first, then the K, Q tiles: all loads in flight at once; the coefficient scans below need
    //      only the gates and run while the tiles are on their way
    const size_t gtok = tok0 + (size_t)(WHOLE ? lane : min(lane, rows - 1)) * d.H;
    float g_al = a.alpha[gtok], g_be = a.beta[gtok], g_mu = a.mu[gtok], g_et = a.eta ? a.eta[gtok] : 1.f;
    typename O::Frag rk[NVK], rq[NVK];
    {
        constexpr int CPR = DK / E;
#pragma unroll
        for (int u = 0; u < NVK; ++u) {
            const int c = tid + u * kThreads, row = WHOLE ? c / CPR : min(c / CPR, rows - 1), cc = c % CPR;
            rk[u] = O::load(kg_ + row * rsk + cc * E);
            rq[u] = O::load(qg + row * rsk + cc * E);
        }
    }
    // 32-bit storage: the rows are loaded a second time in the order of the transposed tiles (in flight until the K, Q
    // tiles are no longer needed) and transposed through LDS.
    Vec16<T> rkt[HALF ? 1 : NVK], rxt[HALF ? 1 : NVX];
    if constexpr (!HALF) {
#pragma unroll
        for (int u = 0; u < NVK; ++u) {
            const int c = tid + u * kThreads, row = WHOLE ? c % 64 : min(c % 64, rows - 1), cc = c / 64;
            rkt[u] = *reinterpret_cast<const Vec16<T> *>(kg_ + row * rsk + cc * E);
        }
        if (BWD) {
#pragma unroll
            for (int u = 0; u < NVX; ++u) {
                const int c = tid + u * kThreads, row = WHOLE ? c % 64 : min(c % 64, rows - 1), cc = c / 64;
                rxt[u] = *reinterpret_cast<const Vec16<T> *>(qg + row * rsk + cc * E);
            }
        }
    }
    if (!WHOLE && rows < 64) { // (wave-uniform: a whole chunk skips this)
        if (lane >= rows) g_al = g_mu = 1.f, g_be = g_et = 0.f;
        constexpr int CPR = DK / E;
#pragma unroll
        for (int u = 0; u < NVK; ++u) {
            if ((tid + u * kThreads) / CPR >= rows) rk[u] = rq[u] = typename O::Frag{};
            if constexpr (!HALF) {
                if ((tid + u * kThreads) % 64 >= rows) {
                    rkt[u] = Vec16<T>{};
                    if (BWD) rxt[u] = Vec16<T>{};
                }
            }
        }
    }

    // ---- gate coefficients.  Matrix Gamma: every wave 16 rows (column scans started from segment maps);
    //      vectors: wave 0, by wave scans (lane i = token i).
    {
        const float al = g_al, be = g_be, mu = g_mu, et = g_et;
        if (w == 0) {
            const float pa = scan_prod(al), pm = scan_prod(mu);
            float c = al, pb = be * pm;
            scan_affine_fwd(c, pb); // b_i = alpha_i b_{i-1} + beta_i m_i
            s_al[lane] = al;
            s_et[lane] = et;
            // alpha_i b_{i-1} (b_{-1} = 0), and the chunk-end values a_C, b_C, m_C into every row
            const f32x4 c0 = {pa, pb, al * wave_up1(pb, 0.f, lane), lane_value(pa, 63)};
            *reinterpret_cast<f32x4 *>(coef + lane * kCoefRows + COEF_A) = c0;
            coef[lane * kCoefRows + COEF_BC] = lane_value(pb, 63);
            coef[lane * kCoefRows + COEF_MC] = lane_value(pm, 63);
        }
        float gC, rC;
        coef_column_scan_blocked<false>(al, be, mu, sG, nullptr, LDG, w, gC, rC);
        if (w == 3) {
            coef[lane * kCoefRows + COEF_GC] = gC * et;
            coef[lane * kCoefRows + COEF_RC] = rC * et;
        }
    }
    {
        constexpr int CPR = DK / E;
#pragma unroll
        for (int u = 0; u < NVK; ++u) {
            const int c = tid + u * kThreads, row = c / CPR, cc = HALF ? (c % CPR) ^ (row & (CPR < 16 ? CPR - 1 : 15)) : c % CPR;
            *reinterpret_cast<typename O::Frag *>(sK + row * LDN + cc * E) = rk[u];
            *reinterpret_cast<typename O::Frag *>(sQ + row * LDN + cc * E) = rq[u];
        }
    }
    __syncthreads();

    // ---- masked intra-chunk products, 16 x 16 tiles (rows i of tile nt, columns j of tile jt).  The ten on or below the diagonal
    //      are formed, three by a wave, without branches; the six above it are zeroed, two by a wave (some twice):
    //        wave 0: (1,0) (2,0) (3,0), zeros (0,1) (0,2)    wave 2: (2,2) (3,2) (0,0), zeros (1,3) (2,3)
    //        wave 1: (1,1) (2,1) (3,1), zeros (0,3) (1,2)    wave 3: (3,3) three times, zeros (1,3) (2,3)
    //      The products are formed in the orientation whose accumulator lanes hold 4 consecutive entries along the contraction
    //      index of the consumer (j for Bm and A, i for Bm^T).  What a masked value needs of Gamma is read by every lane: inside the
    //      selection, each of 32 reads stood in a branch of its own (clocks of a chunk with a CU to itself, this and A's mask: 3 200 +
    //      1 900, now 2 100 + 1 000).
    const int r = lane & 15, kq = lane >> 4, i0 = w * 16;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    auto row_frag = [&](const T *tile, int row, int st) -> typename O::Frag {
        if constexpr (HALF) return token_tile_row_frag<DK>(tile, row, st, kq);
        else return O::load(tile + row * LDN + st * O::KSTEP + kq * E);
    };
    constexpr int KS = DK / O::KSTEP;
    auto pick = [&](int table, int u) { return (table >> (8 * u + 2 * wu)) & 3; };
    auto nt_of = [&](int u) { return pick(0xCFFAE5, u); }; // 1 1 2 3 | 2 2 3 3 | 3 3 0 3
    auto jt_of = [&](int u) { return pick(0xC4E4E4, u); }; // 0 1 2 3 | 0 1 2 3 | 0 1 0 3
    auto nz_of = [&](int u) { return pick(0xA450, u); };   // 0 0 1 1 | 0 1 2 2
    auto jz_of = [&](int u) { return pick(0xFAFD, u); };   // 1 3 3 3 | 2 2 3 3
    {
        f32x4 kk[3], qk[3]; // element x of product u: k_i . k_j, q_i . k_j with i = nt*16 + r, j = jt*16 + kq*4 + x
        zero_acc(kk);
        zero_acc(qk);
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const typename O::Frag fa = row_frag(sK, jt_of(u) * 16 + r, st);
                kk[u] = O::mma(fa, row_frag(sK, nt_of(u) * 16 + r, st), kk[u]);
                if (FWD) qk[u] = O::mma(fa, row_frag(sQ, nt_of(u) * 16 + r, st), qk[u]);
            }
        if (BWD) {
            // qt[nt][x] = q_i . k_j, i = i0 + kq*4 + x, j = nt*16 + r  ->  Bm^T row j, k = i
            f32x4 qt[4];
            zero_acc(qt);
            mma_rows<T, 4, DK>(qt, sQ + i0 * LDN, LDN, sK, LDN);
            T *out = static_cast<T *>(a.BmT) + blk * 4096;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int j = nt * 16 + r;
                const float et = s_et[j];
                f32x4 v;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int i = i0 + kq * 4 + x;
                    const float full = d.scale * et * sG[i * LDG + j] * qt[nt][x];
                    v[x] = (j <= i) ? full : 0.f;
                }
                store4(out + kblk<T>(64, j, i0 + kq * 4), v);
            }
        }
        if (FWD) {
            T *out = static_cast<T *>(a.Bm) + blk * 4096; // Bm row i, k = j
            auto put = [&](int i, int j0, f32x4 v) { store4(at32(out, HALF ? (unsigned)(i * 64 + j0) : (unsigned)kblk<T>(64, i, j0)), v); };
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int i = nt_of(u) * 16 + r, j0 = jt_of(u) * 16 + kq * 4;
                const f32x4 g = *reinterpret_cast<const f32x4 *>(&sG[i * LDG + j0]), et = *reinterpret_cast<const f32x4 *>(&s_et[j0]);
                f32x4 v;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float full = d.scale * et[x] * g[x] * qk[u][x];
                    v[x] = (j0 + x <= i) ? full : 0.f;
                }
                put(i, j0, v);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) put(nz_of(u) * 16 + r, jz_of(u) * 16 + kq * 4, f32x4{0.f, 0.f, 0.f, 0.f});
        }
        if constexpr (!HALF) {
            // ---- 32-bit storage: the transposed tiles take the space of the K, Q tiles (dst[d][row] = src[row][d]),
            //      go out from there, and only then does A move in
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NVK; ++u) {
                const int c = tid + u * kThreads, row = c % 64, cc = c / 64;
#pragma unroll
                for (int e = 0; e < E; ++e) sKT[(cc * E + e) * LDT + row] = rkt[u].e[e];
            }
            if (BWD) {
#pragma unroll
                for (int u = 0; u < NVX; ++u) {
                    const int c = tid + u * kThreads, row = c % 64, cc = c / 64;
#pragma unroll
                    for (int e = 0; e < E; ++e) sXT[(cc * E + e) * LDT + row] = rxt[u].e[e];
                }
            }
            __syncthreads();
            store_tile_64cols<T>(static_cast<T *>(a.KT) + blk * (DK * 64), sKT, LDT, DK, tid);
            if (BWD) store_tile_64cols<T>(static_cast<T *>(a.QT) + blk * (DK * 64), sXT, LDT, DK, tid);
        }
        __syncthreads(); // every wave is done with the tiles: A takes their place
        // (K K^T is symmetric: k_i . k_j whichever of them was the row of the product)
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int i = nt_of(u) * 16 + r, j0 = jt_of(u) * 16 + kq * 4;
            const f32x4 g = *reinterpret_cast<const f32x4 *>(&sG[(i > 0 ? i - 1 : 0) * LDG + j0]), et = *reinterpret_cast<const f32x4 *>(&s_et[j0]);
            const float al_i = s_al[i];
            f32x4 v;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float full = al_i * et[x] * g[x] * kk[u][x];
                v[x] = (j0 + x < i) ? full : 0.f;
            }
            *reinterpret_cast<f32x4 *>(&sA[i * LDA + j0]) = v;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            *reinterpret_cast<f32x4 *>(&sA[(nz_of(u) * 16 + r) * LDA + jz_of(u) * 16 + kq * 4]) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();

    // ---- T = (I + A)^{-1}
    tri_inverse_blocked(sA, LDA, wu);
    __syncthreads();

    if (BWD) {
        T *tt = static_cast<T *>(a.TmT) + blk * 4096; // T^T: row j, k = i
        constexpr int E = O::EPL;
        constexpr int PPS = O::KSTEP / E; // 16-byte pieces per contraction step: consecutive lanes, consecutive pieces
        for (int c = tid; c < 64 * (64 / E); c += kThreads) {
            const int pp = c % PPS, jj = (c / PPS) & 63, cc = (c / (PPS * 64)) * PPS + pp;
            Vec16<T> v;
#pragma unroll
            for (int e = 0; e < E; ++e) v.e[e] = from_f32<T>(sA[(cc * E + e) * LDA + jj]);
            *reinterpret_cast<Vec16<T> *>(tt + kblk<T>(64, jj, cc * E)) = v;
        }
    }

    if (FWD) {
        T *tm = static_cast<T *>(a.Tm) + blk * 4096; // T: row i, k = j
        constexpr int PPS = HALF ? 64 / E : O::KSTEP / E; // consecutive lanes, consecutive pieces of the destination
        for (int c = tid; c < 64 * (64 / E); c += kThreads) {
            const int pp = c % PPS, ii = (c / PPS) & 63, cc = (c / (PPS * 64)) * PPS + pp;
            Vec16<T> v;
#pragma unroll
            for (int e = 0; e < E; ++e) v.e[e] = from_f32<T>(sA[ii * LDA + cc * E + e]);
            *reinterpret_cast<Vec16<T> *>(tm + (HALF ? (size_t)(ii * 64 + cc * E) : kblk<T>(64, ii, cc * E))) = v;
        }
    }
}

template <typename T, int DK, int DV, bool WHOLE>
hipError_t launch_intra_w(const Dims &d, int mode, const IntraArgs &a, hipStream_t s) {
    dim3 grid(chunk_grid_x(d), chunk_grid_y(d)), block(kThreads);
    if constexpr (sizeof(T) == 2) {
        hipLaunchKernelGGL((intra_kernel<T, DK, DV, 0, WHOLE>), grid, block, 0, s, d, a);
    } else {
        if (mode == 0) hipLaunchKernelGGL((intra_kernel<T, DK, DV, 0, WHOLE>), grid, block, 0, s, d, a);
        else if (mode == 1) hipLaunchKernelGGL((intra_kernel<T, DK, DV, 1, WHOLE>), grid, block, 0, s, d, a);
        else hipLaunchKernelGGL((intra_kernel<T, DK, DV, 2, WHOLE>), grid, block, 0, s, d, a);
    }
    return hipGetLastError();
}
template <typename T, int DK, int DV>
hipError_t launch_intra_t(const Dims &d, int mode, const IntraArgs &a, hipStream_t s) {
    return whole_chunks(d) ? launch_intra_w<T, DK, DV, true>(d, mode, a, s) : launch_intra_w<T, DK, DV, false>(d, mode, a, s);
}

} // namespace

hipError_t launch_intra(const Dims &d, int mode, const IntraArgs &a, hipStream_t s) {
    const bool f32 = d.dtype == 1;
    if (d.dk == 64 && d.dv == 64)
        return f32 ? launch_intra_t<float, 64, 64>(d, mode, a, s) : launch_intra_t<bf16_t, 64, 64>(d, mode, a, s);
    if (d.dk == 128 && d.dv == 128)
        return f32 ? launch_intra_t<float, 128, 128>(d, mode, a, s) : launch_intra_t<bf16_t, 128, 128>(d, mode, a, s);
    return hipErrorInvalidValue;
}

} // namespace mdn
