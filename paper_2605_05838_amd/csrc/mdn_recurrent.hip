// Recurrent (decoding) form, Eq. Mt.recurrent / St.recurrent in the operation order of the
// recurrent listing of Appendix E:
//     e = v - S^T (alpha k);  M = mu M - eta k e^T;  S = alpha S - beta M;  o = scale S^T q
// HBM-bound on reading and writing the two fp32 states once per call; plain fp32 FMA, no MFMA
// (a GEMV and a rank-1 update per token).  A workgroup owns COLS = 32 or 64 state columns of one (batch, head) pair;
// thread (slice, column group) holds dk*COLS/1024 rows x 4 consecutive columns of S and M in
// registers, so every state access is a 16-byte vector and every wave-level access covers whole
// 128-byte lines.  The two reductions over dk go over the slices of a wave by shuffles, then over
// the 4 waves through LDS.  The workgroups of one pair follow each other in the grid: together they read its states
// front to back (column blocks a whole grid apart: 226 against 205 us for 256 sequences of 16 heads of 128).  A token's
// operands are requested one token ahead: several tokens per call wait for memory once (64 sequences x 8 tokens: 64 ->
// 59 us, with 64 columns 54 us).
#include "mdn_device.h"
#include "mdn_kernels.h"

namespace mdn {

namespace {

// sum over the slices of a wave (lane = slice_in_wave * CG + column group, CG = 8 or 16 column groups)
template <int CG> __device__ __forceinline__ f32x4 reduce_slices(f32x4 v) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        if (CG == 8) v[x] += dpp_move<0x128>(v[x]); // lane ^ 8 (rotation by half a row)
        v[x] = add_xor32(add_xor16(v[x]));
    }
    return v;
}

// one token's operands of a thread, in storage form
template <typename T, int ROWS> struct TokenOps {
    struct alignas(ROWS * sizeof(T)) Rows { T e[ROWS]; };
    Rows k, q;
    typename Raw4<T>::type v;
    float al, be, mu, et;
};

// NT: past the caches, for states that would not be there any more when they are needed next
template <bool NT> __device__ __forceinline__ f32x4 load_state(const float *p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    else return *reinterpret_cast<const f32x4 *>(p);
}
template <bool NT> __device__ __forceinline__ void store_state(float *p, f32x4 v) {
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p));
    else *reinterpret_cast<f32x4 *>(p) = v;
}

template <typename T, int DK, int DV, int COLS, bool NT>
__global__ __launch_bounds__(kThreads) void recurrent_kernel(Dims d, RecurrentArgs a) {
    constexpr int CG = COLS / 4, ROWS = DK * CG / kThreads, NB = DV / COLS; // column groups, rows per slice, workgroups per pair
    static_assert(ROWS >= 1, "dk too small for the slice count");
    typedef TokenOps<T, ROWS> Ops;
    typedef typename Ops::Rows Rows;
    __shared__ __align__(16) float redE[4][COLS], redO[4][COLS];
    const int bh = blockIdx.x / NB, b = bh / d.H, h = bh % d.H;
    const int cg = threadIdx.x % CG, sl = threadIdx.x / CG, w = wave_id();
    const int j = blockIdx.x % NB * COLS + cg * 4, r0 = sl * ROWS;
    auto fetch = [&](int t) {
        Ops c;
        const size_t g = ((size_t)b * d.T + t) * d.H + h;
        c.k = *reinterpret_cast<const Rows *>(static_cast<const T *>(a.k) + g * DK + r0);
        c.q = *reinterpret_cast<const Rows *>(static_cast<const T *>(a.q) + g * DK + r0);
        c.v = load4_raw(static_cast<const T *>(a.v) + g * DV + j);
        c.al = a.alpha[g];
        c.be = a.beta[g];
        c.mu = a.mu[g];
        c.et = a.eta ? a.eta[g] : 1.f;
        return c;
    };
    Ops c = fetch(0);
    f32x4 S[ROWS], M[ROWS];
    float *Sg = a.S + ((size_t)bh * DK + r0) * DV + j, *Mg = a.M + ((size_t)bh * DK + r0) * DV + j;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        S[i] = load_state<NT>(Sg + (size_t)i * DV);
        M[i] = load_state<NT>(Mg + (size_t)i * DV);
    }
    for (int t = 0; t < d.T; ++t) {
        const Ops nx = fetch(t + 1 < d.T ? t + 1 : t);
        float kk[ROWS];
        f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            kk[i] = to_f32(c.k.e[i]);
            part += (c.al * kk[i]) * S[i];
        }
        part = reduce_slices<CG>(part);
        if ((threadIdx.x & 63) < CG) *reinterpret_cast<f32x4 *>(&redE[w][cg * 4]) = part;
        __syncthreads();
        f32x4 e = widen4(c.v);
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) e -= *reinterpret_cast<const f32x4 *>(&redE[ww][cg * 4]);
        f32x4 po = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            M[i] = c.mu * M[i] - (c.et * kk[i]) * e;
            S[i] = c.al * S[i] - c.be * M[i];
            po += to_f32(c.q.e[i]) * S[i];
        }
        po = reduce_slices<CG>(po);
        if ((threadIdx.x & 63) < CG) *reinterpret_cast<f32x4 *>(&redO[w][cg * 4]) = po;
        __syncthreads();
        if (sl == 0) {
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ww = 0; ww < 4; ++ww) o += *reinterpret_cast<const f32x4 *>(&redO[ww][cg * 4]);
            store4(static_cast<T *>(a.o) + (((size_t)b * d.T + t) * d.H + h) * DV + j, d.scale * o);
        }
        c = nx;
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        store_state<NT>(Sg + (size_t)i * DV, S[i]);
        store_state<NT>(Mg + (size_t)i * DV, M[i]);
    }
}

template <typename T, int DK, int DV, int COLS, bool NT>
hipError_t launch_cols(const Dims &d, const RecurrentArgs &a, hipStream_t s) {
    dim3 grid(d.BH * (DV / COLS)), block(kThreads);
    hipLaunchKernelGGL((recurrent_kernel<T, DK, DV, COLS, NT>), grid, block, 0, s, d, a);
    return hipGetLastError();
}

// 64 columns per workgroup once that leaves every CU 4 workgroups (16 waves), 32 below, where more and shorter workgroups
// are what the chip lacks: 16 heads of 128, 1 / 4 / 16 sequences, one token: 3.5 / 4.2 / 8.6 us with 32, 3.7 / 4.7 / 8.8 us
// with 64; 64 sequences of 8 tokens 59 and 54 us.
// States of more than 352 MiB go past the caches: the 256 MB last-level cache holds too little of them until the next call
// and only delays the traffic (512 MiB: 205 -> 189 us = 5.7 TB/s, where an in-place pass over a large buffer reaches 6.0;
// 384 MiB: 149 -> 144 us; equal at 352); smaller ones are found there in part by a call that follows at once (256 MiB:
// 80 us, past the caches 95 us).
template <typename T, int DK, int DV> hipError_t launch_recurrent_t(const Dims &d, const RecurrentArgs &a, hipStream_t s) {
    const long long state_bytes = 2LL * d.BH * DK * DV * (long long)sizeof(float);
    if ((long long)d.BH * (DV / 64) < 4LL * num_cus()) return launch_cols<T, DK, DV, 32, false>(d, a, s);
    if (state_bytes <= (352LL << 20)) return launch_cols<T, DK, DV, 64, false>(d, a, s);
    return launch_cols<T, DK, DV, 64, true>(d, a, s);
}

} // namespace

hipError_t launch_recurrent(const Dims &d, const RecurrentArgs &a, hipStream_t s) {
    const bool f32 = d.dtype == 1;
    if (d.dk == 64 && d.dv == 64)
        return f32 ? launch_recurrent_t<float, 64, 64>(d, a, s) : launch_recurrent_t<bf16_t, 64, 64>(d, a, s);
    if (d.dk == 128 && d.dv == 128)
        return f32 ? launch_recurrent_t<float, 128, 128>(d, a, s) : launch_recurrent_t<bf16_t, 128, 128>(d, a, s);
    return hipErrorInvalidValue;
}

} // namespace mdn
