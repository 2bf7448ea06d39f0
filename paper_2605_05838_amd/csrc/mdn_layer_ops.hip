// The elementwise operations around the momentum delta rule in the MDN layer (Sec. 3.3, architecture paragraph), and
// their adjoints.  Front end, per token and head, on the short-convolution outputs x_q, x_k, x_v:
//     q' = SiLU(x_q),  k' = SiLU(x_k),  v = SiLU(x_v);   q = L2Norm(q' - d_h k')  (output correction, before the
//     normalisation);   k = L2Norm(k');   L2Norm(x) = x / sqrt(sum x^2 + eps)
// Back end:  y = sigmoid(g) * w * o / sqrt(mean(o^2) + eps)   (head-wise RMS norm with one weight vector, output gate).
// Streaming kernels (arithmetic in fp32, tensors in the storage dtype): a lane holds 16 bytes of a row and a row sum is 3 to 5
// lane exchanges.  With 4 bytes per lane and a row per wave the adjoints were bound by the vector unit: IEEE divisions in the
// sigmoids, row sums over 64 lanes and the 64-bit remainder of the row index took ~60 instructions per element.  In us,
// then / now, 131 072 rows of 128 elements, 16-bit: front end forward 55 / 38, adjoint 78 / 58; back end forward 18.9 / 16.9,
// adjoint 56 / 34 (4.9 to 6.0 TB/s; a large device copy reaches 4.8); 32-bit: 73 / 74, 117 / 117, 33.9 / 32.4, 78 / 64.
// Parameter gradients (dd [H], dw [dv]) are summed per workgroup in LDS, then added with one floating-point atomic per
// entry and workgroup.  Those kernels run at most one workgroup of 1 024 threads per CU: atomics of several dies on one
// address are taken one after the other, ~20 ns each.
#include "../../include/mdn.h"
#include "mdn_device.h"
#include "mdn_kernels.h"

#include <hip/hip_runtime.h>

namespace mdn {

namespace {

constexpr int LT = 256; // threads of the kernels without parameter gradients

// sigmoid: 1 / (1 + e^-x) by the reciprocal instruction (1 ulp) and one Newton step.  Compared for every fp32 value of e^-x
// from 0 to infinity, the quotient is bit for bit that of the IEEE division (ten instructions: the kernels were bound by
// them), denormal quotients to one unit in their last place.  The reciprocal flushes denormal results, which is why it is taken
// of 2^-32 times its argument; at e^-x = infinity its residual is not a number, which the maximum replaces.
// (The bare reciprocal, 16-bit storage: front end forward 33.6 us where it takes 35.7, adjoint 54.9 / 55.6; back end
// 18.7 / 18.7, 32.6 / 33.6.)
__device__ __forceinline__ float sigm(float x) {
    const float d = __builtin_fmaf(__expf(-x), 0x1p-32f, 0x1p-32f), r = __builtin_amdgcn_rcpf(d);
    const float e = fmaxf(__builtin_fmaf(-d, r, 1.f), -1.f);
    return __builtin_fmaf(r, e, r) * 0x1p-32f;
}

// This lane's E elements of a row of D: D / E lanes hold a row, 64 E / D rows a wave.  Tensors need no more than the alignment
// of their elements (a weight sliced out of a flat buffer): the vector types say so, and 16-byte accesses stay 16 bytes wide,
// which the hardware takes at any address.
template <typename T, int D, int E_> struct Row {
    static constexpr int E = E_, LPR = D / E, RPW = 64 / LPR;
    typedef bf16x8 __attribute__((aligned(2))) Half8;
    typedef f32x4 __attribute__((aligned(4))) Float4;
    float v[E];
    __device__ __forceinline__ void load(const T *p) {
        if constexpr (sizeof(T) == 2 && E == 8) {
            const bf16x8 x = *reinterpret_cast<const Half8 *>(p);
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = (float)x[e];
        } else if constexpr (sizeof(T) == 4 && E % 4 == 0) {
#pragma unroll
            for (int u = 0; u < E; u += 4) {
                const f32x4 x = *reinterpret_cast<const Float4 *>(p + u);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[u + e] = x[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = to_f32(p[e]);
        }
    }
    __device__ __forceinline__ void store(T *p) const {
        if constexpr (sizeof(T) == 2 && E == 8) {
            bf16x8 x;
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = (bf16_t)v[e];
            *reinterpret_cast<Half8 *>(p) = x;
        } else if constexpr (sizeof(T) == 4 && E % 4 == 0) {
#pragma unroll
            for (int u = 0; u < E; u += 4) *reinterpret_cast<Float4 *>(p + u) = f32x4{v[u], v[u + 1], v[u + 2], v[u + 3]};
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) p[e] = from_f32<T>(v[e]);
        }
    }
    // sum of x over the lanes of a row, in every one of them
    static __device__ __forceinline__ float row_sum(float x) {
        static_assert(LPR == 8 || LPR == 16 || LPR == 32 || LPR == 64, "lanes of a row");
        if constexpr (LPR == 8) {
            x += dpp_move<0xB1>(x);         // quad_perm [1,0,3,2]
            x += dpp_move<0x4E>(x);         // quad_perm [2,3,0,1]
            return x + dpp_move<0x141>(x);  // row_half_mirror: the other quad of the 8 lanes
        }
        x = reduce16(x);
        if (LPR > 16) x = add_xor16(x);
        if (LPR > 32) x = add_xor32(x);
        return x;
    }
};

struct LayerDims {
    unsigned rows; // B*T*H
    int H;
};

// The rows of one lane: row0, row0 + step, ... and their heads (row % H, carried along).
struct RowWalk {
    unsigned row, step;
    int h, dh;
    __device__ __forceinline__ RowWalk(const LayerDims &d, int rows_per_wave, int lanes_per_row) {
        const unsigned waves = blockDim.x >> 6;
        row = (blockIdx.x * waves + wave_id()) * rows_per_wave + lane_id() / lanes_per_row;
        step = gridDim.x * waves * rows_per_wave;
        h = (int)(row % (unsigned)d.H);
        dh = (int)(step % (unsigned)d.H);
    }
    __device__ __forceinline__ void next(const LayerDims &d) {
        row += step;
        h += dh;
        h = h >= d.H ? h - d.H : h;
    }
};

template <typename T, int D, int E>
__global__ __launch_bounds__(LT) void frontend_fwd_kernel(LayerDims d, const T *xq, const T *xk, const T *xv, const float *dh,
                                                           float eps, T *q, T *k, T *v) {
    typedef Row<T, D, E> R;
    for (RowWalk w(d, R::RPW, R::LPR); w.row < d.rows; w.next(d)) {
        const size_t o = (size_t)w.row * D + (lane_id() % R::LPR) * E;
        R a, b, c;
        a.load(xq + o);
        b.load(xk + o);
        c.load(xv + o);
        const float dc = dh[w.h];
        float sq = 0.f, sk = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            b.v[e] *= sigm(b.v[e]);
            a.v[e] = a.v[e] * sigm(a.v[e]) - dc * b.v[e];
            sq += a.v[e] * a.v[e];
            sk += b.v[e] * b.v[e];
        }
        const float iq = rsqrtf(R::row_sum(sq) + eps), ik = rsqrtf(R::row_sum(sk) + eps);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            a.v[e] *= iq;
            b.v[e] *= ik;
            c.v[e] *= sigm(c.v[e]);
        }
        a.store(q + o);
        b.store(k + o);
        c.store(v + o);
    }
}

template <typename T, int D, int E>
__global__ __launch_bounds__(1024) void frontend_bwd_kernel(LayerDims d, const T *xq, const T *xk, const T *xv, const float *dh,
                                                             float eps, const T *dq, const T *dk, const T *dv, T *dxq, T *dxk,
                                                             T *dxv, float *dd) {
    typedef Row<T, D, E> R;
    extern __shared__ float s_dd[]; // [H]
    for (int c = threadIdx.x; c < d.H; c += blockDim.x) s_dd[c] = 0.f;
    __syncthreads();
    for (RowWalk w(d, R::RPW, R::LPR); w.row < d.rows; w.next(d)) {
        const size_t o = (size_t)w.row * D + (lane_id() % R::LPR) * E;
        R a, b, c, ga, gb, gc;
        a.load(xq + o);
        b.load(xk + o);
        ga.load(dq + o);
        gb.load(dk + o);
        c.load(xv + o);
        gc.load(dv + o);
        const float dc = dh[w.h];
        // SiLU(x) = x s, SiLU'(x) = s (1 + x (1 - s)): the derivatives replace the inputs
        float qc[E], ks[E], sq = 0.f, sk = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float sa = sigm(a.v[e]), sb = sigm(b.v[e]);
            ks[e] = b.v[e] * sb;
            qc[e] = a.v[e] * sa - dc * ks[e];
            a.v[e] = sa * (1.f + a.v[e] * (1.f - sa));
            b.v[e] = sb * (1.f + b.v[e] * (1.f - sb));
            sq += qc[e] * qc[e];
            sk += ks[e] * ks[e];
        }
        const float iq = rsqrtf(R::row_sum(sq) + eps), ik = rsqrtf(R::row_sum(sk) + eps);
        float dotq = 0.f, dotk = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            qc[e] *= iq;
            dotq += qc[e] * ga.v[e];
            dotk += ks[e] * gb.v[e];
        }
        dotq = R::row_sum(dotq);
        dotk = R::row_sum(dotk) * ik * ik;
        float ddp = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float dqc = (ga.v[e] - qc[e] * dotq) * iq; // through the L2 norm of q' - d k'
            const float dks = (gb.v[e] - ks[e] * dotk) * ik - dc * dqc;
            ddp -= dqc * ks[e];
            a.v[e] *= dqc;
            b.v[e] *= dks;
            const float sc = sigm(c.v[e]);
            c.v[e] = gc.v[e] * (sc * (1.f + c.v[e] * (1.f - sc)));
        }
        a.store(dxq + o);
        b.store(dxk + o);
        c.store(dxv + o);
        if (dd) {
            ddp = R::row_sum(ddp);
            if (lane_id() % R::LPR == 0) atomicAdd(&s_dd[w.h], ddp);
        }
    }
    __syncthreads();
    if (dd)
        for (int c = threadIdx.x; c < d.H; c += blockDim.x) atomicAdd(&dd[c], s_dd[c]);
}

template <typename T, int D, int E>
__global__ __launch_bounds__(LT) void epilogue_fwd_kernel(LayerDims d, const T *o, const T *g, const float *w, float eps, T *y) {
    typedef Row<T, D, E> R;
    Row<float, D, E> wr;
    wr.load(w + (lane_id() % R::LPR) * E);
    for (RowWalk k(d, R::RPW, R::LPR); k.row < d.rows; k.next(d)) {
        const size_t off = (size_t)k.row * D + (lane_id() % R::LPR) * E;
        R a, b;
        a.load(o + off);
        b.load(g + off);
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) ss += a.v[e] * a.v[e];
        const float ir = rsqrtf(R::row_sum(ss) * (1.f / D) + eps);
#pragma unroll
        for (int e = 0; e < E; ++e) a.v[e] = sigm(b.v[e]) * wr.v[e] * a.v[e] * ir;
        a.store(y + off);
    }
}

template <typename T, int D, int E>
__global__ __launch_bounds__(1024) void epilogue_bwd_kernel(LayerDims d, const T *o, const T *g, const float *w, float eps,
                                                             const T *dy, T *dout, T *dg, float *dw) {
    typedef Row<T, D, E> R;
    __shared__ float s_dw[D];
    for (int c = threadIdx.x; c < D; c += blockDim.x) s_dw[c] = 0.f;
    __syncthreads();
    const int col = (lane_id() % R::LPR) * E;
    Row<float, D, E> wr;
    wr.load(w + col);
    float dwp[E];
#pragma unroll
    for (int e = 0; e < E; ++e) dwp[e] = 0.f;
    for (RowWalk k(d, R::RPW, R::LPR); k.row < d.rows; k.next(d)) {
        const size_t off = (size_t)k.row * D + col;
        R a, b, c;
        a.load(o + off);
        b.load(g + off);
        c.load(dy + off);
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) ss += a.v[e] * a.v[e];
        const float ir = rsqrtf(R::row_sum(ss) * (1.f / D) + eps);
        float dn[E], dot = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float sg = sigm(b.v[e]), t = c.v[e] * sg;
            a.v[e] *= ir; // normalised output
            dn[e] = t * wr.v[e];
            dot += a.v[e] * dn[e];
            dwp[e] += t * a.v[e];
            b.v[e] = dn[e] * a.v[e] * (1.f - sg);
        }
        dot = R::row_sum(dot) * (1.f / D);
#pragma unroll
        for (int e = 0; e < E; ++e) a.v[e] = (dn[e] - a.v[e] * dot) * ir;
        a.store(dout + off);
        b.store(dg + off);
    }
    if (dw) {
        // the rows of a wave first (lanes with the same columns), then the waves in LDS
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (R::LPR == 8) dwp[e] += dpp_move<0x128>(dwp[e]); // row_ror 8
            if (R::LPR <= 16) dwp[e] = add_xor16(dwp[e]);
            if (R::LPR <= 32) dwp[e] = add_xor32(dwp[e]);
            if (lane_id() < R::LPR) atomicAdd(&s_dw[col + e], dwp[e]);
        }
        __syncthreads();
        for (int c = threadIdx.x; c < D; c += blockDim.x) atomicAdd(&dw[c], s_dw[c]);
    }
}

__global__ void layer_zero_kernel(float *p, int n) {
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) p[c] = 0.f;
}

int check(const mdn_shape *s, LayerDims *d) {
    if (!s) return MDN_ERR_NULL;
    if (s->dtype != MDN_DTYPE_BF16 && s->dtype != MDN_DTYPE_F32) return MDN_ERR_DTYPE;
    if (s->B < 1 || s->T < 1 || s->H < 1 || s->H > 4096) return MDN_ERR_SHAPE;
    if (!((s->dk == 64 && s->dv == 64) || (s->dk == 128 && s->dv == 128))) return MDN_ERR_SHAPE;
    const long long rows = (long long)s->B * s->T * s->H;
    if (rows > 0x7fffffffLL) return MDN_ERR_SHAPE; // (more than 288 GB of tensors)
    d->rows = (unsigned)rows;
    d->H = s->H;
    return MDN_OK;
}

// launch shape of a row-streaming kernel: workgroups of 256 threads, at most 32 per CU
struct Launch { int grid, block; };
Launch stream_launch(unsigned rows, unsigned rows_per_wave) {
    const unsigned per = LT / 64 * rows_per_wave, need = (rows + per - 1) / per, most = 32u * (unsigned)num_cus();
    return Launch{(int)(need < most ? need : most), LT};
}
// the same for a kernel that ends in atomic adds on a few addresses: one workgroup per CU at most, of 1 024 threads once
// there are rows enough to give every CU one (below that, smaller workgroups reach more CUs)
Launch reduce_launch(unsigned rows, unsigned rows_per_wave) {
    const unsigned cus = (unsigned)num_cus();
    const unsigned waves = rows >= cus * 16u * rows_per_wave ? 16u : 4u, per = waves * rows_per_wave, need = (rows + per - 1) / per;
    return Launch{(int)(need < cus ? need : cus), (int)waves * 64};
}

int status() { return hipGetLastError() == hipSuccess ? MDN_OK : MDN_ERR_LAUNCH; }

// F(type tag, row length tag, elements-per-lane tag): 16 bytes per lane; a wave per row for few rows and kernels that sum no
// parameter gradients, where what counts is the chain of one lane's instructions (front end forward in us, wave per row / 16 bytes,
// 16-bit: 800 rows of 128 2.48 / 2.88, 2 000 2.74 / 3.03, 4 000 3.47 / 3.30; of 64 2.43 / 2.86, 2.59 / 2.89, 3.03 / 3.05;
// 32-bit, of 128: 2.60 / 2.69, 3.05 / 3.02, 4.03 / 4.10).
template <typename F> int dispatch(const mdn_shape *s, unsigned rows, bool sums, F &&f) {
    auto lanes = [&](auto t, auto dim) {
        constexpr int D = decltype(dim)::value;
        if (rows < 8u * (unsigned)num_cus() && !sums) return f(t, dim, std::integral_constant<int, D / 64>{});
        return f(t, dim, std::integral_constant<int, 16 / (int)sizeof(t)>{});
    };
    const bool f32 = s->dtype == MDN_DTYPE_F32;
    if (s->dk == 64) return f32 ? lanes(float{}, std::integral_constant<int, 64>{}) : lanes(bf16_t{}, std::integral_constant<int, 64>{});
    return f32 ? lanes(float{}, std::integral_constant<int, 128>{}) : lanes(bf16_t{}, std::integral_constant<int, 128>{});
}

} // namespace

} // namespace mdn

using namespace mdn;

extern "C" {

int mdn_frontend_fwd(const mdn_shape *shape, const void *x_q, const void *x_k, const void *x_v, const float *d, float eps,
                     void *q, void *k, void *v, void *stream) {
    LayerDims ld;
    const int rc = check(shape, &ld);
    if (rc) return rc;
    if (!x_q || !x_k || !x_v || !d || !q || !k || !v) return MDN_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    return dispatch(shape, ld.rows, false, [&](auto t, auto dim, auto el) {
        typedef decltype(t) T;
        constexpr int D = decltype(dim)::value, E = decltype(el)::value;
        const Launch l = stream_launch(ld.rows, Row<T, D, E>::RPW);
        hipLaunchKernelGGL((frontend_fwd_kernel<T, D, E>), dim3(l.grid), dim3(l.block), 0, s, ld,
                           static_cast<const T *>(x_q), static_cast<const T *>(x_k), static_cast<const T *>(x_v), d, eps,
                           static_cast<T *>(q), static_cast<T *>(k), static_cast<T *>(v));
        return status();
    });
}

int mdn_frontend_bwd(const mdn_shape *shape, const void *x_q, const void *x_k, const void *x_v, const float *d, float eps,
                     const void *dq, const void *dk, const void *dv, void *dx_q, void *dx_k, void *dx_v, float *dd,
                     void *stream) {
    LayerDims ld;
    const int rc = check(shape, &ld);
    if (rc) return rc;
    if (!x_q || !x_k || !x_v || !d || !dq || !dk || !dv || !dx_q || !dx_k || !dx_v) return MDN_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dd) hipLaunchKernelGGL(layer_zero_kernel, dim3(1), dim3(256), 0, s, dd, ld.H);
    return dispatch(shape, ld.rows, dd != nullptr, [&](auto t, auto dim, auto el) {
        typedef decltype(t) T;
        constexpr int D = decltype(dim)::value, E = decltype(el)::value;
        const Launch l = dd ? reduce_launch(ld.rows, Row<T, D, E>::RPW) : stream_launch(ld.rows, Row<T, D, E>::RPW);
        hipLaunchKernelGGL((frontend_bwd_kernel<T, D, E>), dim3(l.grid), dim3(l.block), ld.H * sizeof(float), s, ld,
                           static_cast<const T *>(x_q), static_cast<const T *>(x_k), static_cast<const T *>(x_v), d, eps,
                           static_cast<const T *>(dq), static_cast<const T *>(dk), static_cast<const T *>(dv),
                           static_cast<T *>(dx_q), static_cast<T *>(dx_k), static_cast<T *>(dx_v), dd);
        return status();
    });
}

int mdn_epilogue_fwd(const mdn_shape *shape, const void *o, const void *g, const float *w, float eps, void *y, void *stream) {
    LayerDims ld;
    const int rc = check(shape, &ld);
    if (rc) return rc;
    if (!o || !g || !w || !y) return MDN_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    return dispatch(shape, ld.rows, false, [&](auto t, auto dim, auto el) {
        typedef decltype(t) T;
        constexpr int D = decltype(dim)::value, E = decltype(el)::value;
        const Launch l = stream_launch(ld.rows, Row<T, D, E>::RPW);
        hipLaunchKernelGGL((epilogue_fwd_kernel<T, D, E>), dim3(l.grid), dim3(l.block), 0, s, ld, static_cast<const T *>(o),
                           static_cast<const T *>(g), w, eps, static_cast<T *>(y));
        return status();
    });
}

int mdn_epilogue_bwd(const mdn_shape *shape, const void *o, const void *g, const float *w, float eps, const void *dy,
                     void *d_o, void *dg, float *dw, void *stream) {
    LayerDims ld;
    const int rc = check(shape, &ld);
    if (rc) return rc;
    if (!o || !g || !w || !dy || !d_o || !dg) return MDN_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (dw) hipLaunchKernelGGL(layer_zero_kernel, dim3(1), dim3(256), 0, s, dw, shape->dv);
    return dispatch(shape, ld.rows, dw != nullptr, [&](auto t, auto dim, auto el) {
        typedef decltype(t) T;
        constexpr int D = decltype(dim)::value, E = decltype(el)::value;
        const Launch l = dw ? reduce_launch(ld.rows, Row<T, D, E>::RPW) : stream_launch(ld.rows, Row<T, D, E>::RPW);
        hipLaunchKernelGGL((epilogue_bwd_kernel<T, D, E>), dim3(l.grid), dim3(l.block), 0, s, ld, static_cast<const T *>(o),
                           static_cast<const T *>(g), w, eps, static_cast<const T *>(dy), static_cast<T *>(d_o),
                           static_cast<T *>(dg), dw);
        return status();
    });
}

} // extern "C"
