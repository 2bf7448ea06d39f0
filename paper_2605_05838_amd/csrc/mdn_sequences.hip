// How sequences are laid out in 64-token chunks: the device tables of packed variable-length batches, and the padded
// copies of chunk sizes below 64.  A padding token of such a copy has k = v = q = 0, alpha = mu = 1, beta = 0: by
// Eq. Mt.recurrent / St.recurrent it changes neither S nor M, and with dO = 0 on the padding rows the reverse pass is
// exact as well.
#include "mdn_device.h"
#include "mdn_kernels.h"

namespace mdn {

namespace {

// blockIdx.x = sequence of the list
__global__ __launch_bounds__(64) void seq_tables_kernel(SeqList l, SeqEntry *seqs, ChunkEntry *chunks) {
    const SeqEntry e = l.e[blockIdx.x];
    if (threadIdx.x == 0) seqs[l.first + blockIdx.x] = e;
    const int N = (e.len + 63) / 64;
    for (int n = threadIdx.x; n < N; n += 64)
        chunks[e.cb + n] = ChunkEntry{e.t0 + n * 64, min(64, e.len - n * 64), e.cb * l.H + n, N};
}

// blockIdx.x = token of the list; threads over the heads
__global__ __launch_bounds__(64) void clear_at_starts_kernel(StartList l, float *a, float *b) {
    const size_t row = (size_t)l.t[blockIdx.x] * l.H;
    for (int h = threadIdx.x; h < l.H; h += 64) a[row + h] = b[row + h] = 0.f;
}

// blockIdx.y = tensor
__global__ __launch_bounds__(256) void copy_gates_kernel(const float *a, const float *b, float *dst_a, float *dst_b, long long n) {
    const float *src = blockIdx.y ? b : a;
    float *dst = blockIdx.y ? dst_b : dst_a;
    const long long step = (long long)gridDim.x * 256;
    for (long long x = (long long)blockIdx.x * 256 + threadIdx.x; x < n / 4; x += step)
        reinterpret_cast<float4 *>(dst)[x] = reinterpret_cast<const float4 *>(src)[x];
    if (blockIdx.x == 0 && threadIdx.x < n % 4) dst[n / 4 * 4 + threadIdx.x] = src[n / 4 * 4 + threadIdx.x];
}

// chunks of C < 64 tokens as 64-token tiles: blockIdx.y = tensor, first + blockIdx.x = (b, chunk, i, h) row of the padded tensor
template <bool EXPAND> __global__ __launch_bounds__(64) void chunk_copy_kernel(ChunkCopy c, int first) {
    const TileTensor t = c.t[blockIdx.y];
    const int row = first + (int)blockIdx.x, h = row % c.H, i = (row / c.H) % 64, nc = (row / (c.H * 64)) % c.NC, b = row / (c.H * 64 * c.NC);
    const int words = t.row_bytes / 4, tok = nc * c.C + i;
    const bool real = i < c.C && tok < c.T;
    uint32_t *pad = reinterpret_cast<uint32_t *>(static_cast<char *>(t.padded) + (size_t)row * t.row_bytes);
    uint32_t *full = reinterpret_cast<uint32_t *>(static_cast<char *>(const_cast<void *>(t.full)) +
                                                  (((size_t)b * c.T + (real ? tok : 0)) * c.H + h) * t.row_bytes);
    if (EXPAND) {
        for (int x = threadIdx.x; x < words; x += 64) pad[x] = real ? full[x] : t.pad_word;
    } else if (real) {
        for (int x = threadIdx.x; x < words; x += 64) full[x] = pad[x];
    }
}

} // namespace

hipError_t launch_seq_tables(const SeqList &l, SeqEntry *seqs, ChunkEntry *chunks, hipStream_t s) {
    if (l.n < 1) return hipSuccess;
    if (l.n > kSeqsPerLaunch || l.first < 0 || l.H < 1 || !seqs || !chunks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(seq_tables_kernel, dim3(l.n), dim3(64), 0, s, l, seqs, chunks);
    return hipGetLastError();
}

hipError_t launch_clear_at_starts(const StartList &l, float *a, float *b, hipStream_t s) {
    if (l.n < 1) return hipSuccess;
    if (l.n > kStartsPerLaunch || l.H < 1 || !a || !b) return hipErrorInvalidValue;
    hipLaunchKernelGGL(clear_at_starts_kernel, dim3(l.n), dim3(64), 0, s, l, a, b);
    return hipGetLastError();
}

hipError_t launch_copy_gates(const float *a, const float *b, float *dst_a, float *dst_b, long long n, hipStream_t s) {
    if (n < 1 || !a || !b || !dst_a || !dst_b) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)(n / 1024 + 1 < 1024 ? n / 1024 + 1 : 1024);
    hipLaunchKernelGGL(copy_gates_kernel, dim3(blocks, 2), dim3(256), 0, s, a, b, dst_a, dst_b, n);
    return hipGetLastError();
}

hipError_t launch_chunk_copy(const ChunkCopy &c, bool expand, hipStream_t s) {
    if (c.n < 1) return hipSuccess;
    if (c.n > 12 || c.B < 1 || c.H < 1 || c.T < 1 || (c.C != 16 && c.C != 32) || c.NC != (c.T + c.C - 1) / c.C) return hipErrorInvalidValue;
    for (int k = 0; k < c.n; ++k)
        if (!c.t[k].full || !c.t[k].padded || c.t[k].row_bytes < 4 || c.t[k].row_bytes % 4) return hipErrorInvalidValue;
    const long long rows = (long long)c.B * c.NC * 64 * c.H;
    if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
    // (a launch of 2^32 threads or more reports no error and leaves workgroups out)
    constexpr long long kMost = 1 << 25;
    for (long long first = 0; first < rows; first += kMost) {
        const dim3 grid((unsigned)(rows - first < kMost ? rows - first : kMost), c.n), block(64);
        if (expand) hipLaunchKernelGGL(chunk_copy_kernel<true>, grid, block, 0, s, c, (int)first);
        else hipLaunchKernelGGL(chunk_copy_kernel<false>, grid, block, 0, s, c, (int)first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace mdn
