// Launches of the reverse scan for 16-bit storage (mdn_scan_bwd16.h), alone or together with the state reconstruction.
#include "mdn_scan_bwd16.h"
#include "mdn_scan_fwd16.h"

namespace mdn {

namespace {

template <int DK, int DV, int DVB, bool WHOLE, int AHEAD, bool TOUCH>
__global__ __launch_bounds__(kScanThreads, AHEAD == 1 ? 4 : 2) void scan_bwd16_kernel(Dims d, ScanBwdArgs a, int first) {
    __shared__ ScanBwdLds<DK, DV, DVB, AHEAD, TOUCH> lds;
    scan_bwd16<DK, DV, DVB, WHOLE, AHEAD, TOUCH>(d, a, first + blockIdx.x, lds);
}

// Both at once: the first half of the workgroups walks the reverse scan, the second half (its steps are shorter) the
// reconstruction.  Neither needs anything of the other.  One launch after the other, 3 x 1 500 tokens of 8 heads of 64 take
// 20 + 29 us with 96 of the 256 CUs at work; together the shorter chain costs nothing.  Up to two rounds of workgroups the
// second half's start as the first half's end, where the last round would leave CUs empty (see rebuild_in_scan).  Forward and
// backward in us, two launches / one: 3 x 1 500, 8 heads of 64 122 / 105; 2 048, 8 heads of 128 133 / 109; 300, 16 heads 57 / 50;
// 4 x 1 024, 16 heads 188 / 182; packed 24 sequences of 100 tokens, 16 heads of 128 (320 workgroups) 161 / 149.
template <int DK, int DV, int DVB, bool WHOLE>
__global__ __launch_bounds__(kScanThreads) void scan_pair16_kernel(Dims d, ScanBwdArgs b, ScanFwdArgs f) {
    typedef ScanBwdLds<DK, DV, DVB, 2> LB;
    typedef ScanFwdLds<DK, DV, DVB, true, 2> LF;
    __shared__ __align__(16) char lds[sizeof(LB) > sizeof(LF) ? sizeof(LB) : sizeof(LF)];
    const int half = gridDim.x / 2, block = blockIdx.x;
    if (block < half) scan_bwd16<DK, DV, DVB, WHOLE, 2, false>(d, b, block, *reinterpret_cast<LB *>(lds));
    else scan_fwd16<DK, DV, DVB, true, WHOLE, 2, false, false>(d, f, block - half, *reinterpret_cast<LF *>(lds));
}

template <int DK, int DV, int DVB, int AHEAD, bool TOUCH = false> hipError_t launch_t(const Dims &d, const ScanBwdArgs &a, hipStream_t s) {
    return launch_in_parts(scan_blocks<DV, DVB>(d), [&](int first, dim3 grid) {
        const dim3 block(kScanThreads);
        if (whole_chunks(d)) hipLaunchKernelGGL((scan_bwd16_kernel<DK, DV, DVB, true, AHEAD, TOUCH>), grid, block, 0, s, d, a, first);
        else hipLaunchKernelGGL((scan_bwd16_kernel<DK, DV, DVB, false, AHEAD, TOUCH>), grid, block, 0, s, d, a, first);
    });
}
// Two workgroups per CU as in the forward (heads of 64), one / two in us, forward with kept states and backward: 64 x 64 tokens of 16
// heads 98.8 / 88.3, 32 x 64 55.0 / 49.8, 32 x 128 87.0 / 81.2, 32 x 1 024 604 / 603.
template <int DK, int DV> hipError_t pick(const Dims &d, const ScanBwdArgs &a, hipStream_t s) {
    if (scan_dvb(d) == 16)
        return touch_pays(call_bytes(d, false, true), true) ? launch_t<DK, DV, 16, 2, true>(d, a, s) : launch_t<DK, DV, 16, 2>(d, a, s);
    if constexpr (2 * sizeof(ScanBwdLds<DK, DV, 32, 1>) <= 160 * 1024)
        if (!scan_one_per_cu(d)) return launch_t<DK, DV, 32, 1>(d, a, s);
    return launch_t<DK, DV, 32, 2>(d, a, s);
}
template <int DK, int DV, int DVB> hipError_t launch_pair_t(const Dims &d, const ScanBwdArgs &b, const ScanFwdArgs &f, hipStream_t s) {
    const int blocks = scan_blocks<DV, DVB>(d);
    if (2 * blocks > kScanBlocks) { // (a packed batch with a long sequence among a million: not worth parts of both)
        const hipError_t e = launch_scan_fwd16(d, f, true, s);
        return e == hipSuccess ? launch_t<DK, DV, DVB, 2>(d, b, s) : e;
    }
    const dim3 grid(2 * blocks), block(kScanThreads);
    if (whole_chunks(d)) hipLaunchKernelGGL((scan_pair16_kernel<DK, DV, DVB, true>), grid, block, 0, s, d, b, f);
    else hipLaunchKernelGGL((scan_pair16_kernel<DK, DV, DVB, false>), grid, block, 0, s, d, b, f);
    return hipGetLastError();
}
template <int DK, int DV> hipError_t pick_pair(const Dims &d, const ScanBwdArgs &b, const ScanFwdArgs &f, hipStream_t s) {
    return scan_dvb(d) == 16 ? launch_pair_t<DK, DV, 16>(d, b, f, s) : launch_pair_t<DK, DV, 32>(d, b, f, s);
}

bool operands_there(const ScanBwdArgs &a) { return a.coef && a.q && a.k && a.dO && a.Bm && a.Tm; }

} // namespace

hipError_t launch_scan_bwd16(const Dims &d, const ScanBwdArgs &a, hipStream_t s) {
    if (!operands_there(a)) return hipErrorInvalidValue;
    if (d.dk == 64 && d.dv == 64) return pick<64, 64>(d, a, s);
    if (d.dk == 128 && d.dv == 128) return pick<128, 128>(d, a, s);
    return hipErrorInvalidValue;
}

hipError_t launch_rebuild_and_scan_bwd(const Dims &d, const RebuildArgs &r, const ScanBwdArgs &b, hipStream_t s) {
    const ScanFwdArgs f = rebuild_args(r);
    if (d.dtype != 0 || !operands_there(b) || !f.vt_saved || !f.states_saved) return hipErrorInvalidValue;
    if (d.dk == 64 && d.dv == 64) return pick_pair<64, 64>(d, b, f, s);
    if (d.dk == 128 && d.dv == 128) return pick_pair<128, 128>(d, b, f, s);
    return hipErrorInvalidValue;
}

} // namespace mdn
