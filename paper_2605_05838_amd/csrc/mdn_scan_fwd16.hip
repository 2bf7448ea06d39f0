// Launches of the forward scan and of the state reconstruction for 16-bit storage (mdn_scan_fwd16.h).
#include "mdn_scan_fwd16.h"

namespace mdn {

namespace {

template <int DK, int DV, int DVB, bool REBUILD, bool WHOLE>
__global__ __launch_bounds__(kScanThreads) void scan_fwd16_kernel(Dims d, ScanFwdArgs a) {
    __shared__ ScanFwdLds<DK, DV, DVB, REBUILD> lds;
    scan_fwd16<DK, DV, DVB, REBUILD, WHOLE>(d, a, blockIdx.x, lds);
}

template <int DK, int DV, int DVB, bool REBUILD> hipError_t launch_t(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    constexpr int G = DV / DVB;
    const dim3 grid(((d.BH + 7) / 8) * 8 * G), block(kScanThreads);
    if (whole_chunks(d)) hipLaunchKernelGGL((scan_fwd16_kernel<DK, DV, DVB, REBUILD, true>), grid, block, 0, s, d, a);
    else hipLaunchKernelGGL((scan_fwd16_kernel<DK, DV, DVB, REBUILD, false>), grid, block, 0, s, d, a);
    return hipGetLastError();
}
template <int DK, int DV, bool REBUILD> hipError_t pick_dvb(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    return scan_dvb(d) == 16 ? launch_t<DK, DV, 16, REBUILD>(d, a, s) : launch_t<DK, DV, 32, REBUILD>(d, a, s);
}

} // namespace

hipError_t launch_scan_fwd16(const Dims &d, const ScanFwdArgs &a, bool rebuild, hipStream_t s) {
    if (!a.coef || !a.k || (rebuild && (!a.vt_saved || !a.states_saved))) return hipErrorInvalidValue;
    if (d.dk == 64 && d.dv == 64) return rebuild ? pick_dvb<64, 64, true>(d, a, s) : pick_dvb<64, 64, false>(d, a, s);
    if (d.dk == 128 && d.dv == 128) return rebuild ? pick_dvb<128, 128, true>(d, a, s) : pick_dvb<128, 128, false>(d, a, s);
    return hipErrorInvalidValue;
}

} // namespace mdn
