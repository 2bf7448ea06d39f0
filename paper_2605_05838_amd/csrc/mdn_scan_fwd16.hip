// Launches of the forward scan and of the state reconstruction for 16-bit storage (mdn_scan_fwd16.h).
#include "mdn_scan_fwd16.h"

namespace mdn {

namespace {

template <int DK, int DV, int DVB, bool REBUILD, bool WHOLE, int AHEAD, bool QTILE, bool TOUCH>
__global__ __launch_bounds__(kScanThreads, AHEAD == 1 ? 4 : 2) void scan_fwd16_kernel(Dims d, ScanFwdArgs a, int first) {
    __shared__ ScanFwdLds<DK, DV, DVB, REBUILD, AHEAD, QTILE, TOUCH> lds;
    scan_fwd16<DK, DV, DVB, REBUILD, WHOLE, AHEAD, QTILE, TOUCH>(d, a, first + blockIdx.x, lds);
}

template <int DK, int DV, int DVB, bool REBUILD, bool WHOLE, int AHEAD, bool QTILE, bool TOUCH>
hipError_t launch_w(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    static const size_t spread =
        AHEAD == 1 ? 0 : lds_bytes_for_one_workgroup_per_cu(reinterpret_cast<const void *>(&scan_fwd16_kernel<DK, DV, DVB, REBUILD, WHOLE, AHEAD, QTILE, TOUCH>));
    return launch_in_parts(scan_blocks<DV, DVB>(d), [&](int first, dim3 grid) {
        hipLaunchKernelGGL((scan_fwd16_kernel<DK, DV, DVB, REBUILD, WHOLE, AHEAD, QTILE, TOUCH>), grid, dim3(kScanThreads), spread, s, d, a, first);
    });
}
template <int DK, int DV, int DVB, bool REBUILD, int AHEAD, bool QTILE = false, bool TOUCH = false> hipError_t launch_t(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    return whole_chunks(d) ? launch_w<DK, DV, DVB, REBUILD, true, AHEAD, QTILE, TOUCH>(d, a, s) : launch_w<DK, DV, DVB, REBUILD, false, AHEAD, QTILE, TOUCH>(d, a, s);
}
// Two workgroups per CU where there are more of them than CUs and the operands of one chunk less make them fit (all but the forward
// of heads of 128): a workgroup's start and the latencies of its chain then lie beside another one's work.  One / two per CU, forward
// of heads of 64 in us: 64 x 64 tokens of 16 heads 43.4 / 33.9, 32 x 128 36.1 / 30.8, 32 x 1 024 187 / 182, packed 256 sequences of 30
// tokens of 16 heads 156 / 107.  One chunk ahead costs a single workgroup up to a tenth of a step, so up to one per CU it is two.
// (16 columns have a CU for each workgroup: see scan_dvb.)
template <int DK, int DV, bool REBUILD> hipError_t pick(const Dims &d, const ScanFwdArgs &a, hipStream_t s) {
    const int columns = scan_dvb(d);
    [[maybe_unused]] const size_t chunks = ((size_t)d.nchunks * d.H + d.BH - 1) / d.BH, bytes = call_bytes(d, a.vt_saved, a.states_saved);
    [[maybe_unused]] const bool q_tile = q_tile_pays(columns, DK, d.BH, chunks, bytes, a.vt_saved, a.states_saved);
    if (columns == 16) {
        if constexpr (!REBUILD) {
            if (touch_pays(bytes, false)) return launch_t<DK, DV, 16, false, 2, true, true>(d, a, s);
            if (q_tile) return launch_t<DK, DV, 16, false, 2, true>(d, a, s);
        }
        return launch_t<DK, DV, 16, REBUILD, 2>(d, a, s);
    }
    if constexpr (2 * sizeof(ScanFwdLds<DK, DV, 32, REBUILD, 1>) <= 160 * 1024)
        if (!scan_one_per_cu(d)) return launch_t<DK, DV, 32, REBUILD, 1>(d, a, s);
    if constexpr (!REBUILD && DK == 128)
        if (q_tile) return launch_t<DK, DV, 32, REBUILD, 2, true>(d, a, s);
    return launch_t<DK, DV, 32, REBUILD, 2>(d, a, s);
}

} // namespace

hipError_t launch_scan_fwd16(const Dims &d, const ScanFwdArgs &a, bool rebuild, hipStream_t s) {
    if (!a.coef || !a.k || (rebuild && (!a.vt_saved || !a.states_saved))) return hipErrorInvalidValue;
    if (d.dk == 64 && d.dv == 64) return rebuild ? pick<64, 64, true>(d, a, s) : pick<64, 64, false>(d, a, s);
    if (d.dk == 128 && d.dv == 128) return rebuild ? pick<128, 128, true>(d, a, s) : pick<128, 128, false>(d, a, s);
    return hipErrorInvalidValue;
}

} // namespace mdn
