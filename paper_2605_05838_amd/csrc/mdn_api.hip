// C ABI of the MDN library: argument validation, workspace carving, kernel sequencing.
// Declarations and the contract of every entry point are in include/mdn.h.
#include "../../include/mdn.h"
#include "mdn_kernels.h"

#include <hip/hip_runtime.h>
#include <string.h>
#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <vector>

using namespace mdn;

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

int check_shape(const mdn_shape *s, bool chunked, Dims *d) {
    if (!s) return MDN_ERR_NULL;
    if (s->dtype != MDN_DTYPE_BF16 && s->dtype != MDN_DTYPE_F32) return MDN_ERR_DTYPE;
    if (s->B < 1 || s->T < 1 || s->H < 1) return MDN_ERR_SHAPE;
    if (!((s->dk == 64 && s->dv == 64) || (s->dk == 128 && s->dv == 128))) return MDN_ERR_SHAPE;
    if (chunked && s->C != 64 && s->C != 32 && s->C != 16) return MDN_ERR_SHAPE;
    // (chunks of 16 or 32 tokens run as 64-token tiles: up to 4 rows per token)
    const long long tile = chunked ? 64 / s->C : 1;
    if ((long long)s->B * s->H > (1 << 24) || ((long long)s->B * s->T + 64) * s->H * tile > (1LL << 31) - 1) return MDN_ERR_SHAPE;
    *d = Dims{};
    d->B = s->B; d->T = s->T; d->H = s->H; d->N = (int)(((long long)s->T + 63) / 64); d->BH = s->B * s->H;
    d->n0 = 0; d->n1 = d->N; d->nchunks = (int)((long long)s->B * d->N);
    d->dk = s->dk; d->dv = s->dv; d->dtype = s->dtype; d->scale = s->scale;
    return MDN_OK;
}

// chunk blocks of a call: one per chunk and head
size_t chunk_blocks(const Dims &d) { return (size_t)d.nchunks * d.H; }

bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Carves consecutive 256-byte aligned regions out of the workspace.
struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *b) : base(static_cast<char *>(b)) {}
    void *take(size_t bytes) {
        void *p = base ? base + off : nullptr;
        off += align_up(bytes);
        return p;
    }
};

// 32-bit storage: K^T and, for the reverse pass, operands in other orientations (mdn_kernels.h)
bool wide(const Dims &d) { return d.dtype == MDN_DTYPE_F32; }

struct FwdWs { float *coef; void *KT, *Tm, *Bm; float *carryS, *carryM; size_t total; };

// a state tensor that crosses segment boundaries.  (Packed batches are not split: room for one sequence, so that their
// workspace is never below that of one unbroken sequence of as many tokens.)
size_t carry_bytes(const Dims &d) { return (size_t)(d.packed ? d.H : d.BH) * d.dk * d.dv * sizeof(float); }

FwdWs carve_fwd(const Dims &d, void *ws) {
    const size_t es = d.dtype == MDN_DTYPE_F32 ? 4 : 2, nb = chunk_blocks(d);
    Carver c(ws);
    FwdWs w;
    w.coef = static_cast<float *>(c.take(nb * (size_t)(64 * kCoefBlockCols * sizeof(float))));
    w.KT = wide(d) ? c.take(nb * d.dk * 64 * es) : nullptr;
    w.Tm = c.take(nb * 4096 * es);
    w.Bm = c.take(nb * 4096 * es);
    // states handed from one segment of the sequence to the next when the call is split (see segments())
    w.carryS = static_cast<float *>(c.take(carry_bytes(d)));
    w.carryM = static_cast<float *>(c.take(carry_bytes(d)));
    w.total = c.off;
    return w;
}

// Operands of the reverse pass; lives in the backward workspace or in the buffer a training forward keeps for the
// backward.  16-bit storage: the forward's own.
struct RevOps { float *coef; void *Tm, *Bm, *KT, *QT, *BmT, *TmT; size_t total; };

RevOps carve_rev(const Dims &d, void *p) {
    const size_t es = d.dtype == MDN_DTYPE_F32 ? 4 : 2, nb = chunk_blocks(d);
    Carver c(p);
    RevOps w = {};
    w.coef = static_cast<float *>(c.take(nb * (size_t)(64 * kCoefBlockCols * sizeof(float))));
    if (!wide(d)) {
        w.Tm = c.take(nb * 4096 * es);
        w.Bm = c.take(nb * 4096 * es);
        w.total = c.off;
        return w;
    }
    w.KT = c.take(nb * d.dk * 64 * es);
    w.QT = c.take(nb * d.dk * 64 * es);
    w.BmT = c.take(nb * 4096 * es);
    w.TmT = c.take(nb * 4096 * es);
    w.total = c.off;
    return w;
}

struct BwdWs { RevOps ops; void *dstates, *states, *dstates_lo, *states_lo; float *carryS, *carryM; size_t total; };

// `precise`: room for the rounding remainders of the two state tensors as well (16-bit storage, calls that bring
// adjoints of the final states in; see precise_call)
BwdWs carve_bwd(const Dims &d, void *ws, bool precise) {
    const size_t es = d.dtype == MDN_DTYPE_F32 ? 4 : 2, nb = chunk_blocks(d);
    BwdWs w;
    w.ops = carve_rev(d, ws);
    Carver c(ws);
    c.off = w.ops.total;
    w.dstates = c.take(nb * 2 * d.dk * d.dv * es);
    w.states = c.take(nb * 2 * d.dk * d.dv * es);
    w.dstates_lo = precise ? c.take(nb * 2 * d.dk * d.dv * es) : nullptr;
    w.states_lo = precise ? c.take(nb * 2 * d.dk * d.dv * es) : nullptr;
    w.carryS = static_cast<float *>(c.take(carry_bytes(d)));
    w.carryM = static_cast<float *>(c.take(carry_bytes(d)));
    w.total = c.off;
    return w;
}

size_t elem_size(const Dims &d) { return d.dtype == MDN_DTYPE_F32 ? 4 : 2; }
size_t saved_states_total(const Dims &d) { return chunk_blocks(d) * 2 * d.dk * d.dv * elem_size(d); }

int launch_status(hipError_t e) { return e == hipSuccess ? MDN_OK : MDN_ERR_LAUNCH; }

// ---- optional per-kernel timing: event pairs around every launch while enabled.  The list of pairs is shared by
// all threads of the process and guarded by a mutex.
struct TimedLaunch { int id; hipEvent_t start, stop; };
std::atomic<bool> g_profiling{false};
std::atomic<int> g_profile_period{1};          // every period-th launch is bracketed
std::atomic<unsigned> g_profile_seen{0};       // launches since mdn_profile_begin
std::atomic<int> g_launched[MDN_KERNEL_COUNT]; // all launches per kernel id since mdn_profile_begin
std::mutex g_timed_mutex;
std::vector<TimedLaunch> g_timed;

// this thread is inside the entry point that must not allocate: no timing events, no second stream
thread_local bool t_no_alloc = false;

void count_launch(int id) {
    if (g_profiling.load(std::memory_order_relaxed) && !t_no_alloc) g_launched[id].fetch_add(1, std::memory_order_relaxed);
}

template <typename F> int timed(int id, hipStream_t s, F &&launch) {
    if (t_no_alloc || !g_profiling.load(std::memory_order_relaxed)) return launch_status(launch());
    if (id >= 0 && id < MDN_KERNEL_COUNT) g_launched[id].fetch_add(1, std::memory_order_relaxed);
    const unsigned seen = g_profile_seen.fetch_add(1, std::memory_order_relaxed);
    if (seen % (unsigned)g_profile_period.load(std::memory_order_relaxed) != 0) return launch_status(launch());
    TimedLaunch t{id, nullptr, nullptr};
    if (hipEventCreate(&t.start) != hipSuccess || hipEventCreate(&t.stop) != hipSuccess) return MDN_ERR_LAUNCH;
    const bool r0 = hipEventRecord(t.start, s) == hipSuccess;
    const int rc = launch_status(launch());
    const bool r1 = hipEventRecord(t.stop, s) == hipSuccess;
    try {
        std::lock_guard<std::mutex> lock(g_timed_mutex);
        g_timed.push_back(t);
    } catch (const std::bad_alloc &) {
        (void)hipEventDestroy(t.start);
        (void)hipEventDestroy(t.stop);
        return MDN_ERR_LAUNCH;
    }
    return r0 && r1 ? rc : MDN_ERR_LAUNCH;
}

// ---- splitting a backward call into segments of the sequence.  When the serial reverse scan occupies at most half of
// the CUs (few (batch, head) pairs, long sequences), the gradient kernel of segment i runs beside the scan of segment
// i-1, on a second stream of the library's own: the scan's workgroups leave the other CUs to it.  Adjoints cross a
// segment boundary through two small fp32 buffers in the workspace.  The forward is split on request only: its
// chunk-local kernel takes a twentieth to a seventh of the scan's time, less than the boundaries cost.
std::atomic<int> g_segments{0}; // 0: automatic

// the serial scans of a call would occupy at most half of the CUs
bool few_scan_workgroups(const Dims &d) { return 2 * scan_workgroups(d) <= num_cus(); }

// A boundary costs ~10 us (an event pair, the scan's start and its drain) and a segment hides its gradient launch, ~50 us
// per 1 024 chunk blocks of d = 128: one segment per 1 024.  Where the states must be reconstructed, 16-bit storage does that in the
// reverse scan's launch if the call is not split, and on the second stream if it is: then the gradient launches wait for all of it, and
// less of them is hidden: two segments from 2 400 blocks on, another one per 2 048.  Backward in us, unsplit / 2 / 4 / 8 segments,
// d = 128, states kept; reconstructed; reconstructed, with adjoints of the final states:
//   blocks  1 024 (16 heads, T =  4 096):   132 /   142 /   145 /   181;    146 /   164 /   174 /   223;    224 /   240 /   255 /   311
//   blocks  2 048 (16 heads, T =  8 192):   303 /   284 /   280 /   304;    310 /   333 /   337 /   371;    476 /   477 /   487 /   507
//                 ( 4 heads, T = 32 768):   702 /   719 /   724 /   758;    698 /   692 /   707 /   733;    951 /   916 /   910 /   945
//   blocks  2 504 ( 8 heads, T = 20 032):   546 /   521 /   523 /   554;    517 /   516 /   533 /   557;    766 /   714 /   712 /   752
//   blocks  4 096 (16 heads, T = 16 384):   526 /   486 /   470 /   473;    662 /   628 /   622 /   668;    981 /   885 /   873 /   912
//   blocks  8 192 (16 heads, T = 32 768): 1 085 /   947 /   889 /   858;  1 428 / 1 220 / 1 193 / 1 244;  2 012 / 1 744 / 1 706 / 1 721
// and 421 / 385 / 369 / 410; 413 / 398 / 405 / 438; 534 / 504 / 509 / 530 for 4 096 blocks of d = 64.  (With the reconstruction in
// front of the segments 4 096 blocks of d = 128 took 752 in 4.)  32-bit storage takes four times as long per block (512 blocks, 8
// heads, states kept: 445 / 417 / 433 / 557; 2 048 of d = 64, 4 heads: 1 721 / 1 643 / 1 608 / 1 614; reconstructed 580 / 455 / 472 /
// 644 and 2 296 / 1 697 / 1 662 / 1 682); segments of fewer than 32 chunks are all start and drain.  Forward: 161 / 188 / 194 / 219 for
// the second row, 754 / 781 / 766 / 782 for the last.
long long backward_segments(const Dims &d, bool rebuild) {
    const long long grad = (long long)d.N * d.BH * d.dk * (d.dtype == MDN_DTYPE_F32 ? 4 : 1); // its time, in 1/128 blocks
    const long long k = rebuild && !wide(d) ? (grad / 128 + 1696) / 2048 : grad / (128 * 1024);
    return few_scan_workgroups(d) ? std::min({8LL, d.N / 32LL, k}) : 1;
}
int segments(const Dims &d, bool backward, bool rebuild = false) {
    if (t_no_alloc || d.packed) return 1; // (packed batches: the scans of the sequences run beside each other)
    long long k = g_segments.load(std::memory_order_relaxed);
    if (k <= 0) k = backward ? backward_segments(d, rebuild) : 1;
    k = std::min(k, (long long)d.N / 4);
    return (int)std::max(1LL, std::min(16LL, k));
}

// The library's second stream and its events, one set per device, shared by every call on that device.  A call that
// uses them holds the device's mutex while it ENQUEUES (the kernels themselves run after it has returned): an event
// is recorded and waited for inside one such section, so calls from several host threads cannot interleave their
// record / wait pairs; their work on the second stream is simply ordered one call after the other.
struct Side {
    hipStream_t stream = nullptr;
    std::vector<hipEvent_t> ev;
    std::mutex mutex;
};

// the second stream and n events on the current device (created once, default priority); call with the lock held
Side *side_device() {
    static Side per_device[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    return &per_device[dev];
}
Side *side(int n) {
    Side *xp = side_device();
    if (!xp) return nullptr;
    Side &x = *xp;
    if (!x.stream && hipStreamCreateWithFlags(&x.stream, hipStreamNonBlocking) != hipSuccess) return nullptr;
    try {
        x.ev.reserve(n);
    } catch (const std::bad_alloc &) {
        return nullptr;
    }
    while ((int)x.ev.size() < n) {
        hipEvent_t e;
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return nullptr;
        x.ev.push_back(e);
    }
    return &x;
}

Dims segment(const Dims &d, int i, int k) {
    Dims r = d;
    r.n0 = (int)((long long)d.N * i / k);
    r.n1 = (int)((long long)d.N * (i + 1) / k);
    return r;
}

// ---- the forward over all chunks of the tensors in `c`
struct FwdCall {
    const void *q, *k, *v;
    const float *beta, *alpha, *mu, *eta, *S0, *M0;
    void *o;
    float *S_final, *M_final;
    void *vt_saved, *states_saved, *operands_saved;
};

int run_fwd(const Dims &d, const FwdCall &c, const FwdWs &w, hipStream_t s) {
    int rc;
    IntraArgs ia = {};
    ia.q = c.q; ia.k = c.k; ia.alpha = c.alpha; ia.beta = c.beta; ia.mu = c.mu; ia.eta = c.eta;
    ia.coef = w.coef; ia.KT = w.KT; ia.Tm = w.Tm; ia.Bm = w.Bm;
    if (c.operands_saved) {
        // training forward: one precompute pass writes the reverse pass's operands as well (16-bit storage: they are the same)
        const RevOps ro = carve_rev(d, c.operands_saved);
        ia.coef = ro.coef; ia.KT = ro.KT; ia.QT = ro.QT; ia.BmT = ro.BmT; ia.TmT = ro.TmT;
        if (!wide(d)) ia.Tm = ro.Tm, ia.Bm = ro.Bm;
    }
    ScanFwdArgs sa = {};
    sa.q = c.q; sa.k = c.k; sa.v = c.v; sa.coef = ia.coef; sa.KT = ia.KT; sa.Tm = ia.Tm; sa.Bm = ia.Bm;
    sa.S0 = c.S0; sa.M0 = c.M0; sa.o = c.o; sa.vt_saved = c.vt_saved; sa.states_saved = c.states_saved;
    sa.S_final = c.S_final; sa.M_final = c.M_final;
    const int mode = c.operands_saved && wide(d) ? 2 : 0;
    const int nseg = segments(d, false);
    if (nseg == 1) {
        rc = timed(MDN_KERNEL_INTRA_FWD, s, [&] { return launch_intra(d, mode, ia, s); });
        if (rc) return rc;
        return timed(MDN_KERNEL_SCAN_FWD, s, [&] { return launch_scan_fwd(d, sa, s); });
    }
    // segments: precompute of segment i+1 on the second stream beside the scan of segment i on the caller's
    Side *sdev = side_device();
    if (!sdev) return MDN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(sdev->mutex);
    Side *sd = side(nseg + 1);
    if (!sd) return MDN_ERR_LAUNCH;
    if (hipEventRecord(sd->ev[nseg], s) != hipSuccess || hipStreamWaitEvent(sd->stream, sd->ev[nseg], 0) != hipSuccess)
        return MDN_ERR_LAUNCH; // whatever the caller's stream holds so far comes first
    // (from here on the second stream holds work of this call: whatever happens, the caller's stream waits for it
    //  before the call returns, so that "complete when the stream reaches the end of the call" also holds for a
    //  call that fails half-way)
    for (int i = 0; i < nseg; ++i) {
        const Dims di = segment(d, i, nseg);
        rc = timed(MDN_KERNEL_INTRA_FWD, sd->stream, [&] { return launch_intra(di, mode, ia, sd->stream); });
        const bool joined = hipEventRecord(sd->ev[i], sd->stream) == hipSuccess && hipStreamWaitEvent(s, sd->ev[i], 0) == hipSuccess;
        if (rc) return rc;
        if (!joined) return MDN_ERR_LAUNCH;
        sa.S0 = i == 0 ? c.S0 : w.carryS;
        sa.M0 = i == 0 ? c.M0 : w.carryM;
        sa.S_final = i == nseg - 1 ? c.S_final : w.carryS;
        sa.M_final = i == nseg - 1 ? c.M_final : w.carryM;
        rc = timed(MDN_KERNEL_SCAN_FWD, s, [&] { return launch_scan_fwd(di, sa, s); });
        if (rc) return rc; // (every launch on the second stream so far has been joined above)
    }
    return MDN_OK;
}

// ---- the backward over all chunks of the tensors in `c`, in two steps: what does not depend on the adjoints coming in
// from the right (the reverse pass's operands, the chunk-start states), then the rest
struct BwdCall {
    const void *q, *k, *v;
    const float *beta, *alpha, *mu, *eta, *S0, *M0;
    const void *vt_saved, *states_saved, *operands_saved, *dO;
    const float *dS_final, *dM_final;
    void *dq, *dk, *dv;
    float *dbeta, *dalpha, *dmu, *deta, *dS0, *dM0;
    size_t state_bytes; // of a state tensor of the whole call
};
struct Prepared {
    RevOps ro;
    const void *states;
    enum { DONE, IN_SCAN, BESIDE_SEGMENTS } rebuild; // the states are there, or still to be reconstructed (`how`): in one launch
    RebuildArgs how;                                 // with the reverse scan, or on the second stream beside its segments
};

// Adjoints of the final states that come in from outside can be large against everything dO puts into the states;
// the sums of dk dv products that they enter (the state traces, the products with V~) then carry the 16-bit storage
// rounding of the chunk states and chunk adjoints at full weight.  Such a call keeps the rounding remainders of both
// tensors as well (which also means it reconstructs the states rather than taking the forward's 16-bit copy).
bool precise_call(const Dims &d, const BwdCall &c) {
    return d.dtype == MDN_DTYPE_BF16 && (c.dS_final || c.dM_final);
}

// Whether a state gradient goes where the initial states come from: the reverse scan may then write only when the reconstruction
// has read them all.
bool state_gradients_in_place(const BwdCall &c) {
    auto shared = [&](const float *in, const float *out) {
        const uintptr_t i = reinterpret_cast<uintptr_t>(in), o = reinterpret_cast<uintptr_t>(out);
        return in && out && i < o + c.state_bytes && o < i + c.state_bytes;
    };
    return shared(c.S0, c.dS0) || shared(c.S0, c.dM0) || shared(c.M0, c.dS0) || shared(c.M0, c.dM0);
}

// Whether the reconstruction and the reverse scan of a call that is not split run as one launch (see scan_pair16_kernel):
// below two full rounds of workgroups.  From there on the reconstruction alone runs two to a CU, which it cannot beside the reverse
// scan's LDS.  Forward and backward in us, two launches / one, heads of 128: 8 x 256 tokens of 16 heads (512 workgroups) 107.2 / 109.3,
// 8 x 2 048 677.5 / 677.1; 16 x 256 203.5 / 205.8; 32 x 512 712 / 723; packed 32 768 in 64 sequences 1 404 / 1 428; of 64: 16 x 256
// 99.4 / 101.1, 16 x 1 024 349.7 / 343.0.  32-bit storage has scans of another form.
bool rebuild_in_scan(const Dims &d) {
    return !wide(d) && scan_workgroups(d) < 2 * num_cus();
}

int bwd_prepare(const Dims &d, const BwdCall &c, const BwdWs &w, hipStream_t s, Prepared *out, bool precise, int nseg) {
    int rc;
    // chunk-local operands in the layouts of the reverse pass: kept by the forward, or recomputed
    out->ro = w.ops;
    if (c.operands_saved) {
        out->ro = carve_rev(d, const_cast<void *>(c.operands_saved));
    } else {
        IntraArgs ia = {};
        ia.q = c.q; ia.k = c.k; ia.alpha = c.alpha; ia.beta = c.beta; ia.mu = c.mu; ia.eta = c.eta;
        ia.coef = out->ro.coef; ia.KT = out->ro.KT; ia.QT = out->ro.QT; ia.BmT = out->ro.BmT; ia.TmT = out->ro.TmT;
        ia.Tm = out->ro.Tm; ia.Bm = out->ro.Bm;
        rc = timed(MDN_KERNEL_INTRA_BWD, s, [&] { return launch_intra(d, wide(d) ? 1 : 0, ia, s); });
        if (rc) return rc;
    }
    // chunk-start states: given by the forward, or reconstructed from V~
    out->states = precise ? nullptr : c.states_saved;
    out->rebuild = Prepared::DONE;
    if (!out->states) {
        RebuildArgs ra = {};
        ra.coef = out->ro.coef; ra.k = c.k; ra.KT = out->ro.KT; ra.vt_saved = c.vt_saved; ra.S0 = c.S0; ra.M0 = c.M0;
        ra.states = w.states; ra.states_lo = precise ? w.states_lo : nullptr;
        out->states = w.states;
        out->how = ra;
        if (!state_gradients_in_place(c)) {
            if (nseg > 1) out->rebuild = Prepared::BESIDE_SEGMENTS;
            else if (rebuild_in_scan(d)) out->rebuild = Prepared::IN_SCAN;
            if (out->rebuild != Prepared::DONE) return MDN_OK;
        }
        rc = timed(MDN_KERNEL_REBUILD, s, [&] { return launch_rebuild(d, ra, s); });
        if (rc) return rc;
    }
    return MDN_OK;
}

int bwd_run(const Dims &d, const BwdCall &c, const BwdWs &w, const Prepared &p, hipStream_t s, bool precise, int nseg) {
    int rc;
    const RevOps &ro = p.ro;
    ScanBwdArgs sb = {};
    sb.q = c.q; sb.k = c.k; sb.dO = c.dO; sb.coef = ro.coef; sb.Tm = ro.Tm; sb.Bm = ro.Bm; sb.QT = ro.QT; sb.KT = ro.KT; sb.BmT = ro.BmT;
    sb.TmT = ro.TmT; sb.dS_final = c.dS_final; sb.dM_final = c.dM_final; sb.dv = c.dv; sb.dstates = w.dstates;
    sb.dS0 = c.dS0; sb.dM0 = c.dM0; sb.dstates_lo = precise ? w.dstates_lo : nullptr;
    GradArgs ga = {};
    ga.q = c.q; ga.k = c.k; ga.alpha = c.alpha; ga.beta = c.beta; ga.mu = c.mu; ga.eta = c.eta;
    ga.vt_saved = c.vt_saved; ga.dO = c.dO; ga.dv = c.dv; ga.KT = ro.KT; ga.QT = ro.QT;
    ga.states = p.states; ga.dstates = w.dstates;
    ga.states_lo = precise ? w.states_lo : nullptr; ga.dstates_lo = precise ? w.dstates_lo : nullptr;
    ga.dq = c.dq; ga.dk = c.dk; ga.dalpha = c.dalpha; ga.dbeta = c.dbeta; ga.dmu = c.dmu; ga.deta = c.deta;
    if (nseg == 1) {
        if (p.rebuild == Prepared::IN_SCAN) {
            count_launch(MDN_KERNEL_REBUILD); // (its time stands with the reverse scan's)
            rc = timed(MDN_KERNEL_SCAN_BWD, s, [&] { return launch_rebuild_and_scan_bwd(d, p.how, sb, s); });
        } else {
            rc = timed(MDN_KERNEL_SCAN_BWD, s, [&] { return launch_scan_bwd(d, sb, s); });
        }
        if (rc) return rc;
        return timed(MDN_KERNEL_GRAD, s, [&] { return launch_grad(d, ga, s); });
    }
    // segments, last first: the gradient kernel of segment i on the second stream beside the reverse scan
    // of segment i-1 on the caller's; the caller's stream then waits for the last gradient launch
    Side *sdev = side_device();
    if (!sdev) return MDN_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(sdev->mutex);
    Side *sd = side(nseg + 2);
    if (!sd) return MDN_ERR_LAUNCH;
    rc = MDN_OK;
    if (p.rebuild == Prepared::BESIDE_SEGMENTS) { // in front of the gradient launches, which need it, beside the first scans, which do not
        if (hipEventRecord(sd->ev[nseg + 1], s) != hipSuccess || hipStreamWaitEvent(sd->stream, sd->ev[nseg + 1], 0) != hipSuccess)
            return MDN_ERR_LAUNCH;
        rc = timed(MDN_KERNEL_REBUILD, sd->stream, [&] { return launch_rebuild(d, p.how, sd->stream); });
    }
    for (int i = nseg - 1; i >= 0 && !rc; --i) {
        const Dims di = segment(d, i, nseg);
        sb.dS_final = i == nseg - 1 ? c.dS_final : w.carryS;
        sb.dM_final = i == nseg - 1 ? c.dM_final : w.carryM;
        sb.dS0 = i == 0 ? c.dS0 : w.carryS;
        sb.dM0 = i == 0 ? c.dM0 : w.carryM;
        rc = timed(MDN_KERNEL_SCAN_BWD, s, [&] { return launch_scan_bwd(di, sb, s); });
        if (rc) break;
        if (hipEventRecord(sd->ev[i], s) != hipSuccess || hipStreamWaitEvent(sd->stream, sd->ev[i], 0) != hipSuccess) {
            rc = MDN_ERR_LAUNCH;
            break;
        }
        rc = timed(MDN_KERNEL_GRAD, sd->stream, [&] { return launch_grad(di, ga, sd->stream); });
    }
    // the caller's stream waits for whatever went to the second stream, also when a launch failed on the way
    if (hipEventRecord(sd->ev[nseg], sd->stream) != hipSuccess || hipStreamWaitEvent(s, sd->ev[nseg], 0) != hipSuccess)
        return MDN_ERR_LAUNCH;
    return rc;
}

int bwd_all(const Dims &d, const BwdCall &c, void *workspace, hipStream_t s) {
    const bool precise = precise_call(d, c);
    const BwdWs w = carve_bwd(d, workspace, precise);
    const int nseg = segments(d, true, precise || !c.states_saved); // (asked for once: another thread may change the setting)
    Prepared p;
    const int rc = bwd_prepare(d, c, w, s, &p, precise, nseg);
    return rc ? rc : bwd_run(d, c, w, p, s, precise, nseg);
}

// ---- chunk sizes below 64 (Algorithm 1 lists C in {16, 32, 64}).  The kernels are built around 64-token tiles (four
// waves of 16 tokens, 64-lane coefficient scans), so a chunk of C < 64 tokens runs as one such tile whose rows from C on
// are identity steps of the recurrence (k = v = q = 0, alpha = mu = 1, beta = 0, dO = 0: they change no state and pass
// every adjoint through): the chunk-local coefficients, the triangular solve and the
// state hand-over are exactly those of Algorithm 1 at chunk size C, at 64 / C times the work of the C = 64 path.
// The tokens are expanded into padded copies in the workspace and the results collected from them.
Dims expanded_dims(const Dims &d, int C) {
    Dims e = d;
    const int NC = (d.T + C - 1) / C;
    e.T = NC * 64; e.N = NC; e.n0 = 0; e.n1 = NC; e.nchunks = e.B * NC;
    return e;
}

struct ExpBufs {
    void *q, *k, *v, *o, *vt, *dO, *dq, *dk, *dv;
    float *beta, *alpha, *mu, *eta, *dbeta, *dalpha, *dmu, *deta;
    void *rest;
    size_t total;
};

ExpBufs carve_exp(const Dims &e, bool backward, bool precise, void *p) {
    const size_t es = elem_size(e), rows = (size_t)e.B * e.T * e.H;
    Carver c(p);
    ExpBufs x = {};
    x.q = c.take(rows * e.dk * es);
    x.k = c.take(rows * e.dk * es);
    x.v = c.take(rows * e.dv * es);
    x.vt = c.take(rows * e.dv * es);
    x.beta = static_cast<float *>(c.take(rows * 4));
    x.alpha = static_cast<float *>(c.take(rows * 4));
    x.mu = static_cast<float *>(c.take(rows * 4));
    x.eta = static_cast<float *>(c.take(rows * 4));
    if (!backward) {
        x.o = c.take(rows * e.dv * es);
        x.rest = c.take(carve_fwd(e, nullptr).total);
    } else {
        x.dO = c.take(rows * e.dv * es);
        x.dq = c.take(rows * e.dk * es);
        x.dk = c.take(rows * e.dk * es);
        x.dv = c.take(rows * e.dv * es);
        x.dbeta = static_cast<float *>(c.take(rows * 4));
        x.dalpha = static_cast<float *>(c.take(rows * 4));
        x.dmu = static_cast<float *>(c.take(rows * 4));
        x.deta = static_cast<float *>(c.take(rows * 4));
        x.rest = c.take(carve_bwd(e, nullptr, precise).total);
    }
    x.total = c.off;
    return x;
}

struct ChunkList {
    ChunkCopy c;
    ChunkList(const Dims &d, int C) {
        c = {};
        c.B = d.B; c.T = d.T; c.H = d.H; c.C = C; c.NC = (d.T + C - 1) / C;
    }
    void add(const void *full, void *padded, size_t row_bytes, float pad = 0.f) {
        if (!full || !padded) return;
        TileTensor &t = c.t[c.n++];
        t.full = full; t.padded = padded; t.row_bytes = (int)row_bytes;
        memcpy(&t.pad_word, &pad, 4);
    }
};

int fwd_small_chunks(const Dims &d, int C, const FwdCall &c, void *workspace, hipStream_t s) {
    const Dims e = expanded_dims(d, C);
    const ExpBufs x = carve_exp(e, false, false, workspace);
    const size_t es = elem_size(d);
    ChunkList in(d, C);
    in.add(c.q, x.q, d.dk * es);
    in.add(c.k, x.k, d.dk * es);
    in.add(c.v, x.v, d.dv * es);
    in.add(c.beta, x.beta, 4, 0.f);
    in.add(c.alpha, x.alpha, 4, 1.f);
    in.add(c.mu, x.mu, 4, 1.f);
    in.add(c.eta, x.eta, 4, 1.f);
    int rc = launch_status(launch_chunk_copy(in.c, true, s));
    if (rc) return rc;
    const FwdCall ce = {x.q, x.k, x.v, x.beta, x.alpha, x.mu, c.eta ? x.eta : nullptr, c.S0, c.M0, x.o, c.S_final, c.M_final,
                        c.vt_saved ? x.vt : nullptr, c.states_saved, c.operands_saved};
    rc = run_fwd(e, ce, carve_fwd(e, x.rest), s);
    if (rc) return rc;
    ChunkList out(d, C);
    out.add(c.o, x.o, d.dv * es);
    out.add(c.vt_saved, x.vt, d.dv * es);
    return launch_status(launch_chunk_copy(out.c, false, s));
}

int bwd_small_chunks(const Dims &d, int C, const BwdCall &c, void *workspace, hipStream_t s) {
    const Dims e = expanded_dims(d, C);
    const bool precise = precise_call(d, c);
    const ExpBufs x = carve_exp(e, true, precise, workspace);
    const size_t es = elem_size(d);
    ChunkList in(d, C);
    in.add(c.q, x.q, d.dk * es);
    in.add(c.k, x.k, d.dk * es);
    in.add(c.v, x.v, d.dv * es);
    in.add(c.vt_saved, x.vt, d.dv * es);
    in.add(c.dO, x.dO, d.dv * es);
    in.add(c.beta, x.beta, 4, 0.f);
    in.add(c.alpha, x.alpha, 4, 1.f);
    in.add(c.mu, x.mu, 4, 1.f);
    in.add(c.eta, x.eta, 4, 1.f);
    int rc = launch_status(launch_chunk_copy(in.c, true, s));
    if (rc) return rc;
    const BwdCall ce = {x.q, x.k, x.v, x.beta, x.alpha, x.mu, c.eta ? x.eta : nullptr, c.S0, c.M0, x.vt, c.states_saved,
                        c.operands_saved, x.dO, c.dS_final, c.dM_final, x.dq, x.dk, x.dv, x.dbeta, x.dalpha, x.dmu,
                        c.deta ? x.deta : nullptr, c.dS0, c.dM0, c.state_bytes};
    rc = bwd_all(e, ce, x.rest, s);
    if (rc) return rc;
    ChunkList out(d, C);
    out.add(c.dq, x.dq, d.dk * es);
    out.add(c.dk, x.dk, d.dk * es);
    out.add(c.dv, x.dv, d.dv * es);
    out.add(c.dbeta, x.dbeta, 4);
    out.add(c.dalpha, x.dalpha, 4);
    out.add(c.dmu, x.dmu, 4);
    out.add(c.deta, x.deta, 4);
    return launch_status(launch_chunk_copy(out.c, false, s));
}

// workspace, kept states and kept operands of a call, whatever its chunk size
size_t fwd_ws_call(const Dims &d, const mdn_shape *shape) {
    if (shape->C == 64) return carve_fwd(d, nullptr).total;
    return carve_exp(expanded_dims(d, shape->C), false, false, nullptr).total;
}
size_t bwd_ws_call(const Dims &d, const mdn_shape *shape, bool precise) {
    if (shape->C == 64) return carve_bwd(d, nullptr, precise).total;
    return carve_exp(expanded_dims(d, shape->C), true, precise, nullptr).total;
}

// ---- packed variable-length batches: the sequences lie one after another along T of a [1, T, H, *] tensor; sequence i
// is tokens [cu[i], cu[i+1]).  Every kernel finds its sequence in two small device tables (mdn_kernels.h), so the batch
// is one set of launches: the chunk-parallel kernels over the chunks of all sequences, the scans with one workgroup
// per (sequence, head, dv-block), longest sequences first so that the last workgroups to start are the shortest.
int check_varlen(const mdn_shape *shape, const int32_t *cu, int32_t n_seq, Dims *d) {
    const int rc = check_shape(shape, true, d);
    if (rc) return rc;
    if (shape->C != 64) return MDN_ERR_SHAPE; // (packed batches: chunk size 64 only)
    if (!cu) return MDN_ERR_NULL;
    if (shape->B != 1 || n_seq < 1 || cu[0] != 0 || cu[n_seq] != shape->T) return MDN_ERR_SHAPE;
    for (int i = 0; i < n_seq; ++i)
        if (cu[i + 1] <= cu[i]) return MDN_ERR_SHAPE;
    return MDN_OK;
}

// bytes that a chunk block takes in the workspace of a backward call (see carve_bwd)
size_t bwd_block_bytes(const Dims &d, bool precise) {
    const size_t state = (size_t)2 * d.dk * d.dv; // S and M of a chunk, elements
    return 64 * kCoefBlockCols * sizeof(float) + ((wide(d) ? 2 * d.dk * 64 : 0) + 2 * 4096 + (precise ? 4 : 2) * state) * elem_size(d);
}

// Every sequence has chunk blocks of its own, so sequences far shorter than a chunk need up to 64 times the blocks of
// their tokens, and the remainders of a `precise` backward double the largest part of a block.  A batch that needs too much
// at once runs group by group on one workspace.  A forward's group ends before it needs more than three times the blocks of T
// unbroken tokens, or than 65 536 (1.2 GB of 16-bit storage, d = 128); a backward's before it needs more bytes than 5/4
// of what T unbroken tokens take, or than 512 MiB (3 600 blocks of 16-bit storage, 14 per CU: the boundary between two groups costs a few
// launches and the wait for the longest sequence of the first).  Sequences of 128 tokens and more on average are one group
// unless they are precise; a longer sequence than that is a group of its own, whatever it needs.
struct SeqGroup { int s0, s1; Dims d; }; // sequences [s0, s1); a single one is an ordinary batch of one (no tables)
struct Grouping {
    long long limit, left; // chunks of one group at most; chunks of the groups still to come
    int alone;             // a sequence that is a group of its own, or -1
};
int seq_chunks(const int32_t *cu, int i) { return (int)(((long long)cu[i + 1] - cu[i] + 63) / 64); }
Dims one_sequence(const Dims &d, const int32_t *cu, int i) {
    Dims r = d;
    r.B = 1; r.T = cu[i + 1] - cu[i]; r.BH = d.H; r.N = r.n1 = r.nchunks = seq_chunks(cu, i);
    r.packed = false;
    return r;
}
// The longest sequence of a backward call by itself, before or behind the others, where its gradient kernel can run beside its
// scans (see backward_segments) and that hides more than running them beside the others' scans would: per 1 024 chunk blocks of
// the long one ~44 us hidden, against ~40 us for every group that is added and what the others' scans then take by themselves, ~3.8 us
// a step of their longest or ~0.06 us a chunk block, whichever is more.  (In the unit of a hidden chunk block: 1 000, 88, 3/2.)
// (The line is drawn for gradient launches that are hidden whole.  Behind a reconstruction on the second stream less of them is, 10 to
// 30 us per 1 024 blocks, but on either side of it the two orders are within a tenth.)
// Backward in us, together / alone, 16 heads of 128: 29 500 tokens and 16 of 205 1 370 / 1 248; 31 130 and 1 638 1 374 / 1 248; 60 000 and
// 16 of 300 2 645 / 2 354; 8 heads 851 / 832, 871 / 842, 1 825 / 1 603; 16 heads of 64 898 / 814, 926 / 830, 1 798 / 1 580; near the
// line 100, 20 037 and 63 tokens of 8 heads of 128 524 / 577.  Not taken: 16 384 and 32 of 512, 8 heads 642 / 655; 24 576 and 8 192, 16 heads 1 255 / 1 232.
int long_sequence(const Dims &d, const int32_t *cu, int32_t n_seq) {
    int a = 0;
    for (int i = 1; i < n_seq; ++i)
        if (cu[i + 1] - cu[i] > cu[a + 1] - cu[a]) a = i;
    const Dims r = one_sequence(d, cu, a);
    if (backward_segments(r, true) < 2) return -1;
    long long groups = 0, steps = 0, blocks = 0;
    auto others = [&](int i0, int i1) {
        long long longest = 0;
        for (int i = i0; i < i1; ++i) {
            const long long N = seq_chunks(cu, i);
            longest = std::max(longest, N);
            blocks += N * d.H;
        }
        groups += i1 > i0;
        steps += longest;
    };
    others(0, a);
    others(a + 1, n_seq);
    return (long long)r.N * d.H > 1000 * groups + std::max(88 * steps, 3 * blocks / 2) ? a : -1;
}
Grouping grouping(const Dims &d, const int32_t *cu, int32_t n_seq, bool backward, bool precise) {
    Grouping g{std::max(65536LL / d.H, 3LL * d.N), 0, -1};
    if (backward) {
        const size_t most = std::max((size_t)512 << 20, (size_t)d.N * d.H * bwd_block_bytes(d, false) / 4 * 5);
        g.limit = std::max(1LL, (long long)(most / (d.H * bwd_block_bytes(d, precise))));
    }
    for (int i = 0; i < n_seq; ++i) g.left += seq_chunks(cu, i);
    if (backward && n_seq > 1) g.alone = long_sequence(d, cu, n_seq);
    return g;
}
SeqGroup next_group(const Dims &d, const int32_t *cu, int32_t n_seq, int s0, Grouping *gr) {
    // (as few groups as the limit allows share the chunks evenly)
    const long long groups = (gr->left + gr->limit - 1) / gr->limit, share = (gr->left + groups - 1) / groups;
    const int end = s0 == gr->alone ? s0 + 1 : s0 < gr->alone ? gr->alone : n_seq;
    const int last = std::min(end, s0 + std::max(1, (1 << 24) / d.H));
    long long chunks = 0, longest = 0;
    int i = s0;
    for (; i < last && chunks < share; ++i) {
        const long long N = seq_chunks(cu, i);
        if (i > s0 && chunks + N > gr->limit) break;
        chunks += N;
        longest = std::max(longest, N);
    }
    gr->left -= chunks;
    SeqGroup g{s0, i, d};
    if (i - s0 == 1) {
        g.d = one_sequence(d, cu, s0);
        return g;
    }
    g.d.B = i - s0; g.d.BH = g.d.B * d.H; g.d.N = g.d.n1 = (int)longest; g.d.nchunks = (int)chunks;
    g.d.packed = true;
    return g;
}

// the tables at the start of the workspace (none for a single sequence), the rest behind them
struct PackedWs { SeqEntry *seqs; ChunkEntry *chunks; void *rest; size_t head; };
PackedWs carve_packed(const Dims &d, void *ws) {
    Carver c(ws);
    PackedWs w = {};
    if (d.packed) {
        w.seqs = static_cast<SeqEntry *>(c.take((size_t)d.B * sizeof(SeqEntry)));
        w.chunks = static_cast<ChunkEntry *>(c.take((size_t)d.nchunks * sizeof(ChunkEntry)));
    }
    w.head = c.off;
    w.rest = ws ? static_cast<char *>(ws) + c.off : nullptr;
    return w;
}

// What a packed call brings in and asks for, which decides the form it runs in: without states it may be merged (see
// merge_short); with adjoints of the final states a 16-bit backward is precise (see precise_call).
struct PackedForm { bool backward, states, adjoints; };
bool precise_form(const Dims &d, PackedForm f) { return f.adjoints && d.dtype == MDN_DTYPE_BF16; }

// what the largest group needs
size_t packed_ws_total(const Dims &d, const int32_t *cu, int32_t n_seq, PackedForm f) {
    const bool precise = precise_form(d, f);
    Grouping gr = grouping(d, cu, n_seq, f.backward, precise);
    size_t most = 0;
    for (int s0 = 0; s0 < n_seq;) {
        const SeqGroup g = next_group(d, cu, n_seq, s0, &gr);
        most = std::max(most, carve_packed(g.d, nullptr).head +
                                  (f.backward ? carve_bwd(g.d, nullptr, precise).total : carve_fwd(g.d, nullptr).total));
        s0 = g.s1;
    }
    return most;
}

// builds the tables on the stream and points the group's sizes at them
int packed_tables(SeqGroup *g, const int32_t *cu, const PackedWs &w, hipStream_t s) {
    if (!g->d.packed) return MDN_OK;
    const int n = g->s1 - g->s0;
    std::vector<SeqEntry> e;
    try {
        e.resize(n);
    } catch (const std::bad_alloc &) {
        return MDN_ERR_LAUNCH;
    }
    int cb = 0;
    for (int i = 0; i < n; ++i) {
        const int32_t *c = cu + g->s0 + i;
        e[i] = SeqEntry{c[0], c[1] - c[0], cb, g->s0 + i};
        cb += (e[i].len + 63) / 64;
    }
    std::sort(e.begin(), e.end(), [](const SeqEntry &a, const SeqEntry &b) { return a.len != b.len ? a.len > b.len : a.t0 < b.t0; });
    SeqList l;
    l.H = g->d.H;
    for (l.first = 0; l.first < n; l.first += l.n) {
        l.n = n - l.first < kSeqsPerLaunch ? n - l.first : kSeqsPerLaunch;
        memcpy(l.e, e.data() + l.first, (size_t)l.n * sizeof(SeqEntry));
        if (launch_seq_tables(l, w.seqs, w.chunks, s) != hipSuccess) return MDN_ERR_LAUNCH;
    }
    g->d.seqs = w.seqs;
    g->d.chunks = w.chunks;
    return MDN_OK;
}

// A call on one sequence of a packed batch, as a batch of one: its first token (a row of the [T, H, *] tensors) and its index
// in the state tensors.
struct SeqOffset {
    size_t qk, v, gate, state; // bytes
    SeqOffset(const Dims &d, int token, int seq)
        : qk((size_t)token * d.H * d.dk * elem_size(d)), v((size_t)token * d.H * d.dv * elem_size(d)),
          gate((size_t)token * d.H * sizeof(float)), state((size_t)seq * d.H * d.dk * d.dv * sizeof(float)) {}
    template <typename P> static void move(P *&p, size_t bytes) {
        if (p) p = reinterpret_cast<P *>(reinterpret_cast<uintptr_t>(p) + bytes);
    }
};
FwdCall at_sequence(FwdCall c, const SeqOffset &o) {
    o.move(c.q, o.qk); o.move(c.k, o.qk); o.move(c.v, o.v); o.move(c.o, o.v); o.move(c.vt_saved, o.v);
    o.move(c.beta, o.gate); o.move(c.alpha, o.gate); o.move(c.mu, o.gate); o.move(c.eta, o.gate);
    o.move(c.S0, o.state); o.move(c.M0, o.state); o.move(c.S_final, o.state); o.move(c.M_final, o.state);
    return c;
}
BwdCall at_sequence(BwdCall c, const SeqOffset &o) {
    o.move(c.q, o.qk); o.move(c.k, o.qk); o.move(c.dq, o.qk); o.move(c.dk, o.qk);
    o.move(c.v, o.v); o.move(c.vt_saved, o.v); o.move(c.dO, o.v); o.move(c.dv, o.v);
    o.move(c.beta, o.gate); o.move(c.alpha, o.gate); o.move(c.mu, o.gate); o.move(c.eta, o.gate);
    o.move(c.dbeta, o.gate); o.move(c.dalpha, o.gate); o.move(c.dmu, o.gate); o.move(c.deta, o.gate);
    o.move(c.S0, o.state); o.move(c.M0, o.state); o.move(c.dS_final, o.state); o.move(c.dM_final, o.state);
    o.move(c.dS0, o.state); o.move(c.dM0, o.state);
    return c;
}

// run(sizes of a group, its call, workspace behind its tables) for every group, one after the other on the stream
template <typename C, typename F>
int packed_run(const Dims &d, const int32_t *cu, int32_t n_seq, PackedForm f, const C &c, void *workspace, hipStream_t s, F &&run) {
    Grouping gr = grouping(d, cu, n_seq, f.backward, precise_form(d, f));
    for (int s0 = 0; s0 < n_seq;) {
        SeqGroup g = next_group(d, cu, n_seq, s0, &gr);
        const PackedWs w = carve_packed(g.d, workspace);
        int rc = packed_tables(&g, cu, w, s);
        if (!rc) rc = run(g.d, g.d.packed ? c : at_sequence(c, SeqOffset(d, cu[s0], s0)), w.rest);
        if (rc) return rc;
        s0 = g.s1;
    }
    return MDN_OK;
}

// ---- short sequences without states.  A sequence shorter than a chunk leaves most of its chunk empty.  By Eq.
// Mt.recurrent / St.recurrent a token with alpha = mu = 0 sees nothing of the states before it (e = v, M = -eta k e^T,
// S = -beta M: what a sequence that starts from zero states computes at its first token, whose own alpha and mu multiply
// those zeros) and passes no adjoint back to them.  So a call that neither gives nor asks for states may merge
// neighbouring sequences into one piece, with alpha and mu zeroed (in copies) at the starts inside it; the gradients of
// those gates are zero and are set so.  Pieces hold up to 512 tokens, fewer (down to 128) where the scans of longer ones
// would leave CUs idle; a longer sequence is a piece of its own.  Merging costs 2 launches forward and 3 backward, so it
// is done where it saves at least an eighth of the chunks.  Forward + backward in us, one piece per sequence / merged (16 heads of 128, bf16):
//   32 768 tokens:   512 sequences  2 419 / 1 542;   1 024   3 588 / 1 540;   4 096   12 214 / 1 571
//    4 096 tokens:   128 sequences    454 /   219;     512   1 550 /   210
//    1 024 tokens:    64 sequences    214 /    93
struct Merged { std::vector<int32_t> cu, starts; bool used = false; }; // piece offsets; starts inside the pieces

int merge_short(const Dims &d, const int32_t *cu, int32_t n_seq, Merged *m) {
    if (n_seq == 1) return MDN_OK;
    const long long limit = std::max(128LL, std::min(512LL, (long long)d.T * d.H * (d.dv / 32) / std::max(1, num_cus())));
    long long own = 0, merged = 0;
    try {
        m->cu.assign(1, 0);
        for (int i = 0; i < n_seq; ++i) {
            own += ((long long)cu[i + 1] - cu[i] + 63) / 64;
            if (cu[i] > m->cu.back()) { // the piece holds sequences already
                if (cu[i + 1] - m->cu.back() <= limit) m->starts.push_back(cu[i]);
                else m->cu.push_back(cu[i]);
            }
        }
        m->cu.push_back(cu[n_seq]);
    } catch (const std::bad_alloc &) {
        return MDN_ERR_LAUNCH;
    }
    for (size_t i = 0; i + 1 < m->cu.size(); ++i) merged += ((long long)m->cu[i + 1] - m->cu[i] + 63) / 64;
    m->used = 8 * merged <= 7 * own;
    return MDN_OK;
}

int clear_at_starts(const Dims &d, const Merged &m, float *a, float *b, hipStream_t s) {
    StartList l;
    l.H = d.H;
    const int n = (int)m.starts.size();
    for (int i = 0; i < n; i += l.n) {
        l.n = std::min(n - i, kStartsPerLaunch);
        memcpy(l.t, m.starts.data() + i, (size_t)l.n * sizeof(int));
        if (launch_clear_at_starts(l, a, b, s) != hipSuccess) return MDN_ERR_LAUNCH;
    }
    return MDN_OK;
}

// the copies of alpha and mu at the start of the workspace, the rest behind them
struct MergedWs { float *alpha, *mu; void *rest; size_t head; };
MergedWs carve_merged(const Dims &d, void *ws) {
    Carver c(ws);
    MergedWs w = {};
    w.alpha = static_cast<float *>(c.take((size_t)d.T * d.H * sizeof(float)));
    w.mu = static_cast<float *>(c.take((size_t)d.T * d.H * sizeof(float)));
    w.head = c.off;
    w.rest = ws ? static_cast<char *>(ws) + c.off : nullptr;
    return w;
}
// the workspace of a call of this form, and whether (and how) it is merged
int packed_need(const Dims &d, const int32_t *cu, int32_t n_seq, PackedForm f, Merged *m, size_t *bytes) {
    if (!f.states) {
        const int rc = merge_short(d, cu, n_seq, m);
        if (rc) return rc;
    }
    *bytes = m->used ? carve_merged(d, nullptr).head + packed_ws_total(d, m->cu.data(), (int)m->cu.size() - 1, f)
                     : packed_ws_total(d, cu, n_seq, f);
    return MDN_OK;
}
int merged_gates(const Dims &d, const Merged &m, const float *alpha, const float *mu, const MergedWs &w, hipStream_t s) {
    if (launch_copy_gates(alpha, mu, w.alpha, w.mu, (long long)d.T * d.H, s) != hipSuccess) return MDN_ERR_LAUNCH;
    return clear_at_starts(d, m, w.alpha, w.mu, s);
}

// ---- the forward's workspace as a fixed array in device memory, for callers that cannot allocate.  Every GPU the
// library runs on holds its own copy of the array (at its own address) until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress: the address it returns, per device, is what is passed on.
static __device__ __align__(256) unsigned char scratch[MDN_NOALLOC_SCRATCH_BYTES];

// device address of `scratch` on the current device (asked for once per device, with that device current)
int scratch_address(void **out) {
    static std::mutex mutex;
    static void *per_device[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MDN_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(mutex);
    if (!per_device[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MDN_ERR_DEVICE;
        per_device[dev] = p;
    }
    *out = per_device[dev];
    return MDN_OK;
}

} // namespace

extern "C" {

int mdn_version(void) { return 200; }

int mdn_set_segments(int k) { return g_segments.exchange(k < 0 ? 0 : k); }

int mdn_profile_begin_sampled(int period) {
    if (period < 1) return MDN_ERR_SHAPE;
    g_profile_period.store(period);
    g_profile_seen.store(0);
    for (auto &c : g_launched) c.store(0);
    g_profiling.store(true);
    return MDN_OK;
}

int mdn_profile_begin(void) { return mdn_profile_begin_sampled(1); }

int mdn_profile_launch_counts(int *launched, int n) {
    if (!launched) return MDN_ERR_NULL;
    for (int i = 0; i < n && i < MDN_KERNEL_COUNT; ++i) launched[i] = g_launched[i].load();
    return MDN_OK;
}

int mdn_profile_end(float *ms, int *launches, int n) {
    g_profiling.store(false);
    int rc = MDN_OK;
    std::vector<TimedLaunch> taken;
    {
        std::lock_guard<std::mutex> lock(g_timed_mutex);
        taken.swap(g_timed);
    }
    for (const TimedLaunch &t : taken) {
        float e = 0.f;
        if (hipEventSynchronize(t.stop) != hipSuccess || hipEventElapsedTime(&e, t.start, t.stop) != hipSuccess)
            rc = MDN_ERR_LAUNCH;
        else if (t.id < n) {
            if (ms) ms[t.id] += e;
            if (launches) launches[t.id] += 1;
        }
        if (hipEventDestroy(t.start) != hipSuccess || hipEventDestroy(t.stop) != hipSuccess) rc = MDN_ERR_LAUNCH;
    }
    return rc;
}

const char *mdn_strerror(int code) {
    switch (code) {
    case MDN_OK: return "ok";
    case MDN_ERR_NULL: return "a required pointer is NULL";
    case MDN_ERR_SHAPE: return "unsupported shape (need dk = dv in {64,128}, C in {16,32,64}, sizes >= 1)";
    case MDN_ERR_DTYPE: return "unsupported dtype";
    case MDN_ERR_WORKSPACE: return "workspace too small (or, for mdn_chunk_fwd_noalloc, the shape needs more than its fixed scratch array)";
    case MDN_ERR_ALIGN: return "pointer not 16-byte aligned";
    case MDN_ERR_LAUNCH: return "kernel launch failed";
    case MDN_ERR_DEVICE: return "current device is not gfx950";
    default: return "unknown error code";
    }
}

int mdn_workspace_bytes(const mdn_shape *shape, int which, size_t *bytes_out) {
    Dims d;
    if (!bytes_out) return MDN_ERR_NULL;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    if (which == MDN_WS_FWD) *bytes_out = fwd_ws_call(d, shape);
    else if (which == MDN_WS_BWD) *bytes_out = bwd_ws_call(d, shape, false);
    else if (which == MDN_WS_BWD_STATE_ADJOINTS) *bytes_out = bwd_ws_call(d, shape, d.dtype == MDN_DTYPE_BF16);
    else return MDN_ERR_SHAPE;
    return MDN_OK;
}

int mdn_saved_states_bytes(const mdn_shape *shape, size_t *bytes_out) {
    Dims d;
    if (!bytes_out) return MDN_ERR_NULL;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    *bytes_out = saved_states_total(shape->C == 64 ? d : expanded_dims(d, shape->C));
    return MDN_OK;
}

int mdn_saved_operands_bytes(const mdn_shape *shape, size_t *bytes_out) {
    Dims d;
    if (!bytes_out) return MDN_ERR_NULL;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    *bytes_out = carve_rev(shape->C == 64 ? d : expanded_dims(d, shape->C), nullptr).total;
    return MDN_OK;
}

int mdn_chunk_fwd(const mdn_shape *shape, const void *q, const void *k, const void *v, const float *beta,
                  const float *alpha, const float *mu, const float *eta, const float *S0, const float *M0,
                  void *o, float *S_final, float *M_final, void *vt_saved, void *states_saved,
                  void *operands_saved, void *workspace, size_t workspace_bytes, void *stream) {
    Dims d;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !o || !workspace) return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved, states_saved,
                          operands_saved, workspace};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    if (workspace_bytes < fwd_ws_call(d, shape)) return MDN_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FwdCall c = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved, states_saved, operands_saved};
    if (shape->C != 64) return fwd_small_chunks(d, shape->C, c, workspace, s);
    return run_fwd(d, c, carve_fwd(d, workspace), s);
}

int mdn_chunk_fwd_noalloc(const mdn_shape *shape, const void *q, const void *k, const void *v, const float *beta,
                          const float *alpha, const float *mu, const float *eta, const float *S0, const float *M0,
                          void *o, float *S_final, float *M_final, void *vt_saved, void *stream) {
    Dims d;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !o) return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    if (fwd_ws_call(d, shape) > (size_t)MDN_NOALLOC_SCRATCH_BYTES) return MDN_ERR_WORKSPACE;
    void *ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    // Nothing in the forward's workspace has to start from zero: the chunk-local operands are written in full by the
    // chunk-parallel kernel before the scan reads them, the padded copies of chunks below 64 tokens by the copy kernel.
    FwdCall c = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved, nullptr, nullptr};
    t_no_alloc = true; // one stream, no timing events: nothing below creates a stream, an event or memory
    rc = shape->C != 64 ? fwd_small_chunks(d, shape->C, c, ws, static_cast<hipStream_t>(stream))
                        : run_fwd(d, c, carve_fwd(d, ws), static_cast<hipStream_t>(stream));
    t_no_alloc = false;
    return rc;
}

int mdn_chunk_bwd(const mdn_shape *shape, const void *q, const void *k, const void *v, const float *beta,
                  const float *alpha, const float *mu, const float *eta, const float *S0, const float *M0,
                  const void *vt_saved, const void *states_saved, const void *operands_saved, const void *dO,
                  const float *dS_final,
                  const float *dM_final, void *dq, void *dk, void *dv, float *dbeta, float *dalpha,
                  float *dmu, float *deta, float *dS0, float *dM0, void *workspace, size_t workspace_bytes,
                  void *stream) {
    Dims d;
    int rc = check_shape(shape, true, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !vt_saved || !dO || !dq || !dk || !dv || !dbeta || !dalpha ||
        !dmu || !workspace)
        return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S0, M0, vt_saved, states_saved, operands_saved, dO, dS_final, dM_final,
                          dq, dk, dv, dbeta, dalpha, dmu, deta, dS0, dM0, workspace};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    BwdCall c = {q, k, v, beta, alpha, mu, eta, S0, M0, vt_saved, states_saved, operands_saved, dO, dS_final, dM_final,
                 dq, dk, dv, dbeta, dalpha, dmu, deta, dS0, dM0, (size_t)d.BH * d.dk * d.dv * sizeof(float)};
    if (workspace_bytes < bwd_ws_call(d, shape, precise_call(d, c))) return MDN_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (shape->C != 64) return bwd_small_chunks(d, shape->C, c, workspace, s);
    return bwd_all(d, c, workspace, s);
}

int mdn_workspace_bytes_varlen(const mdn_shape *shape, const int32_t *cu_seqlens, int32_t n_seq, int which, size_t *bytes_out) {
    Dims d;
    if (!bytes_out) return MDN_ERR_NULL;
    const int rc = check_varlen(shape, cu_seqlens, n_seq, &d);
    if (rc) return rc;
    const bool backward = which == MDN_WS_BWD || which == MDN_WS_BWD_NO_STATES || which == MDN_WS_BWD_NO_STATE_ADJOINTS;
    if (!backward && which != MDN_WS_FWD && which != MDN_WS_FWD_NO_STATES) return MDN_ERR_SHAPE;
    // of the forms that such a call may take, the most that one of them needs
    const bool states = which != MDN_WS_FWD_NO_STATES && which != MDN_WS_BWD_NO_STATES, adjoints = which == MDN_WS_BWD;
    size_t most = 0;
    for (int i = 0; i < 1 + states + adjoints; ++i) {
        Merged m;
        size_t bytes = 0;
        const int rf = packed_need(d, cu_seqlens, n_seq, PackedForm{backward, i > 0, i > 1}, &m, &bytes);
        if (rf) return rf;
        most = std::max(most, bytes);
    }
    *bytes_out = most;
    return MDN_OK;
}

int mdn_chunk_fwd_varlen(const mdn_shape *shape, const int32_t *cu_seqlens, int32_t n_seq, const void *q, const void *k,
                         const void *v, const float *beta, const float *alpha, const float *mu, const float *eta,
                         const float *S0, const float *M0, void *o, float *S_final, float *M_final, void *vt_saved,
                         void *workspace, size_t workspace_bytes, void *stream) {
    Dims d;
    int rc = check_varlen(shape, cu_seqlens, n_seq, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !o || !workspace) return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved, workspace};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    const PackedForm form = {false, S0 || M0 || S_final || M_final, false};
    Merged m;
    size_t need = 0;
    rc = packed_need(d, cu_seqlens, n_seq, form, &m, &need);
    if (rc) return rc;
    if (workspace_bytes < need) return MDN_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    FwdCall c = {q, k, v, beta, alpha, mu, eta, S0, M0, o, S_final, M_final, vt_saved, nullptr, nullptr};
    auto run = [&](const Dims &g, const FwdCall &cg, void *ws) { return run_fwd(g, cg, carve_fwd(g, ws), s); };
    if (!m.used) return packed_run(d, cu_seqlens, n_seq, form, c, workspace, s, run);
    const MergedWs w = carve_merged(d, workspace);
    rc = merged_gates(d, m, alpha, mu, w, s);
    if (rc) return rc;
    c.alpha = w.alpha; c.mu = w.mu;
    return packed_run(d, m.cu.data(), (int)m.cu.size() - 1, form, c, w.rest, s, run);
}

int mdn_chunk_bwd_varlen(const mdn_shape *shape, const int32_t *cu_seqlens, int32_t n_seq, const void *q, const void *k,
                         const void *v, const float *beta, const float *alpha, const float *mu, const float *eta,
                         const float *S0, const float *M0, const void *vt_saved, const void *dO, const float *dS_final,
                         const float *dM_final, void *dq, void *dk, void *dv, float *dbeta, float *dalpha, float *dmu,
                         float *deta, float *dS0, float *dM0, void *workspace, size_t workspace_bytes, void *stream) {
    Dims d;
    int rc = check_varlen(shape, cu_seqlens, n_seq, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !vt_saved || !dO || !dq || !dk || !dv || !dbeta || !dalpha || !dmu ||
        !workspace)
        return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S0, M0, vt_saved, dO, dS_final, dM_final, dq, dk, dv, dbeta, dalpha,
                          dmu, deta, dS0, dM0, workspace};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    const PackedForm form = {true, S0 || M0 || dS_final || dM_final || dS0 || dM0, dS_final || dM_final};
    Merged m;
    size_t need = 0;
    rc = packed_need(d, cu_seqlens, n_seq, form, &m, &need);
    if (rc) return rc;
    if (workspace_bytes < need) return MDN_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    BwdCall c = {q, k, v, beta, alpha, mu, eta, S0, M0, vt_saved, nullptr, nullptr, dO, dS_final, dM_final,
                 dq, dk, dv, dbeta, dalpha, dmu, deta, dS0, dM0, (size_t)n_seq * d.H * d.dk * d.dv * sizeof(float)};
    auto run = [&](const Dims &g, const BwdCall &cg, void *ws) { return bwd_all(g, cg, ws, s); };
    if (!m.used) return packed_run(d, cu_seqlens, n_seq, form, c, workspace, s, run);
    const MergedWs w = carve_merged(d, workspace);
    rc = merged_gates(d, m, alpha, mu, w, s);
    if (rc) return rc;
    c.alpha = w.alpha; c.mu = w.mu;
    rc = packed_run(d, m.cu.data(), (int)m.cu.size() - 1, form, c, w.rest, s, run);
    return rc ? rc : clear_at_starts(d, m, dalpha, dmu, s);
}

int mdn_recurrent_step(const mdn_shape *shape, const void *q, const void *k, const void *v, const float *beta,
                       const float *alpha, const float *mu, const float *eta, float *S, float *M, void *o,
                       void *stream) {
    Dims d;
    int rc = check_shape(shape, false, &d);
    if (rc) return rc;
    if (!q || !k || !v || !beta || !alpha || !mu || !S || !M || !o) return MDN_ERR_NULL;
    const void *ptrs[] = {q, k, v, beta, alpha, mu, eta, S, M, o};
    for (const void *p : ptrs)
        if (p && misaligned(p)) return MDN_ERR_ALIGN;
    RecurrentArgs ra = {};
    ra.q = q; ra.k = k; ra.v = v; ra.alpha = alpha; ra.beta = beta; ra.mu = mu; ra.eta = eta;
    ra.S = S; ra.M = M; ra.o = o;
    hipStream_t s = static_cast<hipStream_t>(stream);
    return timed(MDN_KERNEL_RECURRENT, s, [&] { return launch_recurrent(d, ra, s); });
}

} // extern "C"
