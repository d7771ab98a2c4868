// hybrid.hip -- hybrid BP -> CA-SCL decoder (Sec. III, Fig. 3).
//
// The CPU scheduling loop of Fig. 3 becomes two kernels on one stream with no
// host round trip: BP on every frame, which writes the information bits of the
// frames it keeps and appends the others to a device queue (the failed-codeword
// buffer of Fig. 3), and persistent CA-SCL workgroups that read the queue
// length on the device and write the information bits of its frames.  Beside
// them the queue's counter is cleared, and the statistics are gathered where
// they are asked for.  (Compaction, flags and the merge of the information bits
// were kernels of their own, between BP and the list decoder and after it: 64
// frames at 2 dB took 370 us with them, 364 us without; six pipelined batches of
// 65536 7.09 ms, 6.99 ms without.)
#include <atomic>
#include <mutex>

#include "internal.hpp"

// Device memory of hybrid_decode_batch_static: the per-batch state and the
// list decoder's global slice of one call.  Each device the library runs on
// holds its own copy until the process ends; host code reaches it only
// through the address hipGetSymbolAddress returns on that device (the name
// itself is a host-side stand-in).
static constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace polarhip {
namespace {

__global__ void clear_count_kernel(int32_t* count) {
    if (lid_x() == 0) *count = 0;
}

// The statistics of a decoded batch: frames, BP successes, list-decoded frames,
// BP iterations, list-decoded frames whose CRC failed; one set of atomics per
// workgroup.
__global__ __launch_bounds__(256) void stats_kernel(const uint8_t* __restrict__ ok, const int32_t* __restrict__ iters,
                                                    const uint8_t* __restrict__ scl_ok, int64_t B,
                                                    unsigned long long* __restrict__ stats, int grid) {
    __shared__ unsigned long long red[4][4];
    unsigned long long s[4] = {0, 0, 0, 0};  // ok, list-decoded, iterations, CRC failures
    for (int64_t f = gid_x() * 256 + lid_x(); f < B; f += (int64_t)grid * 256) {
        const bool good = ok[f] != 0;
        s[0] += good;
        s[1] += !good;
        s[2] += (unsigned long long)iters[f];
        s[3] += !good && !scl_ok[f];
    }
    for (int i = 0; i < 4; ++i) {
        for (int m = 32; m >= 1; m >>= 1) s[i] += __shfl_xor(s[i], m, 64);
        if ((lid_x() & 63) == 0) red[i][lid_x() >> 6] = s[i];
    }
    __syncthreads();
    if (lid_x() < 4) {
        const int i = lid_x();
        const unsigned long long v = red[i][0] + red[i][1] + red[i][2] + red[i][3];
        if (v) atomicAdd(&stats[i + 1], v);
        if (i == 0 && gid_x() == 0) atomicAdd(&stats[0], (unsigned long long)B);
    }
}

struct HybridWs {
    uint8_t* ok;
    int32_t* iters;
    int32_t* queue;
    int32_t* count;
    uint8_t* scl_ok;
    void* scl_glob;
    size_t total;
};

// per-batch state of B frames from `off`; returns the end offset
size_t carve_batch(int64_t B, size_t off, char* base, HybridWs* w) {
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    const size_t o_ok = take((size_t)B);
    const size_t o_it = take((size_t)B * 4);
    const size_t o_q = take((size_t)B * 4);
    const size_t o_c = take(4);
    const size_t o_s = take((size_t)B);
    if (base) {
        w->ok = reinterpret_cast<uint8_t*>(base + o_ok);
        w->iters = reinterpret_cast<int32_t*>(base + o_it);
        w->queue = reinterpret_cast<int32_t*>(base + o_q);
        w->count = reinterpret_cast<int32_t*>(base + o_c);
        w->scl_ok = reinterpret_cast<uint8_t*>(base + o_s);
    }
    return off;
}

// `slots` copies of the per-batch state followed by one list-decoder slice
size_t carve(int64_t B, const SclPlan& plan, void* base, HybridWs* w, int slots) {
    char* b = static_cast<char*>(base);
    size_t off = 0;
    for (int s = 0; s < slots; ++s) off = carve_batch(B, off, b, w ? &w[s] : nullptr);
    const size_t o_g = off;
    off = align_up(off + plan.glob_per_wg * plan.grid, 256);
    if (b && w)
        for (int s = 0; s < slots; ++s) {
            w[s].scl_glob = plan.glob_per_wg ? (void*)(b + o_g) : nullptr;
            w[s].total = off;
        }
    return off;
}

// BP and list-decoder workgroups per CU in the pipelined hybrid (0: no limit)
std::atomic<int> g_pipe_bp_wgs{0};
std::atomic<int> g_pipe_scl_wgs{0};

// per-batch states in flight in the pipelined hybrid: batch j + kPipeSlots
// reuses batch j's state, so its BP waits for batch j's list decoding (three states
// measured no faster than two: the list decoder and the next BP compete for
// the same CUs, not for the state)
constexpr int kPipeSlots = 2;

// the events (BP done and SCL done, per slot) of the calling thread on the
// current device, created on first use and kept: a later call re-records them
// after every wait that an earlier call enqueued on them
polar_status pipeline_events(hipEvent_t** out) {
    constexpr int kMaxDev = 64;
    thread_local hipEvent_t ev[kMaxDev][2 * kPipeSlots] = {};
    int dev = 0;
    polar_status st = hip_check(hipGetDevice(&dev), "get device");
    if (st != POLAR_OK) return st;
    if (dev < 0 || dev >= kMaxDev) return set_error(POLAR_ERR_UNSUPPORTED, "device index out of range");
    for (int i = 0; i < 2 * kPipeSlots; ++i)
        if (!ev[dev][i] &&
            (st = hip_check(hipEventCreateWithFlags(&ev[dev][i], hipEventDisableTiming), "event create")) != POLAR_OK)
            return st;
    *out = ev[dev];
    return POLAR_OK;
}

// BP on `stream`: it writes the information bits of the frames it keeps straight
// to info_hat and queues the others
polar_status enqueue_bp_part(const polar_code* code, const float* llr, int64_t B, const bp_params* p,
                             const HybridWs& w, uint8_t* info_hat, uint8_t* used_scl, hipStream_t stream,
                             int wgs_per_cu = 0) {
    BpQueue q;
    q.ids = w.queue;
    q.count = w.count;
    q.used_scl = used_scl;
    return launch_bp(code, llr, B, p, nullptr, nullptr, w.iters, w.ok, stream, wgs_per_cu, info_hat, q);
}

// the queue's length back to 0 (a kernel, so that the work can be captured)
polar_status enqueue_clear(const HybridWs& w, hipStream_t stream) {
    hipLaunchKernelGGL(clear_count_kernel, dim3(1), dim3(64), 0, stream, w.count);
    return hip_check(hipGetLastError(), "clear launch");
}

// CA-SCL on the queued frames, writing their information bits, and the
// statistics, on `stream`
polar_status enqueue_scl_part(const polar_code* code, const SclPlan& plan, const float* llr, int64_t B, int L,
                              const HybridWs& w, uint8_t* info_hat, int64_t* stats, hipStream_t stream) {
    SclOut out;
    out.info = info_hat;
    out.crc_ok = w.scl_ok;
    polar_status st = launch_scl(code, plan, llr, L, SclWork::list(w.queue, w.count, 0), out, w.scl_glob, stream);
    if (st != POLAR_OK || !stats) return st;
    int64_t grid = (B + 255) / 256;
    if (grid > 64) grid = 64;
    hipLaunchKernelGGL(stats_kernel, dim3((unsigned)grid), dim3(256), 0, stream, w.ok, w.iters, w.scl_ok, B,
                       reinterpret_cast<unsigned long long*>(stats), (int)grid);
    return hip_check(hipGetLastError(), "stats launch");
}

}  // namespace
}  // namespace polarhip

using namespace polarhip;

static polar_status check_bp_params(const polar_code* code, const bp_params* p) {
    if (p->max_iter < 1) return set_error(POLAR_ERR_INVALID_ARG, "max_iter must be >= 1");
    if (p->stop < 0 || p->stop > 2) return set_error(POLAR_ERR_INVALID_ARG, "stop must be 0, 1 or 2");
    if (p->stop == 2 && code->c == 0) return set_error(POLAR_ERR_INVALID_ARG, "CRC stop needs a code with a CRC");
    if (!(p->llr_max > 0.0f)) return set_error(POLAR_ERR_INVALID_ARG, "llr_max must be > 0");
    if (p->rule != 0 && p->rule != 1) return set_error(POLAR_ERR_INVALID_ARG, "rule must be 0 or 1");
    if (p->rule == 1 && p->weights) return set_error(POLAR_ERR_UNSUPPORTED, "the exact rule has no weighted form");
    if (p->weights && p->weight_iters < p->max_iter) return set_error(POLAR_ERR_INVALID_ARG, "weight_iters < max_iter");
    if (p->weight_layout != 0 && p->weight_layout != 1) return set_error(POLAR_ERR_INVALID_ARG, "weight_layout must be 0 or 1");
    if (p->variant != 0 && !bp_variant_supported(code->n, p->variant))
        return set_error(POLAR_ERR_INVALID_ARG, "unknown BP variant");
    return POLAR_OK;
}

extern "C" polar_status polar_workspace_size(const polar_code* code, int64_t B, int32_t L, const bp_params* params,
                                             size_t* bytes) {
    if (!code || !bytes || B < 0) return set_error(POLAR_ERR_INVALID_ARG, "polar_workspace_size: bad argument");
    SclPlan plan;
    polar_status st = scl_plan(code, L, B > 0 ? B : 1, &plan);
    if (st != POLAR_OK) return st;
    *bytes = params ? carve(B, plan, nullptr, nullptr, 1) : plan.glob_per_wg * plan.grid;
    return ok_status();
}

extern "C" polar_status polar_pipeline_workspace_size(const polar_code* code, int64_t B, int32_t L,
                                                      const bp_params* params, size_t* bytes) {
    if (!code || !bytes || !params || B < 0)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_pipeline_workspace_size: bad argument");
    SclPlan plan;
    polar_status st = scl_plan(code, L, B > 0 ? B : 1, &plan);
    if (st != POLAR_OK) return st;
    *bytes = carve(B, plan, nullptr, nullptr, kPipeSlots);
    return ok_status();
}

namespace {

std::atomic<int> g_graph_mode{1};

polar_status enqueue_hybrid(const polar_code* code, const SclPlan& plan, const float* llr, int64_t B,
                            const bp_params* p, int32_t L, uint8_t* info_hat, uint8_t* used_scl, int64_t* stats,
                            void* ws, hipStream_t stream) {
    HybridWs w;
    carve(B, plan, ws, &w, 1);
    polar_status st = enqueue_clear(w, stream);
    if (st == POLAR_OK) st = enqueue_bp_part(code, llr, B, p, w, info_hat, used_scl, stream);
    if (st != POLAR_OK) return st;
    return enqueue_scl_part(code, plan, llr, B, L, w, info_hat, stats, stream);
}

}  // namespace

extern "C" polar_status hybrid_decode_batch(const polar_code* code, const float* llr, int64_t B,
                                            const bp_params* p, int32_t L, uint8_t* info_hat, uint8_t* used_scl,
                                            int64_t* stats, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (!code || !p) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch: null code or params");
    if (B < 0 || B > (int64_t)INT32_MAX) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch: bad batch size");
    if (B > 0 && (!llr || !info_hat)) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch: null buffer");
    polar_status st = check_bp_params(code, p);
    if (st != POLAR_OK) return st;
    SclPlan plan;
    if ((st = scl_plan(code, L, B > 0 ? B : 1, &plan)) != POLAR_OK) return st;
    const size_t need = carve(B, plan, nullptr, nullptr, 1);
    if (!ws || ws_bytes < need) return set_error(POLAR_ERR_WORKSPACE, "hybrid_decode_batch: workspace too small");
    if (B == 0) return ok_status();
    // Direct launches on the caller's stream (recorded there if it is being
    // captured).  Replaying a captured graph of these three or four kernels cost
    // 29 us of host time a call, launching them 13 us; with six and more kernels
    // it had been the other way round.
    st = enqueue_hybrid(code, plan, llr, B, p, L, info_hat, used_scl, stats, ws, stream);
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status polar_set_hybrid_graphs(int32_t mode) {
    if (mode != 0 && mode != 1) return set_error(POLAR_ERR_INVALID_ARG, "polar_set_hybrid_graphs: mode must be 0 or 1");
    g_graph_mode.store(mode);
    return ok_status();
}

extern "C" int32_t polar_get_hybrid_graphs(void) { return g_graph_mode.load(); }

// device address of `scratch` on the current device, looked up once per device
static polar_status static_scratch(void** out) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static void* addr[kMaxDev] = {};
    int dev = 0;
    polar_status st = hip_check(hipGetDevice(&dev), "get device");
    if (st != POLAR_OK) return st;
    if (dev < 0 || dev >= kMaxDev) return set_error(POLAR_ERR_UNSUPPORTED, "device index out of range");
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        st = hip_check(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "scratch symbol address");
        if (st != POLAR_OK) return st;
        if (!p) return set_error(POLAR_ERR_DEVICE, "scratch symbol address is null");
        addr[dev] = p;
    }
    *out = addr[dev];
    return POLAR_OK;
}

extern "C" polar_status hybrid_decode_batch_static(const polar_code* code, const float* llr, int64_t B,
                                                   const bp_params* p, int32_t L, uint8_t* info_hat,
                                                   uint8_t* used_scl, int64_t* stats, hipStream_t stream) {
    if (!code || !p) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch_static: null code or params");
    if (B < 0 || B > (int64_t)INT32_MAX)
        return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch_static: bad batch size");
    if (B > 0 && (!llr || !info_hat))
        return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_batch_static: null buffer");
    polar_status st = check_bp_params(code, p);
    if (st != POLAR_OK) return st;
    SclPlan plan;
    if ((st = scl_plan(code, L, B > 0 ? B : 1, &plan)) != POLAR_OK) return st;
    // Which batches this entry point takes is part of its interface: the
    // per-batch state with N bytes of decisions a frame and one list decode's
    // share have to fit.  The decoders need less (no decisions, a share for
    // one frame at a time no larger), so what is taken fits with room for more
    // shares.
    SclPlan least;
    if ((st = scl_plan(code, L, B > 0 ? B : 1, &least, 1)) != POLAR_OK) return st;
    const size_t batch = carve_batch(B, 0, nullptr, nullptr);
    const size_t need = batch + align_up((size_t)B * code->N, 256) + scl_static_share(code->n, L);
    if (need > kStaticScratchBytes)
        return set_error(POLAR_ERR_INVALID_ARG,
                         "hybrid_decode_batch_static: batch needs " + std::to_string(need) +
                             " bytes of scratch, the maximum is " + std::to_string(kStaticScratchBytes));
    // as many persistent workgroups as slices fit in the rest (at least one)
    if (batch + plan.glob_per_wg * plan.grid > kStaticScratchBytes) {
        plan = least;
        const size_t fit = (kStaticScratchBytes - batch) / plan.glob_per_wg;
        if ((size_t)plan.grid > fit) plan.grid = (int)fit;
    }
    if (B == 0) return ok_status();
    void* ws = nullptr;
    if ((st = static_scratch(&ws)) != POLAR_OK) return st;
    HybridWs w;
    carve(B, plan, ws, &w, 1);
    if ((st = enqueue_clear(w, stream)) != POLAR_OK) return st;
    if ((st = enqueue_bp_part(code, llr, B, p, w, info_hat, used_scl, stream)) != POLAR_OK) return st;
    if ((st = enqueue_scl_part(code, plan, llr, B, L, w, info_hat, stats, stream)) != POLAR_OK) return st;
    return ok_status();
}

extern "C" polar_status hybrid_decode_pipelined(const polar_code* code, int64_t nbatch, const float* const* llr,
                                                int64_t B, const bp_params* p, int32_t L, uint8_t* const* info_hat,
                                                uint8_t* const* used_scl, int64_t* stats, void* ws, size_t ws_bytes,
                                                hipStream_t stream_bp, hipStream_t stream_scl) {
    if (!code || !p) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_pipelined: null code or params");
    if (nbatch < 0 || B < 0 || B > (int64_t)INT32_MAX)
        return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_pipelined: bad batch count or size");
    if (stream_bp == stream_scl) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_pipelined: streams must differ");
    if (nbatch > 0 && B > 0) {
        if (!llr || !info_hat) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_pipelined: null pointer array");
        for (int64_t j = 0; j < nbatch; ++j)
            if (!llr[j] || !info_hat[j]) return set_error(POLAR_ERR_INVALID_ARG, "hybrid_decode_pipelined: null buffer");
    }
    polar_status st = check_bp_params(code, p);
    if (st != POLAR_OK) return st;
    SclPlan plan;
    if ((st = scl_plan(code, L, B > 0 ? B : 1, &plan)) != POLAR_OK) return st;
    // Wavefronts before one takes several frames.  Beside the BP of a long batch
    // their number matters more than their latency: four per CU (six batches of
    // 65536, 1600 list-decoded: 7.04 ms, against 7.34 ms with eight; L = 8, four
    // batches of 8192, N = 512, 2181 list-decoded: 1002 us, with eight 1014).  With
    // L = 32 the list decoding of shorter batches is the longer of the two: eight
    // below 256 frames a CU (four batches of 16384, N = 1024, 1367 list-decoded:
    // 2775 us with four, 2380 with eight), as many as alone up to 64 a CU (8192, N =
    // 512, 2181: 1455 with eight, 1306 with twelve; but 32768, N = 1024, 2700: 3655
    // and 4113)
    const int64_t cus = device_cu_count();
    if (L != 32 || B >= 256 * cus) plan.target = (int)(4 * cus);
    else if (B > 64 * cus && plan.target > 8 * cus) plan.target = (int)(8 * cus);
    // fewer persistent list-decoder workgroups (each walks more of the queue)
    // use fewer global slices, so the workspace size query stays an upper bound
    if (const int cap_wgs = g_pipe_scl_wgs.load(); cap_wgs > 0) {
        const int64_t cap = (int64_t)device_cu_count() * cap_wgs;
        if (plan.grid > cap) plan.grid = (int)(cap > 0 ? cap : 1);
    }
    const size_t need = carve(B, plan, nullptr, nullptr, kPipeSlots);
    if (!ws || ws_bytes < need) return set_error(POLAR_ERR_WORKSPACE, "hybrid_decode_pipelined: workspace too small");
    if (nbatch == 0 || B == 0) return ok_status();
    HybridWs w[kPipeSlots];
    carve(B, plan, ws, w, kPipeSlots);
    hipEvent_t* ev = nullptr;
    if ((st = pipeline_events(&ev)) != POLAR_OK) return st;
    hipEvent_t* bp_done = ev;
    hipEvent_t* scl_done = ev + kPipeSlots;
    // the first batches must not start before work already queued on stream_scl
    // has finished with the shared list-decoder slice of an earlier call
    if (st == POLAR_OK) st = hip_check(hipEventRecord(scl_done[0], stream_scl), "event record");
    if (st == POLAR_OK) st = hip_check(hipStreamWaitEvent(stream_bp, scl_done[0], 0), "stream wait");
    for (int64_t j = 0; j < nbatch && st == POLAR_OK; ++j) {
        const int s = (int)(j % kPipeSlots);
        // the queue of slot s is empty: cleared here for the first batches, by
        // stream_scl behind the list decoding that read it for the later ones
        if (j >= kPipeSlots) st = hip_check(hipStreamWaitEvent(stream_bp, scl_done[s], 0), "stream wait");
        else st = enqueue_clear(w[s], stream_bp);
        if (st == POLAR_OK)
            st = enqueue_bp_part(code, llr[j], B, p, w[s], info_hat[j], used_scl ? used_scl[j] : nullptr, stream_bp,
                                 g_pipe_bp_wgs.load());
        if (st == POLAR_OK) st = hip_check(hipEventRecord(bp_done[s], stream_bp), "event record");
        if (st == POLAR_OK) st = hip_check(hipStreamWaitEvent(stream_scl, bp_done[s], 0), "stream wait");
        if (st == POLAR_OK)
            st = enqueue_scl_part(code, plan, llr[j], B, L, w[s], info_hat[j], stats, stream_scl);
        if (st == POLAR_OK) st = enqueue_clear(w[s], stream_scl);
        if (st == POLAR_OK) st = hip_check(hipEventRecord(scl_done[s], stream_scl), "event record");
    }
    if (st == POLAR_OK)
        st = hip_check(hipStreamWaitEvent(stream_bp, scl_done[(int)((nbatch - 1) % kPipeSlots)], 0), "stream wait");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status polar_set_pipeline_bp_occupancy(int32_t wgs_per_cu) {
    if (wgs_per_cu < 0 || wgs_per_cu > 64)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_set_pipeline_bp_occupancy: must be in [0, 64]");
    g_pipe_bp_wgs.store(wgs_per_cu);
    return ok_status();
}

extern "C" int32_t polar_get_pipeline_bp_occupancy(void) { return g_pipe_bp_wgs.load(); }

extern "C" polar_status polar_set_pipeline_scl_occupancy(int32_t wgs_per_cu) {
    if (wgs_per_cu < 0 || wgs_per_cu > 64)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_set_pipeline_scl_occupancy: must be in [0, 64]");
    g_pipe_scl_wgs.store(wgs_per_cu);
    return ok_status();
}

extern "C" int32_t polar_get_pipeline_scl_occupancy(void) { return g_pipe_scl_wgs.load(); }
