// mixed.hip -- hybrid decoding of ragged batches that mix several codes
// (block lengths and rates), as one device pipeline or one replayed hipGraph.
//
// A call: a one-thread kernel stores the call's arguments in a device block;
// counters are cleared by a kernel (no memset node, so the pipeline can be
// captured); a bucketing kernel appends every frame id to the list of its
// block length; then, per block length, as concurrent branches on the plan's
// streams: a persistent BP kernel walks the list (its length read on the
// device) decoding every frame with its own code and appends the frames whose
// verdict is not ok to their code's queue, and a persistent CA-SCL kernel
// drains the queues of the group's codes (a wavefront decodes several frames
// of one code at once).  Both write their frames' information bits; after the
// branches join, a kernel writes the list-decoder flags and the statistics.
// (Codes shorter than 32 bits form one group each.)  No host round trip and no per-call
// allocation: the plan owns its workspace.  Because the kernels read the
// per-call buffers through the argument block, the same captured graph
// serves every call.
#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.hpp"

namespace polarhip {
namespace {

constexpr int kMaxCodes = 16;
constexpr int kMaxBranches = 4;
static_assert(kMaxCodes <= kSclQueues, "a group's codes are queues of one list-decoder launch");

struct MixedArgs {
    MixedIo io;                    // LLR rows, information bits and codes
    int64_t B;
    const int32_t* code_of_frame;  // [B]
    uint8_t* used_scl;             // [B] or null
    int64_t* stats;                // [8] or null
};

__global__ void set_args_kernel(MixedArgs* d, MixedArgs v) {
    if (lid_x() == 0) *d = v;
}

__global__ void clear_kernel(int32_t* c, int n) {
    if ((int)lid_x() < n) c[lid_x()] = 0;
}

// ids of group g (the group of the frame's code): lists[g * cap + ...], cnt[g] of them
__global__ __launch_bounds__(256) void bucket_kernel(const MixedArgs* __restrict__ a, int n_codes, int n_groups,
                                                     int64_t cap,
                                                     const int32_t* __restrict__ group_of_code,
                                                     int32_t* __restrict__ lists, int32_t* __restrict__ cnt) {
    const int64_t f = gid_x() * 256 + lid_x();
    int g = -1;
    if (f < a->B && f < cap) {
        const int c = a->code_of_frame[f];
        if (c >= 0 && c < n_codes) g = group_of_code[c];
    }
    // one atomic per wavefront and group
    const int lane = lid_x() & 63;
    for (int h = 0; h < n_groups; ++h) {
        const uint64_t m = __ballot(g == h);
        if (m == 0) continue;
        int base = 0;
        if (lane == 0) base = atomicAdd(&cnt[h], (int)__popcll(m));
        base = __shfl(base, 0, 64);
        if (g == h) lists[(int64_t)h * cap + base + __popcll(m & ((1ull << lane) - 1ull))] = (int32_t)f;
    }
}

// list-decoder flags and statistics (the decoders wrote the information bits);
// one set of atomics per workgroup
__global__ __launch_bounds__(256) void mixed_flags_kernel(const MixedArgs* __restrict__ a, int n_codes,
                                                          const uint8_t* __restrict__ ok,
                                                          const int32_t* __restrict__ iters,
                                                          const uint8_t* __restrict__ scl_ok) {
    __shared__ unsigned long long red[5][4];
    unsigned long long s[5] = {0, 0, 0, 0, 0};  // frames, BP ok, list-decoded, iterations, CRC failures
    const int64_t f = gid_x() * 256 + lid_x();
    if (f < a->B) {
        const int c = a->code_of_frame[f];
        if (c >= 0 && c < n_codes) {
            const bool good = ok[f] != 0;
            if (a->used_scl) a->used_scl[f] = good ? 0 : 1;
            s[0] = 1;
            s[1] = good;
            s[2] = !good;
            s[3] = (unsigned long long)iters[f];
            s[4] = !good && !scl_ok[f];
        }
    }
    if (!a->stats) return;
    for (int i = 0; i < 5; ++i) {
        for (int m = 32; m >= 1; m >>= 1) s[i] += __shfl_xor(s[i], m, 64);
        if ((lid_x() & 63) == 0) red[i][lid_x() >> 6] = s[i];
    }
    __syncthreads();
    if (lid_x() < 5) {
        const int i = lid_x();
        const unsigned long long v = red[i][0] + red[i][1] + red[i][2] + red[i][3];
        if (v) atomicAdd(reinterpret_cast<unsigned long long*>(a->stats) + i, v);
    }
}

}  // namespace
}  // namespace polarhip

using namespace polarhip;

struct polar_mixed {
    int device = 0;
    int n_codes = 0;
    int64_t cap = 0;  // max frames per call
    int L = 0;
    std::vector<const polar_code*> codes;
    // groups: codes of one block length (one code each below 32 bits)
    int n_groups = 0;
    std::vector<int> rep;           // per group: its first code
    std::vector<int> order;         // groups by block length, longest first
    std::vector<SclWork> work;      // per group: the failure queues of its codes
    std::vector<bp_params> params;  // per group (the first code's variant)
    std::vector<SclPlan> scl;       // per group
    std::vector<int> bp_grid;       // per group
    // device memory (one allocation)
    void* mem = nullptr;
    MixedArgs* dargs = nullptr;
    CodeDev* dcodes = nullptr;
    int32_t* gmap = nullptr;    // [n_codes] group of each code
    int32_t* counts = nullptr;  // [3 * n_codes]: bucket sizes by group, queue sizes by code, tickets by group
    int32_t* lists = nullptr;   // [n_groups][cap]
    int32_t* queues = nullptr;  // [n_codes][cap] failed frames of each code
    uint8_t* ok = nullptr;
    int32_t* iters = nullptr;
    uint8_t* scl_ok = nullptr;
    std::vector<void*> glob;  // per list-decoder launch: its global slice
    int nbr = 0;
    hipStream_t br[kMaxBranches] = {};  // branch 0 is the calling stream
    hipEvent_t ev_fork = nullptr;
    hipEvent_t ev_join[kMaxBranches] = {};
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

static void mixed_release(polar_mixed* m) {
    if (!m) return;
    if (m->exec) hipGraphExecDestroy(m->exec);
    if (m->graph) hipGraphDestroy(m->graph);
    for (int s = 0; s < m->nbr; ++s) {
        if (m->ev_join[s]) hipEventDestroy(m->ev_join[s]);
        if (m->br[s]) hipStreamDestroy(m->br[s]);
    }
    if (m->ev_fork) hipEventDestroy(m->ev_fork);
    if (m->cap_stream) hipStreamDestroy(m->cap_stream);
    if (m->mem) hipFree(m->mem);
    delete m;
}

extern "C" polar_status polar_mixed_create(const polar_code* const* codes, int32_t n_codes, int64_t max_frames,
                                           const bp_params* params, int32_t L, const int32_t* variants,
                                           polar_mixed** out) {
    if (!out || !codes || !params) return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: null argument");
    *out = nullptr;
    if (n_codes < 1 || n_codes > kMaxCodes)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: n_codes must be in [1, 16]");
    if (max_frames < 1 || max_frames > (int64_t)INT32_MAX)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: max_frames must be in [1, 2^31)");
    if (params->weights) return set_error(POLAR_ERR_UNSUPPORTED, "polar_mixed_create: weighted BP is per code");
    if (params->max_iter < 1 || params->stop < 0 || params->stop > 2 || !(params->llr_max > 0.0f) || params->rule != 0)
        return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: bad BP parameters");
    int dev = 0;
    polar_status st = hip_check(hipGetDevice(&dev), "get device");
    if (st != POLAR_OK) return st;
    polar_mixed* m = new polar_mixed();
    m->device = dev;
    m->n_codes = n_codes;
    m->cap = max_frames;
    m->L = L;
    for (int c = 0; c < n_codes; ++c) {
        const polar_code* code = codes[c];
        if (!code || code->device != dev) {
            mixed_release(m);
            return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: null code or code of another device");
        }
        if (params->stop == 2 && code->c == 0) {
            mixed_release(m);
            return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: CRC stop needs codes with a CRC");
        }
        const int v = variants ? variants[c] : 0;
        if (v != 0 && !bp_variant_supported(code->n, v)) {
            mixed_release(m);
            return set_error(POLAR_ERR_INVALID_ARG, "polar_mixed_create: unknown BP variant");
        }
        m->codes.push_back(code);
    }
    // groups: one per block length (one BP kernel and one list-decoder kernel
    // serve the group's codes); a code shorter than 32 bits forms its own
    std::vector<int32_t> gmap(n_codes);
    for (int c = 0; c < n_codes; ++c) {
        int g = -1;
        if (codes[c]->n >= 5)
            for (int h = 0; h < m->n_groups; ++h)
                if (codes[m->rep[h]]->N == codes[c]->N) g = h;
        if (g < 0) {
            g = m->n_groups++;
            m->rep.push_back(c);
        }
        gmap[c] = g;
    }
    for (int g = 0; g < m->n_groups; ++g) {
        const int c = m->rep[g];
        bp_params p = *params;
        p.variant = variants ? variants[c] : 0;
        int grid = 0;
        SclPlan sp;
        if ((st = bp_gather_grid(codes[c], &p, max_frames, &grid)) != POLAR_OK ||
            (st = scl_plan_dims(codes[c]->n, L, max_frames, &sp)) != POLAR_OK) {
            mixed_release(m);
            return st;
        }
        m->params.push_back(p);
        m->bp_grid.push_back(grid);
        m->scl.push_back(sp);
    }
    for (int g = 0; g < m->n_groups; ++g) m->order.push_back(g);
    std::stable_sort(m->order.begin(), m->order.end(),
                     [&](int x, int y) { return codes[m->rep[x]]->N > codes[m->rep[y]]->N; });
    // one device allocation, carved
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    const size_t o_args = take(sizeof(MixedArgs));
    const size_t o_codes = take(sizeof(CodeDev) * n_codes);
    const size_t o_gmap = take(sizeof(int32_t) * n_codes);
    const size_t o_cnt = take(sizeof(int32_t) * 3 * n_codes);
    const size_t o_lists = take(sizeof(int32_t) * m->n_groups * max_frames);
    const size_t o_queues = take(sizeof(int32_t) * n_codes * max_frames);
    const size_t o_ok = take(max_frames);
    const size_t o_it = take(sizeof(int32_t) * max_frames);
    const size_t o_sok = take(max_frames);
    std::vector<size_t> o_g(m->scl.size());
    for (size_t j = 0; j < m->scl.size(); ++j) o_g[j] = take(m->scl[j].glob_per_wg * m->scl[j].grid);
    if ((st = hip_check(hipMalloc(&m->mem, off), "polar_mixed_create: hipMalloc")) != POLAR_OK) {
        m->mem = nullptr;
        mixed_release(m);
        return set_error(POLAR_ERR_NO_MEMORY, "polar_mixed_create: device allocation failed");
    }
    char* b = static_cast<char*>(m->mem);
    m->dargs = reinterpret_cast<MixedArgs*>(b + o_args);
    m->dcodes = reinterpret_cast<CodeDev*>(b + o_codes);
    m->gmap = reinterpret_cast<int32_t*>(b + o_gmap);
    m->counts = reinterpret_cast<int32_t*>(b + o_cnt);
    m->lists = reinterpret_cast<int32_t*>(b + o_lists);
    m->queues = reinterpret_cast<int32_t*>(b + o_queues);
    m->ok = reinterpret_cast<uint8_t*>(b + o_ok);
    m->iters = reinterpret_cast<int32_t*>(b + o_it);
    m->scl_ok = reinterpret_cast<uint8_t*>(b + o_sok);
    for (int g = 0; g < m->n_groups; ++g) {
        SclWork w{};
        w.ids = m->queues;
        w.queue_stride = max_frames;
        w.count_dev = m->counts + n_codes;
        for (int c = 0; c < n_codes; ++c)
            if (gmap[c] == g) w.code_ids[w.n_queues++] = c;
        m->work.push_back(w);
    }
    for (size_t j = 0; j < m->scl.size(); ++j) m->glob.push_back(m->scl[j].glob_per_wg ? (void*)(b + o_g[j]) : nullptr);
    std::vector<CodeDev> hc(n_codes);
    for (int c = 0; c < n_codes; ++c) hc[c] = codes[c]->dev();
    st = hip_check(hipMemcpy(m->dcodes, hc.data(), sizeof(CodeDev) * n_codes, hipMemcpyHostToDevice), "copy codes");
    if (st == POLAR_OK)
        st = hip_check(hipMemcpy(m->gmap, gmap.data(), sizeof(int32_t) * n_codes, hipMemcpyHostToDevice), "copy map");
    m->nbr = m->n_groups < kMaxBranches ? m->n_groups : kMaxBranches;
    for (int s = 1; s < m->nbr && st == POLAR_OK; ++s) {
        st = hip_check(hipStreamCreateWithFlags(&m->br[s], hipStreamNonBlocking), "stream create");
        if (st == POLAR_OK) st = hip_check(hipEventCreateWithFlags(&m->ev_join[s], hipEventDisableTiming), "event");
    }
    if (st == POLAR_OK) st = hip_check(hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming), "event");
    if (st != POLAR_OK) {
        mixed_release(m);
        return st;
    }
    *out = m;
    return ok_status();
}

extern "C" void polar_mixed_free(polar_mixed* m) {
    if (!m) return;
    int cur = 0;
    hipGetDevice(&cur);
    hipSetDevice(m->device);
    hipDeviceSynchronize();
    mixed_release(m);
    hipSetDevice(cur);
}

// everything after the argument block, on `st` (with branches on the plan's streams)
static polar_status mixed_pipeline(polar_mixed* m, hipStream_t st) {
    polar_status r;
    const int nc = m->n_codes, ng = m->n_groups;
    hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(64), 0, st, m->counts, 3 * nc);
    const unsigned bgrid = (unsigned)((m->cap + 255) / 256);
    hipLaunchKernelGGL(bucket_kernel, dim3(bgrid), dim3(256), 0, st, m->dargs, nc, ng, m->cap, m->gmap, m->lists,
                       m->counts);
    if ((r = hip_check(hipGetLastError(), "bucket launch")) != POLAR_OK) return r;
    if ((r = hip_check(hipEventRecord(m->ev_fork, st), "event record")) != POLAR_OK) return r;
    for (int s = 1; s < m->nbr; ++s)
        if ((r = hip_check(hipStreamWaitEvent(m->br[s], m->ev_fork, 0), "stream wait")) != POLAR_OK) return r;
    // The longest chains first, so that they get the first places on the chip;
    // the first branch is the calling stream itself: with four more streams
    // beside it two of them share one of the process's four hardware queues, and
    // the longest chain waited behind another (direct launches, twelve codes:
    // 3.1 ms, 2.0 ms this way; 2.3 ms in a process whose other streams hold some
    // of the queues, where the graph takes 1.9 ms)
    for (int i = 0; i < ng; ++i) {
        const int g = m->order[i];
        hipStream_t bs = i % m->nbr == 0 ? st : m->br[i % m->nbr];
        const polar_code* code = m->codes[m->rep[g]];
        if ((r = launch_bp_gather(code, &m->dargs->io, m->lists + (int64_t)g * m->cap, m->counts + g,
                                  m->counts + 2 * nc + g, &m->params[g], m->iters, m->ok, m->queues, m->cap,
                                  m->counts + nc, m->bp_grid[g], bs)) != POLAR_OK)
            return r;
        SclOut out;
        out.crc_ok = m->scl_ok;
        if ((r = launch_scl(code, m->scl[g], nullptr, m->L, m->work[g], out, m->glob[g], bs, &m->dargs->io)) !=
            POLAR_OK)
            return r;
    }
    for (int s = 1; s < m->nbr; ++s) {
        if ((r = hip_check(hipEventRecord(m->ev_join[s], m->br[s]), "event record")) != POLAR_OK) return r;
        if ((r = hip_check(hipStreamWaitEvent(st, m->ev_join[s], 0), "stream wait")) != POLAR_OK) return r;
    }
    hipLaunchKernelGGL(mixed_flags_kernel, dim3(bgrid), dim3(256), 0, st, m->dargs, nc, m->ok, m->iters, m->scl_ok);
    return hip_check(hipGetLastError(), "mixed flags launch");
}

static polar_status mixed_set_args(polar_mixed* m, int64_t B, const float* llr, const int32_t* code_of_frame,
                                   const int64_t* llr_off, const int64_t* out_off, uint8_t* info_hat,
                                   uint8_t* used_scl, int64_t* stats, hipStream_t stream) {
    if (!m) return set_error(POLAR_ERR_INVALID_ARG, "mixed decode: null plan");
    if (B < 0 || B > m->cap) return set_error(POLAR_ERR_INVALID_ARG, "mixed decode: B outside [0, max_frames]");
    if (B > 0 && (!llr || !code_of_frame || !llr_off || !out_off || !info_hat))
        return set_error(POLAR_ERR_INVALID_ARG, "mixed decode: null buffer");
    int dev = 0;
    polar_status r = hip_check(hipGetDevice(&dev), "get device");
    if (r != POLAR_OK) return r;
    if (dev != m->device) return set_error(POLAR_ERR_INVALID_ARG, "mixed decode: plan belongs to another device");
    MixedArgs a;
    a.io.llr = llr;
    a.io.off = llr_off;
    a.io.code_of = code_of_frame;
    a.io.codes = m->dcodes;
    a.io.info = info_hat;
    a.io.out_off = out_off;
    a.B = B;
    a.code_of_frame = code_of_frame;
    a.used_scl = used_scl;
    a.stats = stats;
    hipLaunchKernelGGL(set_args_kernel, dim3(1), dim3(64), 0, stream, m->dargs, a);
    return hip_check(hipGetLastError(), "set args launch");
}

extern "C" polar_status polar_mixed_decode(polar_mixed* m, int64_t B, const float* llr, const int32_t* code_of_frame,
                                           const int64_t* llr_off, const int64_t* out_off, uint8_t* info_hat,
                                           uint8_t* used_scl, int64_t* stats, hipStream_t stream) {
    polar_status r = mixed_set_args(m, B, llr, code_of_frame, llr_off, out_off, info_hat, used_scl, stats, stream);
    if (r != POLAR_OK) return r;
    if (B == 0) return ok_status();
    r = mixed_pipeline(m, stream);
    return r == POLAR_OK ? ok_status() : r;
}

extern "C" polar_status polar_mixed_decode_graph(polar_mixed* m, int64_t B, const float* llr,
                                                 const int32_t* code_of_frame, const int64_t* llr_off,
                                                 const int64_t* out_off, uint8_t* info_hat, uint8_t* used_scl,
                                                 int64_t* stats, hipStream_t stream) {
    polar_status r = mixed_set_args(m, B, llr, code_of_frame, llr_off, out_off, info_hat, used_scl, stats, stream);
    if (r != POLAR_OK) return r;
    if (B == 0) return ok_status();
    if (!m->exec) {
        // capture once on a stream of the plan's own, made for it here (a plan
        // that launches directly does not need one more stream beside its
        // branches); the graph reads its inputs through the argument block, so
        // later calls reuse it
        if (!m->cap_stream &&
            (r = hip_check(hipStreamCreateWithFlags(&m->cap_stream, hipStreamNonBlocking), "stream create")) != POLAR_OK)
            return r;
        r = hip_check(hipStreamBeginCapture(m->cap_stream, hipStreamCaptureModeRelaxed), "begin capture");
        if (r != POLAR_OK) return r;
        polar_status rp = mixed_pipeline(m, m->cap_stream);
        hipGraph_t g = nullptr;
        r = hip_check(hipStreamEndCapture(m->cap_stream, &g), "end capture");
        if (rp != POLAR_OK) {
            if (g) hipGraphDestroy(g);
            return rp;
        }
        if (r != POLAR_OK) return r;
        hipGraphExec_t ex = nullptr;
        r = hip_check(hipGraphInstantiate(&ex, g, nullptr, nullptr, 0), "graph instantiate");
        if (r != POLAR_OK) {
            hipGraphDestroy(g);
            return r;
        }
        m->graph = g;
        m->exec = ex;
    }
    r = hip_check(hipGraphLaunch(m->exec, stream), "graph launch");
    return r == POLAR_OK ? ok_status() : r;
}
