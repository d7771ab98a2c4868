// internal.hpp -- definitions shared by the host side and the kernels of
// libpolarhip (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/polar.h"

namespace polarhip {

// Work-item and workgroup indices read from the registers the dispatch
// initialises.  HIP's index variables go through device-library functions
// built with packed FP32 on; the inliner keeps them out of code built with it
// off, so every read would be a call and the workgroup id a per-lane value.
// Workgroup sizes are constants and grid sizes kernel arguments: the dispatch
// packet holds them too, but it lies in host memory, and the more CUs read it
// the longer each waits (encoder, N = 1024: 64 frames 6.8 us either way, 1024
// frames 17.9 us with the packet read, 6.5 us with the argument).
__device__ __forceinline__ int lid_x() { return (int)__builtin_amdgcn_workitem_id_x(); }
__device__ __forceinline__ int64_t gid_x() { return (int64_t)__builtin_amdgcn_workgroup_id_x(); }
__device__ __forceinline__ int64_t gid_y() { return (int64_t)__builtin_amdgcn_workgroup_id_y(); }

// Device-side view of a code, passed to kernels by value.
struct CodeDev {
    const uint32_t* frozen_bits;  // [max(N/32,1)] bit i of word i/32 set = frozen
    const int16_t* info_pos;      // [k] non-frozen positions in ascending order
    const uint32_t* syn;          // [N] CRC syndrome contribution of u_i = 1
    const uint32_t* syn_nib;      // [N/4][16] syndrome of each nibble value
    const uint32_t* da_bits;      // [max(N/32,1)] decision-aided positions of the list decoder
    int32_t N, n, K, c, k;
};

}  // namespace polarhip

struct polar_code {
    int32_t N, n, K, c, k;
    uint32_t poly;
    int device;
    std::vector<uint8_t> frozen;    // host [N]
    std::vector<int16_t> info_pos;  // host [k]
    std::vector<uint8_t> da;        // host [N], decision-aided positions
    int32_t n_da;                   // how many
    // device allocations (owned)
    uint32_t* d_frozen_bits = nullptr;
    int16_t* d_info_pos = nullptr;
    uint32_t* d_syn = nullptr;
    uint32_t* d_syn_nib = nullptr;
    uint32_t* d_da_bits = nullptr;
    polarhip::CodeDev dev() const {
        polarhip::CodeDev d;
        d.frozen_bits = d_frozen_bits;
        d.info_pos = d_info_pos;
        d.syn = d_syn;
        d.syn_nib = d_syn_nib;
        d.da_bits = d_da_bits;
        d.N = N;
        d.n = n;
        d.K = K;
        d.c = c;
        d.k = k;
        return d;
    }
};

namespace polarhip {

// error reporting (thread local)
polar_status set_error(polar_status st, const std::string& msg);
polar_status ok_status();
polar_status hip_check(hipError_t e, const char* what);

// launch helpers implemented in the kernel translation units
// wgs_per_cu > 0: at most that many BP workgroups per CU at a time (a
// persistent grid), where such a kernel exists (min-sum, unweighted or
// per-stage weights); otherwise one workgroup per frame group
// info_out (or null): [B][K] information bits of the frames whose verdict is ok
// queue: where the ids of the other frames go
struct BpQueue {
    int32_t* ids = nullptr;       // or null: no queue
    int32_t* count = nullptr;     // its length, 0 before the launch
    uint8_t* used_scl = nullptr;  // [B] 1 for a queued frame, 0 for the others, or null
};
polar_status launch_bp(const polar_code* code, const float* llr, int64_t B, const bp_params* p,
                       uint8_t* u_hat, float* llr_u, int32_t* iters, uint8_t* ok,
                       hipStream_t stream, int wgs_per_cu = 0, uint8_t* info_out = nullptr,
                       BpQueue queue = BpQueue());
polar_status launch_bp_save(const polar_code* code, const float* llr, int64_t B, int T, float llr_max,
                            const float* W, int variant, uint8_t* u_hat, float* llr_u, uint8_t* ok, float* saved,
                            hipStream_t stream);
// Per-call inputs of a ragged batch, read by the kernels from device memory
// (so a captured graph stays valid across calls with other buffers)
struct MixedIo {
    const float* llr;     // LLR rows
    const int64_t* off;   // row of frame f starts at element off[f]
    // frame f is decoded with codes[code_of[f]]
    const int32_t* code_of;
    const CodeDev* codes;
    uint8_t* info;           // K information bits of frame f from element out_off[f] on
    const int64_t* out_off;
};

// persistent BP over a device list of frame ids with ragged row offsets: the
// information bits of the frames whose verdict is ok go to io->info; a failed
// frame of code c is appended to the queue at fail_ids + c * fail_stride, of
// length fail_count[c].  *ticket (0 before the launch) hands out the list.
polar_status bp_gather_grid(const polar_code* code, const bp_params* p, int64_t max_frames, int* grid);
polar_status launch_bp_gather(const polar_code* code, const MixedIo* io, const int32_t* ids, const int32_t* count,
                              int32_t* ticket, const bp_params* p, int32_t* iters, uint8_t* ok, int32_t* fail_ids,
                              int64_t fail_stride, int32_t* fail_count, int grid, hipStream_t stream);
bool bp_variant_supported(int n, int variant);
int bp_default_variant(int n);
int bp_list_variants(int n, int32_t* ids, int cap);

// Where a workgroup's state lies for a number of path slots
struct SclForm {
    int slots;       // L times the frames it may decode at once
    int surv_off;    // LDS byte offset of the survivor list
    int trace_glob;  // 1: the per-block trace lives in the global slice
    int tb_off;      // LDS byte offset of the trace when !trace_glob
};

struct SclPlan {
    SclForm form[2];     // for one frame, for several
    size_t lds_bytes;    // dynamic LDS per workgroup, either form
    size_t trace_off;    // byte offset of the trace inside the global slice
    size_t glob_per_wg;  // global slice bytes per workgroup (levels > 5, trace)
    int grid;            // workgroups launched
    int target;          // wavefronts to fill before one takes a second frame
    int lay_n;           // log2 of the largest block length the layout holds
    int rank;            // survivor selection the plan is laid out for
};
// at most max_fpw frames per workgroup at once (their state then takes no more
// room than that)
polar_status scl_plan(const polar_code* code, int L, int64_t max_frames, SclPlan* plan, int max_fpw = 64);
// a plan that holds any code with n <= max_n (n >= 5); aided: for frames with many
// decision-aided positions
polar_status scl_plan_dims(int max_n, int L, int64_t max_frames, SclPlan* plan, int max_fpw = 64, bool aided = false);

// bytes beside the per-batch state that hybrid_decode_batch_static asks for
size_t scl_static_share(int n, int L);

// The frames of one list-decoder launch: queue k holds the frame ids
// ids[code_ids[k] * queue_stride + i] of code code_ids[k], i < its length
// (count_dev[code_ids[k]], or count_host without count_dev).  One plain list
// is queue 0 with code id 0; without ids frame i is i.
constexpr int kSclQueues = 16;
struct SclWork {
    const int32_t* ids;
    const int32_t* count_dev;
    int64_t count_host;
    int64_t queue_stride;
    int32_t n_queues;
    int32_t code_ids[kSclQueues];
    static SclWork list(const int32_t* ids, const int32_t* count_dev, int64_t count_host) {
        SclWork w{};
        w.ids = ids;
        w.count_dev = count_dev;
        w.count_host = count_host;
        w.n_queues = 1;
        return w;
    }
};

// Where the results go; each may be null but crc_ok.  info: the K information
// bits of frame f at f * K.
struct SclOut {
    uint8_t* u_hat = nullptr;
    uint8_t* info = nullptr;
    uint8_t* crc_ok = nullptr;
    float* pm = nullptr;
};

// io (optional): a ragged batch -- LLR rows at io->off[f], information bits at
// io->info + io->out_off[f] (and no u_hat); queue k's frames are decoded with
// io->codes[code_ids[k]]
polar_status launch_scl(const polar_code* code, const SclPlan& plan, const float* llr, int L, const SclWork& work,
                        const SclOut& out, void* glob, hipStream_t stream, const MixedIo* io = nullptr);

int device_cu_count();

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace polarhip
