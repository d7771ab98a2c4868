// scl.hip -- CRC-aided successive-cancellation list decoder (Sec. II-A).
//
// One wavefront decodes up to 64 / L frames of one code at a time; workgroups
// stay resident and walk lists of frames whose lengths may live on the device
// (the hybrid decoder feeds it the queue of BP failures without a host round
// trip).  Frames of one code take the same branches -- which bits are frozen,
// how long the list is -- so path slot l of the wavefront's frame s is lane
// s L + l, and every instruction and lane exchange of the bit loop serves all
// of them.  Where there are fewer frames than wavefronts the chip runs at once,
// a wavefront takes fewer (down to one): a frame's latency is shortest when
// its block starts have the wavefront to themselves.
//
// The LLR tree of a path (level d holds 2^d values, level n is the channel) and
// its partial sums (level d holds 2^d bits) are split in two:
//   - levels below BL = min(n, 5) live in the registers of the owning lane;
//   - level BL lives in LDS and the levels above it in the workgroup's global
//     slice, but for the two below the channel, which are computed from the
//     channel again when they are needed (partial sums of levels 5 and 6 in LDS,
//     the others in the slice); they are shared lazily:
//     each slot keeps, per level, the slot whose array it reads.  A block start
//     rewrites levels ctz(i)..BL of every path into the path's own slot and
//     reads level ctz(i)+1 through the pointer, which no path writes there;
//     partial sums are handled the same way.  The pointers change at block
//     boundaries only: inside a block a path keeps the slot it held at the
//     block start, and takes that slot's pointers at the block's end.
// Bits are processed in blocks of 2^BL.  Inside a block, ctz(i) and the number
// of trailing ones of i are compile-time constants, so a block is unrolled
// into straight-line code: a bit recomputes levels ctz(i)..0 in registers
// (level BL is read from LDS at the block start and once in the middle),
// decides, and folds the decided bit into the partial sums held in registers.
// A branching path is copied by pulling from the parent's lane exactly the
// registers that later bits of the block still read.  The candidates of a
// branching bit are listed parent by parent (bit 0 first); the L smallest under
// the strict order (metric, parent list position, bit) survive -- the pruned
// pseudo sort of Sec. II-A with a strict tie rule -- and keep that candidate
// order, so a survivor's slot is the number of survivors listed before it
// (found with two wavefront ballots) and slot index and list position coincide.
// Each lane holds its path's two candidates.  Which survive follows from the
// L-th smallest metric of the frame, found by a sorting network on the metrics
// alone (or bit by bit, or by counting, see below); candidates that tie
// with it are taken in candidate order.  The CRC is tracked per path as a
// running syndrome (linear in the decided bits).  Each path carries its
// decided bits of the current block in a register word and the slot it held
// at the block start (both pulled from the parent on a branch); at every
// block end each path writes that pair to the trace, so the chosen path is
// recovered by one step per block (its slot at each block end), after which
// every lane writes its outputs from the block words.
//
// A frame's decode is a long chain of dependent steps, so throughput comes
// from many frames in flight: the kernel is held to 128 VGPRs (four waves per
// SIMD); the trace (5 bytes per block and path) moves to the workgroup's
// global slice when it does not fit the LDS budget.
#include <atomic>
#include <type_traits>

#include "internal.hpp"
#include "lane_ops.hpp"

namespace polarhip {
namespace scl {

// Min-sum f (the check-node rule with min-sum, Sec. II-A): sgn(a) sgn(b)
// min(|a|, |b|), as b clamped to [-|a|, |a|] with a's sign applied -- one med3
// and one bit operation; a zero result may carry the other sign, which no
// decision, penalty or metric depends on.
__device__ __forceinline__ float f_ms(float a, float b) {
    const float m = __builtin_amdgcn_fmed3f(b, -fabsf(a), fabsf(a));
    return __uint_as_float(__float_as_uint(m) ^ (__float_as_uint(a) & 0x80000000u));
}

// g(a, b) = b + (1 - 2u) a with the partial-sum bit u at bit position q of
// word w (q known at compile time where it is called): the bit becomes the
// sign of a 1.0 and one fused multiply-add does the rest (the product with
// +-1 is exact, so the sum rounds as b + a or b - a does)
__device__ __forceinline__ float g_bit(float a, float b, uint32_t w, int q) {
    const float sg = __uint_as_float(((w << (31 - q)) & 0x80000000u) | 0x3F800000u);
    return __fmaf_rn(a, sg, b);
}

__device__ __forceinline__ void wg_mem_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Pointers typed by address space: LDS (3) and global (1).  Generic pointers
// would compile to flat instructions, whose waits also wait for every
// outstanding global access, and an LDS access through them takes the slower
// flat path; so LDS and global data are never reached through one pointer.
template <typename T>
using lds_ptr = __attribute__((address_space(3))) T*;
template <typename T>
using glb_ptr = __attribute__((address_space(1))) T*;

// plain 4-lane vectors (the HIP vector classes do not bind to pointers of a
// named address space)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ lds_ptr<T> as_lds(void* p) {
    return (lds_ptr<T>)p;
}
template <typename T>
__device__ __forceinline__ glb_ptr<T> as_glb(const void* p) {
    return (glb_ptr<T>)const_cast<void*>(p);
}

// a value every lane holds alike, moved to scalar registers (so what is read
// through it becomes scalar or uniform-address work)
__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// the slot read at each shared level, one byte per level: only levels 5..12
// are shared through slots (levels below 5 live in registers, N <= 4096), so
// eight bytes, one 64-bit register pair, hold them all (a branch pulls one
// pair per vector from the parent)
struct PtrVec {
    uint64_t w;
};

__device__ __forceinline__ int get_byte(const PtrVec& v, int idx) {
    const int sh = idx > 5 ? 8 * (idx - 5) : 0;  // levels below 5 are never read here
    return (int)((v.w >> sh) & 0xFFull);
}

__device__ __forceinline__ void set_byte(PtrVec& v, int idx, int val) {
    const int sh = idx > 5 ? 8 * (idx - 5) : 0;
    v.w = (v.w & ~(0xFFull << sh)) | ((uint64_t)val << sh);
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
    return (uint64_t)__shfl((unsigned long long)v, src, 64);
}

// A slot's row of the workgroup's global slice, 2^row_log words: LLR level d
// >= 6 at word 2^d and, in the words the levels leave free, the partial-sum
// levels from 7 on.  Partial-sum level d >= 5 is 2^(d - 5) words: levels 5 and
// 6, read and written at half and a quarter of the block starts, live in LDS,
// levels 7 to 10 in words 0..59 of the row, level 11 (N = 4096) in the middle
// of the row.  With all of them in LDS (12 KB more at N = 1024 with 64 slots)
// nine instead of sixteen wavefronts fit a CU.
// Two forms, by the frames a wavefront takes:
//   - several (deep): levels 6 .. n - 3 are kept; n - 2 and n - 1 are computed
//     from the channel row, which all paths share, whenever a block start needs
//     them.  The slices of a full chip go through HBM, and the top levels are
//     40 % of that traffic, which bounds large batches at L = 32;
//   - one: every level is kept (at N = 4096 up to n - 2), which has the shorter
//     chain of operations.
// 8192 frames of N = 1024 at L = 32: 1342 us with all levels kept, 1225 us deep;
// one frame: 429 and 465 us.
constexpr int kPsLds = 7;     // first partial-sum level outside LDS
constexpr int kPsWords = 3;   // LDS words per slot, levels 5 and 6
__host__ __device__ __forceinline__ constexpr int row_log(int n, bool deep) {
    return deep ? (n == 12 ? 11 : n > 8 ? n - 2 : 6) : n;
}
// whether LLR level d > 5 of block length 2^n is kept
__device__ __forceinline__ constexpr bool kept(int n, int d, bool deep) {
    return deep ? d <= n - 3 : n < 12 || d <= n - 2;
}
// word offset inside a slot's LDS words (d < 7) or its row
__device__ __forceinline__ constexpr int ps_off(int d, int rlog) {
    return d < kPsLds ? (1 << (d - 5)) - 1 : d == 11 ? 1 << (rlog - 1) : (1 << (d - 5)) - (1 << (kPsLds - 5));
}

// Level 5 of a slot is 32 floats in LDS, without padding: the 16-byte group e
// is kept at e ^ swz(slot), so that the same group of 8 (32 banks) or 16 (64
// banks) neighbouring slots is spread over all banks
constexpr int kSlotFloats = 32;
__device__ __forceinline__ int swz(int slot) { return ((slot >> 1) ^ (slot << 2)) & 7; }

constexpr int ctz_c(int v) {
    int c = 0;
    while (((v >> c) & 1) == 0) ++c;
    return c;
}

// partial-sum block of 2^T bits finished by `bit`, from the T levels below it
template <int T>
__device__ __forceinline__ uint32_t combine(uint32_t bit, const uint32_t (&ps)[5]) {
    uint32_t cur = bit;
#pragma unroll
    for (int d = 0; d < T; ++d) {
        const uint32_t h = 1u << d;
        const uint32_t lowmask = (h >= 32u) ? 0xFFFFFFFFu : ((1u << h) - 1u);
        cur = ((ps[d] ^ cur) & lowmask) | (cur << h);
    }
    return cur;
}

// ------------------------------------------------------------ survivors
// A lane holds the two candidates of its path as metric bits (metrics are
// non-negative, so their bit patterns order them): kh, the hard decision of
// the path's LLR, which keeps the path metric, and kf >= kh, the other.

enum : int { kRankCount = 0, kRankNetwork = 1, kRankThreshold = 2 };

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}

// the value of lane ^ J, all in VALU: data-parallel-primitive moves inside a
// row of 16 lanes (J = 4: half-row mirror, then quad reversal; J = 8: row
// rotation by 8)
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (J == 1) {
        return dpp_mov<0xB1>(v);  // quad_perm [1,0,3,2]
    } else if constexpr (J == 2) {
        return dpp_mov<0x4E>(v);  // quad_perm [2,3,0,1]
    } else if constexpr (J == 4) {
        return dpp_mov<0x1B>(dpp_mov<0x141>(v));
    } else {
        static_assert(J == 8, "distance");
        return dpp_mov<0x128>(v);  // row_ror:8
    }
}

// the value of the mirrored lane of each group of 2^M lanes, M <= 4
template <int M>
__device__ __forceinline__ uint32_t lane_mirror(uint32_t v) {
    if constexpr (M == 1) return dpp_mov<0xB1>(v);        // quad_perm [1,0,3,2]
    else if constexpr (M == 2) return dpp_mov<0x1B>(v);   // quad_perm [3,2,1,0]
    else if constexpr (M == 3) return dpp_mov<0x141>(v);  // row_half_mirror
    else return dpp_mov<0x140>(v);                        // row_mirror
}

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
// the smaller of a and b where k = 0, the larger where k = ~0 (one median)
__device__ __forceinline__ uint32_t pick_minmax(uint32_t a, uint32_t b, uint32_t k) {
    return umax(umin(a, b), umin(umax(a, b), k));
}
// ~0 where bit b of the lane is set, else 0
__device__ __forceinline__ uint32_t lane_bit_mask(int lane, int b) {
    return (uint32_t)((int32_t)((uint32_t)lane << (31 - b)) >> 31);
}

// The L-th smallest of the 2 L metrics of each frame's L lanes (x0 <= x1 in
// every lane), in all of them: a bitonic network over the metrics alone.
// Element 2 l + r of a frame is register r of its lane l; runs are merged in
// ascending order, the first exchange of each merge being the mirror of the
// run (so no lane sorts the other way round), up to two sorted runs of L;
// the smaller ones of the pairs (i, 2 L - 1 - i) are then the L smallest, and
// their largest is the answer.  Every exchange is one lane move and one median
// per register: about 60 VALU instructions for L = 32 and 25 for L = 8,
// whatever the number of frames, where a 64-bit (metric, lane) network took
// 16 stages of seven for one frame.
template <int L>
__device__ __forceinline__ uint32_t lth_smallest(uint32_t x0, uint32_t x1, int lane) {
    constexpr int LOGL = ctz_c(L);
    static_for<1, (LOGL > 0 ? LOGL : 1)>([&](auto MC) {
        constexpr int m = decltype(MC)::value;  // merge into runs of 2^m lanes
        {
            const uint32_t k = lane_bit_mask(lane, m - 1);
            const uint32_t p0 = lane_mirror<m>(x0), p1 = lane_mirror<m>(x1);
            x0 = pick_minmax(x0, p1, k);
            x1 = pick_minmax(x1, p0, k);
        }
        static_for<0, m - 1>([&](auto JC) {
            constexpr int j = m - 2 - decltype(JC)::value;  // lane distance 2^j
            const uint32_t k = lane_bit_mask(lane, j);
            const uint32_t p0 = lane_xor<(1 << j)>(x0), p1 = lane_xor<(1 << j)>(x1);
            x0 = pick_minmax(x0, p0, k);
            x1 = pick_minmax(x1, p1, k);
        });
        const uint32_t lo = umin(x0, x1), hi = umax(x0, x1);
        x0 = lo;
        x1 = hi;
    });
    if constexpr (LOGL == 0) {
        return x0;
    } else {
        uint32_t p0, p1;
        if constexpr (LOGL == 5) {
            // the mirror of 32 lanes: the row mirror of the other row
            const auto r0 = __builtin_amdgcn_permlane16_swap(lane_mirror<4>(x0), lane_mirror<4>(x0), false, false);
            const auto r1 = __builtin_amdgcn_permlane16_swap(lane_mirror<4>(x1), lane_mirror<4>(x1), false, false);
            p0 = (lane & 16) ? r0[0] : r0[1];
            p1 = (lane & 16) ? r1[0] : r1[1];
        } else {
            p0 = lane_mirror<LOGL>(x0);
            p1 = lane_mirror<LOGL>(x1);
        }
        uint32_t v = umax(umin(x0, p1), umin(x1, p0));
        // a lane and its mirror hold the same pairs, so half the lanes do
        if constexpr (LOGL >= 5) v = umax(v, lane_mirror<4>(v));
        if constexpr (LOGL >= 4) v = umax(v, lane_mirror<3>(v));
        if constexpr (LOGL >= 3) v = umax(v, lane_xor<2>(v));
        if constexpr (LOGL >= 2) v = umax(v, lane_xor<1>(v));
        return v;
    }
}

// set bits of a wavefront mask, counted in two 32-bit halves (a uniform
// 32-bit count keeps the comparisons that use it in scalar instructions)
__device__ __forceinline__ uint32_t mask_count(uint64_t m) {
    return (uint32_t)__builtin_popcount((uint32_t)m) + (uint32_t)__builtin_popcount((uint32_t)(m >> 32));
}

// set bits of a wavefront mask below this lane
__device__ __forceinline__ int mask_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// the lanes of this lane's frame
template <int L>
__device__ __forceinline__ uint64_t frame_lanes(int lane) {
    return ((1ull << L) - 1ull) << (lane & ~(L - 1));
}

// Which of this lane's candidates are among the frame's L smallest under
// (metric, parent, bit), given the L-th smallest metric tau: all below it, and
// of those equal to it the first in candidate order, as many as are missing.
template <int L>
__device__ __forceinline__ void keep_ties(uint32_t kh, uint32_t kf, uint32_t tau, bool hard1, bool alive, int lane,
                                          bool& keep_h, bool& keep_f) {
    const uint64_t mine = frame_lanes<L>(lane);
    const bool lt_h = alive && kh < tau, lt_f = alive && kf < tau;
    const bool eq_h = alive && kh == tau, eq_f = alive && kf == tau;
    const uint64_t qh = __ballot(eq_h) & mine, qf = __ballot(eq_f) & mine;
    const int need = L - (int)(mask_count(__ballot(lt_h) & mine) + mask_count(__ballot(lt_f) & mine));
    const int before = mask_below(qh) + mask_below(qf);
    keep_h = lt_h || (eq_h && before + (hard1 && eq_f ? 1 : 0) < need);
    keep_f = lt_f || (eq_f && before + (!hard1 && eq_h ? 1 : 0) < need);
}

// Threshold selection of the same value for a single frame, its paths on the
// first L lanes: found bit by bit from the top as the largest value with fewer
// than L metrics below it.  A step waits for the one before, so the 2 L metrics
// are spread over as many lanes, which makes a step one comparison, and value and
// count stay in scalar registers (N = 1024, L = 32, one frame: 1478 us with two
// comparisons and counts per lane, 677 us so; with eight steps unrolled 770).
// The value lies in [tau, tau + 2^b) after the step of bit b; once exactly L
// metrics lie below that end, any value up to it tells the survivors, and the
// lower bits need not be found (677 -> 534 us; half decision-aided, where the
// metrics lie closer, 403 -> 389).  At L = 8 the test costs the kernel registers
// (3000 frames, two a wavefront, 869 us without it and 907 with).
template <int L>
__device__ __forceinline__ uint32_t lth_smallest_by_bits(uint32_t kh, uint32_t kf, bool alive, int lane) {
    static_assert(L == 8 || L == 32, "list size");
    uint32_t moved;  // kf of lane - L
    if constexpr (L == 32) moved = __builtin_amdgcn_permlane32_swap(kf, kf, false, false)[0];
    else moved = lane_xor<8>(kf);
    const uint32_t key = alive ? kh : lane < 2 * L ? moved : 0xFFFFFFFFu;
    auto count = [](uint64_t m) -> uint32_t {
        return L == 32 ? mask_count(m) : (uint32_t)__builtin_popcount((uint32_t)m);
    };
    uint32_t tau = 0u;
#pragma unroll
    for (int b = 30; b >= 0; --b) {
        const uint32_t trial = tau | (1u << b);
        const uint64_t m = __ballot(key < trial);
        tau = count(m) < (uint32_t)L ? trial : tau;
        if (L == 32 && b <= 23 && b % 3 == 2) {
            const uint32_t end = tau + (1u << b);
            if (count(__ballot(key < end)) == (uint32_t)L) return end - 1u;
        }
    }
    return tau;
}

// The pruned pseudo sort: each candidate counts the frame's candidates before
// it.  The metrics go through LDS once, candidate by candidate.  Two candidates
// a lane, for the frames whose candidates do not all find a lane.
template <int L>
__device__ __forceinline__ void keep_by_count(lds_ptr<u32x2> cand, uint32_t kh, uint32_t kf, bool hard1, bool alive,
                                              int lane, bool& keep_h, bool& keep_f) {
    const uint32_t k0 = hard1 ? kf : kh, k1 = hard1 ? kh : kf;
    if (alive) cand[lane] = u32x2{k0, k1};
    wave_lds_sync();
    const int first = lane & ~(L - 1), pl = lane & (L - 1);
    int r0 = 0, r1 = 0;
    if (alive) {
#pragma unroll 4
        for (int i = 0; i < L; ++i) {
            const u32x2 v = cand[first + i];
            r0 += (v.x < k0 || (v.x == k0 && i < pl)) ? 1 : 0;
            r0 += (v.y < k0 || (v.y == k0 && i < pl)) ? 1 : 0;
            r1 += (v.x < k1 || (v.x == k1 && i <= pl)) ? 1 : 0;
            r1 += (v.y < k1 || (v.y == k1 && i < pl)) ? 1 : 0;
        }
    }
    wave_lds_sync();
    const bool keep0 = alive && r0 < L, keep1 = alive && r1 < L;
    keep_h = hard1 ? keep1 : keep0;
    keep_f = hard1 ? keep0 : keep1;
}

// Counting and threshold selection with one candidate a lane: candidate c (bit c
// & 1 of the path of lane c >> 1) of the wavefront's frames, 2 L to a frame, on
// lane c, so at most 32 / L frames fit.  A lane decides whether its candidate
// survives, by counting the frame's candidates before it, read from LDS in
// vectors of four, or (several frames) against the L-th smallest metric, found bit
// by bit.  N = 1024, L = 8: 1559 frames, one a wavefront, 765 us by counting with
// two candidates a lane, 528 us so; 3000 frames, two a wavefront, 1922 us by
// threshold with two candidates a lane, 874 us so.
template <int L, int RANK>
__device__ __forceinline__ uint32_t select_one_a_lane(lds_ptr<u32x2> surv, float lam0, float& PM, int nf, bool alive,
                                                      int lane) {
    constexpr int NC = 2 * L;
    const bool hard1 = lam0 < 0.0f;
    const uint32_t kh = __float_as_uint(PM), kf = __float_as_uint(PM + fabsf(lam0));
    if (alive) surv[lane] = u32x2{hard1 ? kf : kh, hard1 ? kh : kf};
    wave_lds_sync();
    const lds_ptr<const uint32_t> key = (lds_ptr<const uint32_t>)surv;
    const bool mine = lane < nf * NC;
    const int first = mine ? lane & ~(NC - 1) : 0;  // the frame's first candidate
    const uint32_t own = mine ? key[lane] : 0xFFFFFFFFu;
    bool keep;
    if constexpr (RANK == kRankCount) {
        constexpr int G = NC / 4 > 4 ? 4 : NC / 4;  // vectors in flight
        int rank = 0;
        for (int c0 = first; c0 < first + NC; c0 += 4 * G) {
            u32x4 v[G];
#pragma unroll
            for (int g = 0; g < G; ++g) v[g] = ((lds_ptr<const u32x4>)(key + c0))[g];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    rank += (v[g][i] < own || (v[g][i] == own && c0 + 4 * g + i < lane)) ? 1 : 0;
        }
        keep = mine && rank < L;
    } else {
        static_assert(NC < 32, "a frame's lanes within half a wavefront");
        const bool upper = lane >= 32;
        auto count = [&](uint64_t m) -> int {  // of the frame's lanes
            return __builtin_popcount(((upper ? (uint32_t)(m >> 32) : (uint32_t)m) >> (first & 31)) & ((1u << NC) - 1u));
        };
        uint32_t tau = 0u;
        for (int b = 30; b >= 0; --b) {
            const uint32_t trial = tau | (1u << b);
            tau = count(__ballot(own < trial)) < L ? trial : tau;
        }
        const uint64_t eq = __ballot(own == tau);
        const int need = L - count(__ballot(own < tau));
        const int before = mask_below(eq) - __builtin_popcountll(eq & ((1ull << first) - 1ull));
        keep = own < tau || (own == tau && before < need);
    }
    wave_lds_sync();
    const uint64_t m = __ballot(keep);
    if (keep) surv[mask_below(m)] = u32x2{(uint32_t)lane, own};
    wave_lds_sync();
    u32x2 r{0u, 0u};
    if (alive) r = surv[lane];
    wave_lds_sync();
    PM = __uint_as_float(r.y);
    return r.x;
}

// The survivors of one branching bit of frames with full lists (nf frames).
// They keep the candidate order, so a survivor goes to the slot with as many
// survivors before it; frames before this one hold L each, so the count over
// the wavefront is the lane.  Returns, for this lane's new path, (parent lane
// << 1 | bit) and the metric; lanes without a path get some valid lane.
template <int L, int RANK>
__device__ __forceinline__ uint32_t select_survivors(lds_ptr<u32x2> surv, float lam0, float& PM, int nf, bool alive,
                                                     int lane) {
    // (a plan for these two holds at most frames_room frames a wavefront)
    if constexpr (RANK != kRankNetwork && L == 8) {
        if (RANK == kRankCount || nf > 1) return select_one_a_lane<L, RANK>(surv, lam0, PM, nf, alive, lane);
    } else if constexpr (RANK == kRankCount) {
        if (nf == 1) return select_one_a_lane<L, RANK>(surv, lam0, PM, nf, alive, lane);
    }
    const bool hard1 = lam0 < 0.0f;
    const uint32_t kh = __float_as_uint(PM), kf = __float_as_uint(PM + fabsf(lam0));
    if constexpr (L == 1) {
        // The hard decision, or bit 0 where the metrics tie (one frame of N = 1024,
        // half its positions decision-aided: 232 us through the selection below, 153
        // us so, with nothing pulled from other lanes).
        return ((uint32_t)lane << 1) | (hard1 && kf != kh ? 1u : 0u);
    }
    bool keep_h, keep_f;
    if constexpr (RANK == kRankCount) {
        keep_by_count<L>(surv, kh, kf, hard1, alive, lane, keep_h, keep_f);
    } else {
        uint32_t tau;
        if constexpr (RANK == kRankThreshold) tau = lth_smallest_by_bits<L>(kh, kf, alive, lane);
        else tau = lth_smallest<L>(kh, kf, lane);
        keep_h = alive && kh <= tau;
        keep_f = alive && kf <= tau;
        // every frame keeps at least L this way; more only where metrics tie
        if (mask_count(__ballot(keep_h)) + mask_count(__ballot(keep_f)) != (uint32_t)(L * nf))
            keep_ties<L>(kh, kf, tau, hard1, alive, lane, keep_h, keep_f);
    }
    const bool keep0 = hard1 ? keep_f : keep_h, keep1 = hard1 ? keep_h : keep_f;
    const int d0 = mask_below(__ballot(keep_h)) + mask_below(__ballot(keep_f));
    if (keep0) surv[d0 & 63] = u32x2{(uint32_t)lane << 1, hard1 ? kf : kh};
    if (keep1) surv[(d0 + (keep0 ? 1 : 0)) & 63] = u32x2{((uint32_t)lane << 1) | 1u, hard1 ? kh : kf};
    wave_lds_sync();
    u32x2 r{0u, 0u};
    if (alive) r = surv[lane];
    wave_lds_sync();
    PM = __uint_as_float(r.y);
    return r.x;
}

struct Layout {
    SclForm form[2];  // for one frame a wavefront, for several (the traceback's block words sit below the LDS trace)
    int fpw;     // most frames a wavefront decodes at once, a power of two
    int grid[1]; // workgroups launched
    int target;  // wavefronts to fill before one takes a second frame
    int nblk;        // blocks of the largest block length the layout holds (trace rows)
    int64_t gbytes;  // bytes of the global slice per workgroup
    int64_t toff;    // byte offset of the trace inside the slice
};

// Active path a of the wavefront's frames (lists of 2^lg paths, L slots a frame)
template <int L>
__device__ __forceinline__ int slot_of(int a, int lg) {
    return ((a >> lg) << ctz_c(L)) | (a & ((1 << lg) - 1));
}

// Levels top..5 of every path at a block start (top = the highest level whose
// index bit changed).  Level 5 of a path is 32 items, taken as eight groups of
// four; group g of active path a is one chain, run by lane 8 (a mod 8) + g as
// its chain a / 8.  A chain's items of level d are the items e + 32 k of its
// group e, and each depends only on the same chain's items of level d + 1, so a
// lane computes its chains from level top + 1 alone, in registers: the level
// top items are the leaves, taken in bit-reversed order so that each pair of
// consecutive results at one level combines at once into the level below
// (a stack of one pending value per level); every item is stored on the way
// for the later bits and blocks (level 5 in LDS, the levels above in the
// workgroup's global slice), and nothing stored here is read back here.
// The chains of a lane run as one stream of leaves, the loads of the next P
// leaves in flight (two where the stack is deep, N >= 2048, to stay within the
// register budget).  Every load is issued unconditionally (a load past the
// stream's end repeats the last leaf's), so the waits for one leaf's data
// leave the later leaves' loads outstanding.  Chains past the last path repeat
// the last path's, with the same values to the same places, so no store waits
// on a lane mask.  H = top - 5.
//
// Where level top + 1 comes from (SRC): the slots' rows of the slice, or, for
// the top levels, the frame's channel row: SRC = 0 itself (top = n - 1), 1 or 2
// with the one or two levels between computed again (top = n - 2, n - 3).
enum : int { kSrcSlice = 3 };

// 16 bytes of a channel row, which may start at any float (vector loads take
// 4-byte alignment)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

template <int SRC>
struct Leaf {
    static constexpr int kVecs = SRC == kSrcSlice ? 2 : 2 << SRC;
    f32x4 v[kVecs];                          // SRC < 3: channel items e + i 2^top, i ascending; else level top + 1
    uint32_t w;                              // partial-sum bits of level top
    uint32_t w1[SRC == 1 ? 2 : SRC == 2 ? 2 : 1];  // of level top + 1 (SRC 1, 2)
    uint32_t w2[SRC == 2 ? 4 : 1];           // of level top + 2 (SRC 2)
};

// f (psum = false) or g of two groups of four items
__device__ __forceinline__ f32x4 fg4(const f32x4& a, const f32x4& b, uint32_t w, bool psum) {
    f32x4 v;
    if (psum) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = g_bit(a[i], b[i], w, i);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = f_ms(a[i], b[i]);
    }
    return v;
}

// psum, psum1, psum2: whether levels top, top + 1, top + 2 are g of their
// source here (the block is in the right half of the level above).  myslots: the
// slots this lane's path reads -- byte 0 LLR level top + 1, bytes 1, 2, 3
// partial sums of levels top, top + 1, top + 2; a chain takes them from its
// path's lane when it is begun (all chains' at once would take eight registers
// here, of which there are none to spare).
template <int L, int H, int SRC>
__device__ __forceinline__ void block_levels(const int paths, const int lg, const int lane, const int rlog,
                                             const lds_ptr<float> slam, const glb_ptr<float> glam,
                                             const uint64_t chan, const lds_ptr<uint32_t> psw, const bool psum,
                                             const bool psum1, const bool psum2, const bool deep, const int myslots) {
    constexpr int TOP = H + 5;
    constexpr int M = 1 << H;                                  // leaves per chain
    constexpr int P = SRC == 2 ? 1 : (SRC == 1 || H > 4) ? 2 : 4;  // leaves in flight
    constexpr int LP = P == 4 ? 2 : P == 2 ? 1 : 0;            // log2 P
    constexpr int SZT = 1 << TOP;
    const int C = (paths + 7) >> 3;       // chains per lane
    const int S = C << H;                 // leaves per lane
    // the lane index made opaque here, so that the lane offsets below are
    // computed at each block start instead of being hoisted out of the frame
    // loop and held in registers throughout
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int e4 = (ln & 7) << 2;         // the group's first item
    const glb_ptr<const char> gsrc = (glb_ptr<const char>)(glam + (2 << TOP));
    auto leaf_k = [](int m) -> int { return H == 0 ? 0 : (int)(__builtin_bitreverse32((uint32_t)m) >> (32 - H)); };
    auto slot_c = [&](int c) -> int {
        const int a = (ln >> 3) + 8 * c;
        return slot_of<L>(a < paths ? a : paths - 1, lg);
    };
    // word k of partial-sum level D of a slot
    auto ps_word = [&](auto DC, int slot, int k) -> uint32_t {
        constexpr int d = decltype(DC)::value;
        if constexpr (d < kPsLds) return psw[slot * kPsWords + ps_off(d, 0) + k];
        else return ((glb_ptr<uint32_t>)glam)[(uint32_t)((slot << rlog) + ps_off(d, rlog) + k)];
    };
    auto slots_of_chain = [&](int c) -> uint32_t { return (uint32_t)__shfl(myslots, slot_c(c), 64); };
    // leaf st of the lane, whose chain's slots are sv
    auto load = [&](int st, uint32_t sv) {
        Leaf<SRC> o;
        const int k = leaf_k(st & (M - 1));
        const int it = e4 + 32 * k;
        if constexpr (SRC == kSrcSlice) {
            // level top + 1 of the chain's source slot, 32-bit byte offsets
            // from the uniform base
            const uint32_t off = (uint32_t)((int)((sv & 0xFFu) << rlog) + it) * 4u;
            o.v[0] = *(glb_ptr<const f32x4>)(gsrc + off);
            o.v[1] = *(glb_ptr<const f32x4>)(gsrc + off + 4u * SZT);
        } else {
            // the channel row of the chain's frame
            const glb_ptr<const float> q = (glb_ptr<const float>)shfl64(chan, slot_c(st >> H)) + it;
#pragma unroll
            for (int i = 0; i < Leaf<SRC>::kVecs; ++i) o.v[i] = *(glb_ptr<const f32x4_any>)(q + i * SZT);
        }
        // the partial sums (read also where they are not used: the slot
        // pointers of the first block are valid)
        o.w = ps_word(std::integral_constant<int, TOP>{}, (int)((sv >> 8) & 0xFFu), k) >> e4;
        if constexpr (SRC == 1 || SRC == 2) {
            const int s1 = (int)((sv >> 16) & 0xFFu);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                o.w1[i] = ps_word(std::integral_constant<int, TOP + 1>{}, s1, k + i * (SZT / 32)) >> e4;
        }
        if constexpr (SRC == 2) {
            const int s2 = (int)(sv >> 24);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o.w2[i] = ps_word(std::integral_constant<int, TOP + 2>{}, s2, k + i * (SZT / 32)) >> e4;
        }
        return o;
    };
    Leaf<SRC> ring[P];
    f32x4 stk[H > 0 ? H : 1];
    // leaf s0 + q, s0 a multiple of P: the chain and the low bits of the leaf's
    // index in it are known at compile time where the chain is at least P long
    // (sv_next: the slots of the chain of leaf s0 + P, where chains are at least P long)
    auto step = [&](const int s0, auto QC, Leaf<SRC>& slotq, const uint32_t sv_next) {
        constexpr int q = decltype(QC)::value;
        // the levels that are computed again, before the next load takes the
        // registers of their sources
        f32x4 a, b;
        if constexpr (SRC == kSrcSlice || SRC == 0) {
            a = slotq.v[0];
            b = slotq.v[1];
        } else if constexpr (SRC == 1) {
            a = fg4(slotq.v[0], slotq.v[2], slotq.w1[0], psum1);
            b = fg4(slotq.v[1], slotq.v[3], slotq.w1[1], psum1);
        } else {
            a = fg4(fg4(slotq.v[0], slotq.v[4], slotq.w2[0], psum2), fg4(slotq.v[2], slotq.v[6], slotq.w2[2], psum2),
                    slotq.w1[0], psum1);
            b = fg4(fg4(slotq.v[1], slotq.v[5], slotq.w2[1], psum2), fg4(slotq.v[3], slotq.v[7], slotq.w2[3], psum2),
                    slotq.w1[1], psum1);
        }
        const uint32_t wt = slotq.w;
        const int nx = s0 + q + P < S ? s0 + q + P : S - 1;
        slotq = load(nx, M >= P ? sv_next : slots_of_chain(nx >> H));
        const int m = M >= P ? ((s0 & (M - 1)) | q) : (q & (M - 1));
        const int c = M >= P ? (s0 >> H) : ((s0 >> H) + (q >> H));
        const int k = leaf_k(m);
        const int slot = slot_c(c);
        auto put = [&](auto DC, int kk, const f32x4& v) {
            constexpr int d = decltype(DC)::value;
            // with the channel as the source n = TOP + 1 + SRC
            if constexpr (d == 5) *(lds_ptr<f32x4>)(slam + slot * kSlotFloats + (e4 ^ (swz(slot) << 2))) = v;
            else if (SRC == kSrcSlice || kept(TOP + 1 + SRC, d, deep))
                *(glb_ptr<f32x4>)((glb_ptr<char>)glam + (uint32_t)((slot << rlog) + (1 << d) + e4 + 32 * kk) * 4u) = v;
        };
        f32x4 v = fg4(a, b, wt, psum);
        put(std::integral_constant<int, TOP>{}, k, v);
        bool go = true;
        static_for<0, H>([&](auto LC) {
            constexpr int l = decltype(LC)::value;
            // bit l of the leaf's index: compile-time below log2 P
            const bool one = (M >= P && l < LP) ? ((q >> l) & 1) != 0 : ((m >> l) & 1) != 0;
            if (go) {
                if (one) {
                    v = fg4(stk[l], v, 0u, false);
                    put(std::integral_constant<int, TOP - l - 1>{}, k & ((M >> (l + 1)) - 1), v);
                } else {
                    stk[l] = v;
                    go = false;
                }
            }
        });
    };
    {
        const uint32_t sv0 = slots_of_chain(0);
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int st = q < S ? q : S - 1;
            ring[q] = load(st, M >= P ? sv0 : slots_of_chain(st >> H));
        }
    }
    if (M >= P || S % P == 0) {
        for (int s0 = 0; s0 < S; s0 += P) {
            const uint32_t sv = M >= P ? slots_of_chain((s0 + P < S ? s0 + P : S - 1) >> H) : 0u;
            static_for<0, P>([&](auto QC) { step(s0, QC, ring[decltype(QC)::value], sv); });
        }
    } else {
        // a stream not a multiple of P (few paths, lowest levels)
        for (int s0 = 0; s0 < S; s0 += P)
            static_for<0, P>([&](auto QC) {
                if (s0 + decltype(QC)::value < S) step(s0, QC, ring[decltype(QC)::value], 0u);
            });
    }
}

// the decided-bit words of the trace, in LDS or in the global slice
struct TraceRows {
    lds_ptr<uint32_t> l;
    glb_ptr<uint32_t> g;
    bool glob;
    __device__ __forceinline__ uint32_t get(int i) const { return glob ? g[i] : l[i]; }
    __device__ __forceinline__ void set(int i, uint32_t v) const {
        if (glob) g[i] = v;
        else l[i] = v;
    }
};

template <int L, int BL, int RANK>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void scl_kernel(
    CodeDev code_in, const float* __restrict__ llr, SclWork work, SclOut out, unsigned char* __restrict__ glob_all,
    Layout lay, const MixedIo* __restrict__ mio) {
    constexpr int BS = 1 << BL;  // bits per block
    constexpr int LOGL = ctz_c(L);
    extern __shared__ __attribute__((aligned(16))) unsigned char sm[];
    const int lane = lid_x();
    const int sub = lane >> LOGL, pl = lane & (L - 1);  // the lane's frame and path

    auto queue_len = [&](int k) -> int64_t {
        return work.count_dev ? (int64_t)work.count_dev[work.code_ids[k]] : work.count_host;
    };
    // frames per wavefront: one as long as that fills `target` wavefronts
    int64_t all = 0;
    for (int k = 0; k < work.n_queues; ++k) all += queue_len(k);
    const int64_t want = (all + lay.target - 1) / lay.target;
    const int nf_max = uniform_int((int)(want < 1 ? 1 : want > lay.fpw ? lay.fpw : want));
    const bool deep = nf_max > 1;
    // One frame has a layout of its own, whose trace finds room in LDS where that of
    // several does not (hybrid of 4096 frames at 1.5 dB, N = 1024, L = 32, 2665
    // list-decoded one by one: 734 us in the layout of several, 715 us)
    const SclForm form = lay.form[deep ? 1 : 0];
    const int SLOTS = form.slots;

    const lds_ptr<float> slam = as_lds<float>(sm);                          // [slots][32]
    const lds_ptr<uint32_t> psw = (lds_ptr<uint32_t>)(slam + SLOTS * kSlotFloats);   // [slots][3]
    const lds_ptr<u32x2> surv = as_lds<u32x2>(sm + form.surv_off);               // [slots]
    const lds_ptr<uint32_t> words = as_lds<uint32_t>(sm);                   // [fpw][nblk], reuses the LLR area at the end

    unsigned char* gbase = glob_all ? glob_all + (size_t)gid_x() * (size_t)lay.gbytes : nullptr;
    const glb_ptr<float> glam = as_glb<float>(gbase);         // [slots][2^rlog]
    // the trace, per block and slot: the block's decided bits (bit r = bit r of
    // the block) and the slot the path held at the block start; in LDS or, when
    // tg, in the global slice
    const size_t tra_off = (size_t)lay.nblk * SLOTS * sizeof(uint32_t);
    const bool tg = form.trace_glob != 0;
    const TraceRows tru{as_lds<uint32_t>(sm + form.tb_off), as_glb<uint32_t>(gbase + lay.toff), tg};  // [nblk][slots]
    const lds_ptr<uint8_t> tra_l = as_lds<uint8_t>(sm + form.tb_off + tra_off);
    const glb_ptr<uint8_t> tra_g = as_glb<uint8_t>(gbase + lay.toff + tra_off);

    const float* const llr_base = mio ? mio->llr : llr;
    const int64_t* const row_off = mio ? mio->off : nullptr;
    // the grid size, read again where it is used (behind an index the compiler
    // cannot see through): held in a register over a frame's decode it costs spills
    auto grid = [&]() -> int64_t {
        int i = 0;
        asm volatile("" : "+s"(i));
        return lay.grid[i];
    };
    for (int64_t unit = gid_x();; unit += grid()) {
        // the unit's queue and its first entry there
        int64_t q0 = unit, len = 0;
        int k = 0;
        for (; k < work.n_queues; ++k) {
            len = queue_len(k);
            const int64_t units = (len + nf_max - 1) / nf_max;
            if (q0 < units) break;
            q0 -= units;
        }
        if (k == work.n_queues) break;
        q0 *= nf_max;
        const int code_id = uniform_int(work.code_ids[k]);
        const int nf = uniform_int((int)(len - q0 < nf_max ? len - q0 : nf_max));
        const int32_t* const ids = work.ids ? work.ids + code_id * work.queue_stride : nullptr;
        // the frame of a lane (lanes without one: the last frame's)
        auto frame_of = [&](int s) -> int64_t {
            const int64_t q = q0 + (s < nf ? s : nf - 1);
            return ids ? (int64_t)ids[q] : q;
        };
        CodeDev code = code_in;
        if (mio) {
            code = mio->codes[code_id];
            code.frozen_bits = uniform_ptr(code.frozen_bits);
            code.da_bits = uniform_ptr(code.da_bits);
            code.syn = uniform_ptr(code.syn);
            code.n = uniform_int(code.n);
            code.N = uniform_int(code.N);
        }
        const int n = code.n, N = code.N;
        const int rlog = row_log(n, deep);
        // the code's frozen and decision-aided words, lane w holding word w
        // (and word 64 + w): a block reads its word from the lanes
        const int nw = N >= 32 ? N >> 5 : 1;
        const glb_ptr<const uint32_t> fzb = as_glb<const uint32_t>(code.frozen_bits);
        const glb_ptr<const uint32_t> dab = as_glb<const uint32_t>(code.da_bits);
        const uint32_t fzv0 = lane < nw ? fzb[lane] : 0u, fzv1 = 64 + lane < nw ? fzb[64 + lane] : 0u;
        const uint32_t dav0 = lane < nw ? dab[lane] : 0u, dav1 = 64 + lane < nw ? dab[64 + lane] : 0u;
        const glb_ptr<const uint32_t> synp = as_glb<const uint32_t>(code.syn);
        // LLR row of a lane's frame: at row_off[f] (ragged batch) or f * N
        auto chan_of = [&]() -> const float* {
            const int64_t f = frame_of(sub);
            return llr_base + (row_off ? row_off[f] : f * N);
        };

        int act = 1, lgact = 0;  // paths per list, 2^lgact
        float PM = 0.0f;
        uint32_t SYN = 0u;
        // slot read at each LLR level >= BL and partial-sum level >= 5 (their
        // start values are only read by lanes without a path)
        PtrVec ptrL{0ull};
        PtrVec ptrP{0ull};
        float lv[32];             // levels 0..BL-1, heap order: level d at [2^d, 2^(d+1))
        uint32_t ps[5];           // partial-sum levels 0..BL-1: bit e of word d
        uint32_t ublk = 0u;  // this path's decided bits of the current block
        int anc = 0;         // the slot this path held at the block start

        for (int j = 0; j < (N >> BL); ++j) {
            const int i0 = j << BL;
            const uint32_t bmask = BS == 32 ? 0xFFFFFFFFu : ((1u << BS) - 1u);
            const int wi = i0 >> 5;
            const uint32_t fword = (uint32_t)__builtin_amdgcn_readlane((int)(wi < 64 ? fzv0 : fzv1), wi & 63);
            const uint32_t dword = (uint32_t)__builtin_amdgcn_readlane((int)(wi < 64 ? dav0 : dav1), wi & 63);
            const uint32_t fw = (fword >> (i0 & 31)) & bmask;
            const uint32_t dw = (dword >> (i0 & 31)) & bmask;  // decision-aided
            // the block's CRC syndromes, lane r holding position i0 + r (loaded
            // after the block start's fence, which would otherwise wait for it)
            uint32_t synv = 0u;
            bool syn_loaded = false;
            // ---------------- block start: levels top..BL of every path
            if constexpr (BL == 5) {
                if (BL < n) {
                    const int top = (j == 0) ? n - 1 : __builtin_ctz((unsigned)i0);
                    const int paths = nf << lgact;
                    // levels between top + 1 and the channel, as far as they
                    // are computed again (3: level top + 1 is kept)
                    const int depth = top + 1 == n ? 0 : kept(n, top + 1, deep) ? 3 : n - 1 - top;
                    const int my = get_byte(ptrL, top + 1) | (get_byte(ptrP, top) << 8) |
                                   (get_byte(ptrP, top + 1) << 16) | (get_byte(ptrP, top + 2 < 12 ? top + 2 : 12) << 24);
                    // the block's index bit of level top is set (but at the
                    // frame's start), those above tell the levels above
                    const bool psum = j != 0;
                    const bool psum1 = ((i0 >> (top + 1)) & 1) != 0, psum2 = ((i0 >> (top + 2)) & 1) != 0;
                    const uint64_t chan = depth <= 2 ? reinterpret_cast<uint64_t>(chan_of()) : 0ull;
                    // the levels above were written by other lanes at earlier
                    // block starts
                    wg_mem_order();
                    synv = synp[i0 + (lane & (BS - 1))];
                    syn_loaded = true;
#define POLAR_BLOCK_LEVELS(HH, SS) \
    block_levels<L, HH, SS>(paths, lgact, lane, rlog, slam, glam, chan, psw, psum, psum1, psum2, deep, my)
                    if (depth == 0) {
                        switch (top - BL) {
                            case 0: POLAR_BLOCK_LEVELS(0, 0); break;
                            case 1: POLAR_BLOCK_LEVELS(1, 0); break;
                            case 2: POLAR_BLOCK_LEVELS(2, 0); break;
                            case 3: POLAR_BLOCK_LEVELS(3, 0); break;
                            case 4: POLAR_BLOCK_LEVELS(4, 0); break;
                            case 5: POLAR_BLOCK_LEVELS(5, 0); break;
                            default: POLAR_BLOCK_LEVELS(6, 0); break;
                        }
                    } else if (depth == 1) {
                        switch (top - BL) {
                            case 0: POLAR_BLOCK_LEVELS(0, 1); break;
                            case 1: POLAR_BLOCK_LEVELS(1, 1); break;
                            case 2: POLAR_BLOCK_LEVELS(2, 1); break;
                            case 3: POLAR_BLOCK_LEVELS(3, 1); break;
                            case 4: POLAR_BLOCK_LEVELS(4, 1); break;
                            default: POLAR_BLOCK_LEVELS(5, 1); break;
                        }
                    } else if (depth == 2) {
                        switch (top - BL) {
                            case 0: POLAR_BLOCK_LEVELS(0, 2); break;
                            case 1: POLAR_BLOCK_LEVELS(1, 2); break;
                            case 2: POLAR_BLOCK_LEVELS(2, 2); break;
                            case 3: POLAR_BLOCK_LEVELS(3, 2); break;
                            default: POLAR_BLOCK_LEVELS(4, 2); break;
                        }
                    } else {
                        switch (top - BL) {
                            case 0: POLAR_BLOCK_LEVELS(0, kSrcSlice); break;
                            case 1: POLAR_BLOCK_LEVELS(1, kSrcSlice); break;
                            case 2: POLAR_BLOCK_LEVELS(2, kSrcSlice); break;
                            case 3: POLAR_BLOCK_LEVELS(3, kSrcSlice); break;
                            default: POLAR_BLOCK_LEVELS(4, kSrcSlice); break;
                        }
                    }
#undef POLAR_BLOCK_LEVELS
                    // level 5 (LDS) is read by the block's bits
                    wave_lds_sync();
                    for (int d = top; d >= BL; --d) set_byte(ptrL, d, lane & (SLOTS - 1));
                }
            }
            if (!syn_loaded) synv = synp[i0 + (lane & (BS - 1))];
            // the block's register levels and partial sums are all rewritten
            // before they are read again (lanes that join the list during the
            // block pull what they read): they carry nothing from the last block,
            // and the block start above had their registers
#pragma unroll
            for (int e = 0; e < 32; ++e) lv[e] = 0.0f;
#pragma unroll
            for (int d = 0; d < 5; ++d) ps[d] = 0u;
            ublk = 0u;
            anc = lane & (SLOTS - 1);
            // ---------------- the 2^BL bits of the block, unrolled.  Lanes
            // without a path compute along on whatever they hold; nothing of
            // theirs is stored or kept
            static_for<0, BS>([&](auto RC) {
                constexpr int r = decltype(RC)::value;
                // lowest level whose index bit changed at this bit (BL: block start)
                constexpr int top = (r == 0) ? BL : ctz_c(r);
                // register level d (1 <= d < BL) is read next by the bit
                // r' = r - (r mod 2^d) + 2^(d-1) and rewritten by bit
                // r - (r mod 2^d) + 2^d: after bit r it is still to be read
                // exactly when bit d - 1 of r is clear
                constexpr unsigned live_levels = (r + 1 < BS) ? (~(unsigned)r & ((1u << (BL - 1)) - 1u)) : 0u;
                // trailing ones of the bit index (>= BL at the block's last bit)
                constexpr int tb = (r + 1 < BS) ? ctz_c(~r) : BL;

                // ---- LLR levels min(top, BL-1)..0 of this lane's path
                {
                    float src[32];
                    constexpr int sl_lv = (r == 0) ? BL : top + 1;  // level read
                    if constexpr (sl_lv == BL) {
                        if (BL == n) {
                            const glb_ptr<const float> chan = as_glb<const float>(chan_of());
#pragma unroll
                            for (int e = 0; e < BS; ++e) src[e] = chan[e];
                        } else {
                            // written by this path's lane of the block start
                            const lds_ptr<float> p = slam + anc * kSlotFloats;
                            const int sw = swz(anc);
#pragma unroll
                            for (int e4 = 0; e4 < BS / 4; ++e4) {
                                const f32x4 t4 = ((lds_ptr<const f32x4>)p)[e4 ^ sw];
                                src[4 * e4] = t4.x;
                                src[4 * e4 + 1] = t4.y;
                                src[4 * e4 + 2] = t4.z;
                                src[4 * e4 + 3] = t4.w;
                            }
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < (1 << sl_lv); ++e) src[e] = lv[(1 << sl_lv) + e];
                    }
                    constexpr int dhi = sl_lv - 1;  // first level computed here
#pragma unroll
                    for (int d = dhi; d >= 0; --d) {
#pragma unroll
                        for (int e = 0; e < (1 << d); ++e) {
                            const float a = (d == dhi) ? src[e] : lv[(2 << d) + e];
                            const float b = (d == dhi) ? src[e + (1 << d)] : lv[(2 << d) + e + (1 << d)];
                            if (r != 0 && d == top)
                                lv[(1 << d) + e] = g_bit(a, b, ps[d], e);
                            else
                                lv[(1 << d) + e] = f_ms(a, b);
                        }
                    }
                }
                const float lam0 = lv[1];
                // ---- decision
                uint32_t bit = 0;
                if ((fw >> r) & 1u) {
                    PM = PM + (lam0 < 0.0f ? fabsf(lam0) : 0.0f);
                } else if ((dw >> r) & 1u) {
                    // decision-aided position (Sec. II-A): every path keeps its
                    // hard decision; no branching, no metric change, same slots
                    bit = lam0 < 0.0f ? 1u : 0u;
                    SYN ^= bit ? (uint32_t)__builtin_amdgcn_readlane((int)synv, r) : 0u;
                    ublk |= bit << r;
                } else {
                    uint32_t src;  // parent lane << 1 | bit
                    if (act == L) {
                        src = select_survivors<L, RANK>(surv, lam0, PM, nf, sub < nf, lane);
                    } else {
                        // the list is not full: every candidate survives in place
                        const int p = (lane & ~(L - 1)) | (pl >> 1);
                        const uint32_t b = (uint32_t)pl & 1u;
                        const float lp = __shfl(lam0, p, 64);
                        const float pmp = __shfl(PM, p, 64);
                        PM = pmp + ((b != (lp < 0.0f ? 1u : 0u)) ? fabsf(lp) : 0.0f);
                        src = ((uint32_t)p << 1) | b;
                        act *= 2;
                        lgact += 1;
                    }
                    const int par = (int)(src >> 1);
                    bit = src & 1u;
                    const uint32_t syn_i = (uint32_t)__builtin_amdgcn_readlane((int)synv, r);
                    // pull the parent's state: syndrome and live registers
                    // (lanes without a path pull some lane's state, which no one reads)
                    // a list of one stays on its lane: nothing to pull
                    auto pull = [&](auto v) {
                        if constexpr (L == 1) return v;
                        else return __shfl(v, par, 64);
                    };
                    SYN = pull(SYN) ^ (bit ? syn_i : 0u);
                    // partial-sum level d is written at the bits r with r mod
                    // 2^(d+1) = 2^d - 1 and read at those with r mod 2^(d+1) in
                    // [2^d, 2^(d+1) - 1] (g at level d, then the fold at the
                    // end of the 2^(d+1) block): after this point it is still to
                    // be read exactly when bit d of r is set
                    static_for<0, BL>([&](auto DC) {
                        constexpr int d = decltype(DC)::value;
                        if constexpr ((r >> d) & 1) ps[d] = pull(ps[d]);
                    });
                    static_for<1, BL>([&](auto DC) {
                        constexpr int d = decltype(DC)::value;
                        if constexpr ((live_levels >> (d - 1)) & 1u) {
#pragma unroll
                            for (int e = 1 << d; e < (2 << d); ++e) lv[e] = pull(lv[e]);
                        }
                    });
                    anc = pull(anc);
                    ublk = (r > 0 ? pull(ublk) : 0u) | (bit << r);
                }
                // ---- partial sums: the finished block of 2^t bits becomes level t
                if constexpr (tb < BL) ps[tb] = combine<tb>(bit, ps);
                else ps[0] = combine<BL>(bit, ps);
            });
            // ---------------- block end: the pointers of the path's slot at
            // the block start, the finished partial sums, the trace entry
            const bool alive = sub < nf && pl < act;
            if (BL == 5 && BL < n) {
                ptrL.w = shfl64(ptrL.w, anc);
                ptrP.w = shfl64(ptrP.w, anc);
                const int t = BL + __builtin_ctz(~(unsigned)j);
                if (t < n) {
                    // X_0 = this 32-bit block, X_{b+1} = [level 5 + b xor X_b, X_b];
                    // level t is X_{t-5}.  Word p of it is found from the top:
                    // in the first half of X_{b+1} it takes word p of level 5 + b
                    if (t == 5) {
                        if (alive) psw[lane * kPsWords] = ps[0];
                    } else {
                        const int W = 1 << (t - 5);
                        const int items = (nf << lgact) * W;
                        if (t > kPsLds) wg_mem_order();
                        for (int it0 = 0; it0 < items; it0 += 64) {
                            const int it = it0 + lane;
                            const int slot = slot_of<L>(it < items ? it >> (t - 5) : 0, lgact);
                            const int word = it & (W - 1);
                            PtrVec pp{shfl64(ptrP.w, slot)};
                            uint32_t v = __shfl(ps[0], slot, 64);
                            int w = word;
                            for (int d = t - 1; d >= 5; --d) {
                                const int half = 1 << (d - 5);
                                const int pss = get_byte(pp, d);
                                if (w < half) {
                                    if (d < kPsLds) v ^= psw[pss * kPsWords + ps_off(d, 0) + w];
                                    else v ^= ((glb_ptr<uint32_t>)glam)[(uint32_t)((pss << rlog) + ps_off(d, rlog) + w)];
                                } else {
                                    w -= half;
                                }
                            }
                            // a path's level t may be read by no one any more, so
                            // its own slot's words are free
                            if (it < items) {
                                if (t < kPsLds) psw[slot * kPsWords + ps_off(t, 0) + word] = v;
                                else ((glb_ptr<uint32_t>)glam)[(uint32_t)((slot << rlog) + ps_off(t, rlog) + word)] = v;
                            }
                        }
                    }
                    set_byte(ptrP, t, lane & (SLOTS - 1));
                    wave_lds_sync();
                }
            }
            if (alive) {
                tru.set(j * SLOTS + lane, ublk);
                if (tg) tra_g[j * SLOTS + lane] = (uint8_t)anc;
                else tra_l[j * SLOTS + lane] = (uint8_t)anc;
            }
        }
        // ---------------- selection per frame: smallest (CRC fails, metric, position)
        uint64_t key = ~0ull;
        if (sub < nf && pl < act)
            key = ((uint64_t)(SYN != 0u) << 40) | ((uint64_t)__float_as_uint(PM) << 8) | (uint64_t)lane;
        for (int m = L / 2; m >= 1; m >>= 1) {
            const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)key, m, 64);
            key = o < key ? o : key;
        }
        const int best = (int)(key & 63);
        const bool best_ok = ((key >> 40) & 1ull) == 0;
        const float best_pm = __shfl(PM, best, 64);
        // ---------------- trace the chosen paths back, one block at a time: the
        // slot held at each block's end and that block's decided bits (frozen
        // bits are 0 there)
        if (tg) wg_mem_order();
        else wave_lds_sync();
        const int nblk = N >> BL;
        if (pl == 0 && sub < nf) {
            int s = best;
            for (int jj = nblk - 1; jj >= 0; --jj) {
                words[sub * nblk + jj] = tru.get(jj * SLOTS + s);
                s = tg ? tra_g[jj * SLOTS + s] : tra_l[jj * SLOTS + s];
            }
            const int64_t f = frame_of(sub);
            out.crc_ok[f] = best_ok ? 1 : 0;
            if (out.pm) out.pm[f] = best_pm;
        }
        wave_lds_sync();
        for (int s = 0; s < nf; ++s) {
            const int64_t f = frame_of(s);
            // information bits of a hybrid's frame, each from its block's word
            if (uint8_t* const row = mio ? mio->info + mio->out_off[f] : out.info ? out.info + f * code.K : nullptr)
                for (int q = lane; q < code.K; q += 64) {
                    const int pos = code.info_pos[q];
                    row[q] = (uint8_t)((words[s * nblk + (pos >> BL)] >> (pos & (BS - 1))) & 1u);
                }
            if (!out.u_hat) continue;
            uint8_t* const urow = out.u_hat + f * (int64_t)N;
            const glb_ptr<uint8_t> urow_p = as_glb<uint8_t>(urow);
            const bool aligned4 = (reinterpret_cast<uintptr_t>(urow) & 3u) == 0;
            for (int it = 4 * lane; it < N; it += 256) {
                const uint32_t w = words[s * nblk + (it >> BL)] >> (it & (BS - 1));
                if (aligned4) {
                    *(glb_ptr<uint32_t>)(urow_p + it) =
                        (w & 1u) | ((w & 2u) << 7) | ((w & 4u) << 14) | ((w & 8u) << 21);
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b) urow_p[it + b] = (uint8_t)((w >> b) & 1u);
                }
            }
        }
        wave_lds_sync();
    }
}

using KernelFn = void (*)(CodeDev, const float*, SclWork, SclOut, unsigned char*, Layout, const MixedIo*);

template <int L, int RANK>
KernelFn pick_bl(int bl) {
    switch (bl) {
        case 3: return &scl_kernel<L, 3, kRankNetwork>;
        case 4: return &scl_kernel<L, 4, kRankNetwork>;
        case 5: return &scl_kernel<L, 5, RANK>;
        default: return nullptr;
    }
}

// the counting and threshold forms are instantiated for the list sizes the
// comparisons use, with BL = 5; the network serves every list
KernelFn pick(int L, int n, int rank) {
    const int bl = n < 5 ? n : 5;
    if (rank == kRankCount && L == 8) return pick_bl<8, kRankCount>(bl);
    if (rank == kRankCount && L == 32) return pick_bl<32, kRankCount>(bl);
    if (rank == kRankThreshold && L == 8) return pick_bl<8, kRankThreshold>(bl);
    if (rank == kRankThreshold && L == 32) return pick_bl<32, kRankThreshold>(bl);
    switch (L) {
        case 1: return pick_bl<1, kRankNetwork>(bl);
        case 2: return pick_bl<2, kRankNetwork>(bl);
        case 4: return pick_bl<4, kRankNetwork>(bl);
        case 8: return pick_bl<8, kRankNetwork>(bl);
        case 16: return pick_bl<16, kRankNetwork>(bl);
        case 32: return pick_bl<32, kRankNetwork>(bl);
        default: return nullptr;
    }
}

// bytes of the trace: per block of 2^BL bits and path, the block's decided
// bits (32-bit word) and the slot the path held at the block start (byte)
size_t trace_bytes(int slots, int n) {
    const int bl = n < 5 ? n : 5;
    return ((size_t)1 << (n - bl)) * slots * 5;
}

struct LdsPlan {
    size_t bytes;
    int soff;    // survivor list
    int tboff;   // LDS trace (tg == 0)
};

LdsPlan lds_plan(int L, int slots, int n, bool tg) {
    LdsPlan p{};
    const int bl = n < 5 ? n : 5;
    size_t b = (size_t)slots * (kSlotFloats + kPsWords) * 4;  // level 5, partial sums of levels 5 and 6
    b = align_up(b, 16);
    p.soff = (int)b;
    b += (size_t)slots * 8;
    // the traceback's block words reuse the space from 0
    const size_t words_end = (size_t)(slots / L) * ((size_t)1 << (n - bl)) * 4;
    b = align_up(b > words_end ? b : words_end, 16);
    p.tboff = 0;
    if (!tg) {
        p.tboff = (int)b;
        b += trace_bytes(slots, n);
    }
    p.bytes = align_up(b, 16);
    return p;
}

}  // namespace scl

// candidate ranking: 0 automatic (the network, which measured fastest on
// MI355X at every list size), 1 pruned pseudo sort (counting), 2 network, 3
// threshold selection
static std::atomic<int> g_scl_rank_mode{0};

static int rank_kind() {
    switch (g_scl_rank_mode.load(std::memory_order_relaxed)) {
        case 1: return scl::kRankCount;
        case 3: return scl::kRankThreshold;
        default: return scl::kRankNetwork;
    }
}

// LDS per workgroup; 0 (automatic) divides a CU's 160 KB among as many
// one-wave workgroups as the kernel's registers allow on a CU
static std::atomic<int64_t> g_scl_lds_budget{0};
constexpr size_t kLdsPerCu = 160 * 1024;

static size_t scl_budget(scl::KernelFn fn) {
    size_t budget = (size_t)g_scl_lds_budget.load(std::memory_order_relaxed);
    if (budget == 0) {
        int by_regs = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&by_regs, fn, 64, 0) != hipSuccess || by_regs < 1) by_regs = 1;
        budget = (kLdsPerCu / (size_t)by_regs) & ~(size_t)255;
        if (budget < 4096) budget = 4096;
    }
    return budget;
}

// whether a list decode uses counting or threshold selection (elsewhere those
// modes fall back to the network)
static bool other_ranking(int n, int L, int rank) {
    return rank != scl::kRankNetwork && n >= 5 && (L == 8 || L == 32);
}

// Frames a wavefront may take at once: as many as its lanes hold lists; half as
// many where a selection other than the network wants a lane for each candidate
// (L = 8: 16384 frames of N = 1024 by counting 957 us with four, 1086 with eight,
// by threshold 1522 and 2133 us; threshold with L = 32: 8192 frames 2620
// with one, 3091 us with two).  Counting with L = 32 takes two once the chip is
// full (8192 frames 3747 us with one, 2878 with two).
static int frames_room(int n, int L, int rank) {
    const bool half = other_ranking(n, L, rank) && (L == 8 || rank == scl::kRankThreshold);
    return half ? 32 / L : 64 / L;
}

// Wavefronts to fill before one takes a second frame, per CU.  As long as a
// frame's latency decides, one frame each is faster (2048 frames of N = 1024, L =
// 32: 610 us, 714 us with two on half the wavefronts); beyond, issue slots and
// memory do (4096 frames of L = 8: 497 us with two each, 665 us with one).
// The line, one frame each against two (us, 256 CUs):
//   - L <= 16: eight (L = 8, N = 1024, 2049 frames: 505 and 437; L = 16: 565 and
//     519, with half the positions decision-aided 395 and 397);
//   - L = 32, where two lists fill the wavefront and share less: ten at N = 512 and
//     1024 (N = 1024, 2304 frames: 698 and 732; 3000: 767 and 745), twelve with
//     two fifths or more of the positions decision-aided, which leaves less work
//     that two frames share (2304: 515 and 576; 3000: 574 and 594; 3300: 646 and
//     609; N = 512, 2600: 240 and 273), twelve at N = 4096 (2600: 3624 and 3915;
//     3500: 4355 and 4349); eight at N = 256 (2304: 169 and 160) and N = 2048
//     (2600: 1683 and 1623);
//   - counting and threshold selection with L = 32 work frame by frame, so they
//     fill the chip first (counting, 3000 frames: 1555 and 2025).
static int64_t scl_target(int n, int L, int rank, bool aided) {
    int per_cu = 8;
    if (other_ranking(n, L, rank) && L == 32) per_cu = 16;
    else if (L == 32 && (n == 9 || n == 10)) per_cu = aided ? 12 : 10;
    else if (L == 32 && n == 12) per_cu = 12;
    return (int64_t)device_cu_count() * per_cu;
}

polar_status scl_plan(const polar_code* code, int L, int64_t max_frames, SclPlan* plan, int max_fpw) {
    return scl_plan_dims(code->n, L, max_frames, plan, max_fpw, 5 * code->n_da >= 2 * code->k);
}

polar_status scl_plan_dims(int n, int L, int64_t max_frames, SclPlan* plan, int max_fpw, bool aided) {
    const int rank = rank_kind();
    scl::KernelFn fn = scl::pick(L, n, rank);
    if (!fn) return set_error(POLAR_ERR_INVALID_ARG, "scl: L must be a power of two in [1, 32]");
    // frames a wavefront may take at once: as many as its lanes hold lists,
    // if there can be that many frames
    int fpw = 1;
    const int64_t target = scl_target(n, L, rank, aided);
    while (2 * fpw <= frames_room(n, L, rank) && 2 * fpw <= max_fpw && fpw * target < max_frames) fpw *= 2;
    const int slots = L * fpw;
    // tree levels: level 5 in LDS (read by every bit of a block), the levels
    // above in the workgroup's global slice (each written and read once per
    // block start that reaches it, as a stream); the trace in LDS if it fits
    // the budget, else in the global slice
    const size_t budget = scl_budget(fn);
    plan->lds_bytes = 0;
    bool tg = false;  // either form's trace in the slice
    for (int several = 0; several < 2; ++several) {
        const int s = several ? slots : L;
        bool glob = false;
        scl::LdsPlan lp = scl::lds_plan(L, s, n, glob);
        if (lp.bytes > budget) {
            glob = true;
            lp = scl::lds_plan(L, s, n, glob);
        }
        if (lp.bytes > 160 * 1024) return set_error(POLAR_ERR_UNSUPPORTED, "scl: list too large for LDS");
        plan->form[several] = SclForm{s, lp.soff, glob ? 1 : 0, lp.tboff};
        if (lp.bytes > plan->lds_bytes) plan->lds_bytes = lp.bytes;
        tg = tg || glob;
    }
    int per_cu = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64, plan->lds_bytes);
    if (e != hipSuccess || per_cu <= 0) per_cu = 1;
    int64_t grid = (int64_t)device_cu_count() * per_cu;
    if (max_frames < grid) grid = max_frames;
    if (grid < 1) grid = 1;
    size_t lam_b = 0;
    if (n > 6) {  // (level 5 alone needs no row)
        const size_t one = (size_t)L << scl::row_log(n, false), many = (size_t)slots << scl::row_log(n, true);
        lam_b = (fpw > 1 && many > one ? many : one) * 4;
    }
    plan->trace_off = lam_b;
    plan->glob_per_wg = align_up(lam_b + (tg ? scl::trace_bytes(slots, n) : 0), 256);
    plan->grid = (int)grid;
    plan->target = (int)target;
    plan->lay_n = n;
    plan->rank = rank;
    return POLAR_OK;
}

// The share of one list decode by which hybrid_decode_batch_static takes or
// refuses a batch: every LLR level above 5 of L paths, and the trace where it
// did not fit the LDS budget beside a frame's whole state (level 5, all partial
// sums from level 5 on, 64 candidates).
size_t scl_static_share(int n, int L) {
    const size_t trace = scl::trace_bytes(L, n);
    size_t lds = (size_t)L * ((n > 5 ? 36 : 4) + (n <= 5 ? 1 : (1 << (n - 5)) - 1)) * 4 + 256;
    const size_t chain = align_up(((size_t)1 << (n - (n < 5 ? n : 5))) * 4, 16);
    lds = align_up(align_up(lds > chain ? lds : chain, 16) + trace, 16);
    const size_t levels = n > 6 ? ((size_t)L << n) * 4 : 0;
    return align_up(levels + (lds > scl_budget(scl::pick(L, n, rank_kind())) ? trace : 0), 256);
}

polar_status launch_scl(const polar_code* code, const SclPlan& plan, const float* llr, int L, const SclWork& work,
                        const SclOut& out, void* glob, hipStream_t stream, const MixedIo* io) {
    scl::KernelFn fn = scl::pick(L, plan.lay_n, plan.rank);
    scl::Layout lay;
    lay.form[0] = plan.form[0];
    lay.form[1] = plan.form[1];
    lay.fpw = plan.form[1].slots / L;
    lay.grid[0] = plan.grid;
    lay.target = plan.target < plan.grid ? plan.target : plan.grid;
    lay.nblk = (1 << plan.lay_n) >> (plan.lay_n < 5 ? plan.lay_n : 5);
    lay.gbytes = (int64_t)plan.glob_per_wg;
    lay.toff = (int64_t)plan.trace_off;
    unsigned char* gb = plan.glob_per_wg ? reinterpret_cast<unsigned char*>(glob) : nullptr;
    hipLaunchKernelGGL(fn, dim3(plan.grid), dim3(64), plan.lds_bytes, stream, code->dev(), llr, work, out, gb, lay,
                       io);
    return hip_check(hipGetLastError(), "scl_kernel launch");
}

}  // namespace polarhip

using namespace polarhip;

extern "C" polar_status scl_decode_batch(const polar_code* code, const float* llr, int64_t B, int32_t L,
                                         const int32_t* frame_ids, uint8_t* u_hat, uint8_t* crc_ok, float* pm,
                                         void* ws, size_t ws_bytes, hipStream_t stream) {
    if (!code) return set_error(POLAR_ERR_INVALID_ARG, "scl_decode_batch: null code");
    if (B < 0) return set_error(POLAR_ERR_INVALID_ARG, "scl_decode_batch: negative batch");
    if (B > 0 && (!llr || !u_hat || !crc_ok)) return set_error(POLAR_ERR_INVALID_ARG, "scl_decode_batch: null buffer");
    SclPlan plan;
    polar_status st = scl_plan(code, L, B, &plan);
    if (st != POLAR_OK) return st;
    if (B == 0) return ok_status();
    const size_t need = plan.glob_per_wg * plan.grid;
    if (need && (!ws || ws_bytes < need)) return set_error(POLAR_ERR_WORKSPACE, "scl_decode_batch: workspace too small");
    SclOut out;
    out.u_hat = u_hat;
    out.crc_ok = crc_ok;
    out.pm = pm;
    st = launch_scl(code, plan, llr, L, SclWork::list(frame_ids, nullptr, B), out, ws, stream);
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status polar_set_scl_lds_budget(int64_t bytes) {
    if (bytes != 0 && (bytes < 4096 || bytes > 160 * 1024))
        return set_error(POLAR_ERR_INVALID_ARG, "polar_set_scl_lds_budget: bytes must be 0 or in [4096, 163840]");
    g_scl_lds_budget.store(bytes, std::memory_order_relaxed);
    return ok_status();
}

extern "C" int64_t polar_get_scl_lds_budget(void) { return g_scl_lds_budget.load(std::memory_order_relaxed); }

extern "C" polar_status polar_set_scl_ranking(int32_t mode) {
    if (mode < 0 || mode > 3) return set_error(POLAR_ERR_INVALID_ARG, "polar_set_scl_ranking: mode must be 0..3");
    g_scl_rank_mode.store(mode, std::memory_order_relaxed);
    return ok_status();
}

extern "C" int32_t polar_get_scl_ranking(void) { return g_scl_rank_mode.load(std::memory_order_relaxed); }
