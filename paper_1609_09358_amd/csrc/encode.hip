// encode.hip -- polar encoder x = u G (Sec. II, Fig. 1) and the BPSK/AWGN
// channel used to synthesise workloads.
#include "internal.hpp"
#include "lane_ops.hpp"

namespace polarhip {
namespace {

constexpr int ENC_THREADS = 256;
constexpr int ENC_WAVES = ENC_THREADS / 64;

// Bound by HBM: K bytes read and N (with u 2 N) written per frame, one byte
// per bit.  Between the two a frame is held as bits: a wavefront encodes
// 1024 / N frames at a time (one from N = 1024 on), lane l of a frame holding
// nodes 16 l .. 16 l + 15 as 16 bits (N > 1024: of every 1024-node group; N = 8:
// 8 bits), so its bytes are one 16-byte store per output.
//   - The wavefront's information bytes are consecutive in memory: each lane
//     takes aligned 16-byte granules of them (a dot product per four bytes packs
//     their low bits) and puts 16 bits into LDS.
//   - A lane's non-frozen positions take consecutive information bits, from
//     its rank on (a prefix sum of the mask, once per wavefront): two words
//     from LDS, a funnel shift, and a bit deposit in log2(16) steps whose
//     masks are computed once per wavefront (parallel suffix, as in Warren,
//     Hacker's Delight, "expand").
//   - The CRC is the XOR of the per-position syndromes of the set bits,
//     reduced over the frame's lanes; its bits continue the string.
//   - Butterflies: distances 1..8 inside the word, 16..512 lane exchanges,
//     1024 and up between a lane's groups.
// Wavefronts are persistent, so the tables are read once per wavefront.
// Measured at N = 1024, K = 512, CRC-24, 65536 frames (168 MB): 280 us for one
// workgroup per frame with one byte per bit in LDS, 39 us this way.
template <int NLOG>
struct EncGeom {
    static constexpr int N = 1 << NLOG;
    static constexpr int PPL = N < 16 ? 8 : 16;                      // positions per lane and group
    static constexpr int TL = N / PPL > 64 ? 64 : N / PPL;           // lanes per frame
    static constexpr int G = N / (PPL * TL);                         // groups of PPL * TL positions
    static constexpr int FPW = 64 / TL;                              // frames per wavefront
    static constexpr int STEPS = PPL == 16 ? 4 : 3;                  // deposit and in-word butterfly steps
    // LDS words of one wavefront's bit string: up to 15 leading bytes of the
    // first granule, and the second word of the last window
    static constexpr int WORDS = (N > 1024 ? N : 1024) / 32 + 4;
};

// low bits of the 16 bytes of v, byte j to bit j
__device__ __forceinline__ uint32_t pack16(const uint4& v) {
    const uint32_t m = 0x01010101u, lo = 0x08040201u, hi = 0x80402010u;
    uint32_t a = __builtin_amdgcn_udot4(v.x & m, lo, 0u, false);
    a = __builtin_amdgcn_udot4(v.y & m, hi, a, false);
    uint32_t b = __builtin_amdgcn_udot4(v.z & m, lo, 0u, false);
    b = __builtin_amdgcn_udot4(v.w & m, hi, b, false);
    return a | (b << 8);
}

// bits 0..3 of b to the low bits of four bytes
__device__ __forceinline__ uint32_t spread4(uint32_t b) { return ((b & 0xFu) * 0x00204081u) & 0x01010101u; }

template <int PPL, bool ALIGNED>
__device__ __forceinline__ void store_bits(uint8_t* dst, uint32_t b) {
    if constexpr (ALIGNED && PPL == 16) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(spread4(b), spread4(b >> 4), spread4(b >> 8), spread4(b >> 12));
    } else if constexpr (ALIGNED) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(spread4(b), spread4(b >> 4));
    } else {
#pragma unroll
        for (int j = 0; j < PPL; ++j) dst[j] = (uint8_t)((b >> j) & 1u);
    }
}

template <int NLOG, bool ALIGNED>
__global__ __launch_bounds__(ENC_THREADS) void encode_kernel(CodeDev code, const uint8_t* __restrict__ info, int64_t B,
                                                             uint8_t* __restrict__ u_out,
                                                             uint8_t* __restrict__ x_out, int grid) {
    using E = EncGeom<NLOG>;
    constexpr int PPL = E::PPL, TL = E::TL, G = E::G, FPW = E::FPW, STEPS = E::STEPS;
    constexpr uint32_t FULL = (1u << PPL) - 1u;
    __shared__ uint32_t bits_all[ENC_WAVES][E::WORDS];
    const int lane = lid_x() & 63, wave = lid_x() >> 6;
    const int sub = lane & (TL - 1), slot = lane / TL;
    uint32_t* bits = bits_all[wave];
    uint16_t* bits16 = reinterpret_cast<uint16_t*>(bits);
    const int K = code.K, c = code.c;

    // this lane's positions in each group: mask of the non-frozen ones, the
    // rank of the first, deposit masks and CRC syndromes
    uint32_t mask[G], step[G][STEPS], syn[G][PPL];
    int rank[G];
    int before = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int p0 = g * PPL * TL + sub * PPL;
        mask[g] = ~(code.frozen_bits[p0 >> 5] >> (p0 & 31)) & FULL;
        const int cnt = __popc(mask[g]);
        int sum = cnt;  // inclusive prefix over the frame's lanes
#pragma unroll
        for (int d = 1; d < TL; d <<= 1) {
            const int o = __shfl_up(sum, d, 64);
            if (sub >= d) sum += o;
        }
        rank[g] = before + sum - cnt;
        before += __shfl(sum, lane | (TL - 1), 64);
        uint32_t m = mask[g], mk = (~m << 1) & FULL;
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            uint32_t mp = mk ^ (mk << 1);
            mp ^= mp << 2;
            mp ^= mp << 4;
            mp ^= mp << 8;
            step[g][i] = mp & m;
            m = (m ^ step[g][i]) | (step[g][i] >> (1 << i));
            mk &= ~mp;
        }
#pragma unroll
        for (int j = 0; j < PPL; ++j) syn[g][j] = c ? code.syn[p0 + j] : 0u;
    }
    // the low bits of s to the set positions of mask[g], in order
    auto deposit = [&](int g, uint32_t s) {
#pragma unroll
        for (int i = STEPS - 1; i >= 0; --i) s = (s & ~step[g][i]) | ((s << (1 << i)) & step[g][i]);
        return s & mask[g];
    };

    const uint8_t* const info_end = info + B * (int64_t)K;
    const int64_t stride = (int64_t)grid * (ENC_WAVES * FPW);
    for (int64_t f0 = (gid_x() * ENC_WAVES + wave) * FPW; f0 < B; f0 += stride) {
        // ---- information bytes of the wavefront's frames, as bits in LDS
        const int64_t left = B - f0;
        const int bytes = (left < FPW ? (int)left : FPW) * K;
        const uint8_t* first = info + f0 * K;
        const int lead = (int)(reinterpret_cast<uintptr_t>(first) & 15u);
        const uint8_t* base = first - lead;  // granule boundary
        for (int q = lane; 16 * q < lead + bytes; q += 64) {
            const uint8_t* p = base + 16 * q;
            uint32_t w = 0;
            if (p >= info && p + 16 <= info_end) {
                w = pack16(*reinterpret_cast<const uint4*>(p));
            } else {  // a granule that reaches past either end of the buffer
                for (int j = 0; j < 16; ++j)
                    if (p + j >= info && p + j < info_end) w |= (uint32_t)(p[j] & 1u) << j;
            }
            bits16[q] = (uint16_t)w;
        }
        wave_lds_sync();
        // ---- u: information bits, then the CRC's
        uint32_t u[G];
        uint32_t s = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int o = lead + slot * K + rank[g];
            const uint64_t win = ((uint64_t)bits[(o >> 5) + 1] << 32) | bits[o >> 5];
            uint32_t w = (uint32_t)(win >> (o & 31));
            const int nk = K - rank[g];  // positions before the CRC's
            w = nk >= PPL ? w : (nk > 0 ? w & ((1u << nk) - 1u) : 0u);
            u[g] = deposit(g, w);
            if (c) {
#pragma unroll
                for (int j = 0; j < PPL; ++j) s ^= syn[g][j] & (uint32_t)(((int32_t)(u[g] << (31 - j))) >> 31);
            }
        }
        if (c) {
            // CRC bit j of the string is bit c - 1 - j of the register
            const uint32_t str = __builtin_bitreverse32(group_xor<TL>(s)) >> (32 - c);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int nk = K - rank[g];
                const uint32_t w = nk >= PPL ? 0u : (nk >= 0 ? str << nk : (nk > -32 ? str >> -nk : 0u));
                u[g] |= deposit(g, w);
            }
        }
        const int64_t f = f0 + slot;
        const bool valid = FPW == 1 || f < B;
        const int64_t row = f * E::N + sub * PPL;
        if (u_out && valid) {
#pragma unroll
            for (int g = 0; g < G; ++g) store_bits<PPL, ALIGNED>(u_out + row + g * PPL * TL, u[g]);
        }
        // ---- x = u G
#pragma unroll
        for (int g = 0; g < G; ++g) {
            u[g] ^= (u[g] >> 1) & 0x5555u;
            u[g] ^= (u[g] >> 2) & 0x3333u;
            u[g] ^= (u[g] >> 4) & 0x0F0Fu;
            if constexpr (PPL == 16) u[g] ^= (u[g] >> 8) & 0x00FFu;
            static_for<0, 6>([&](auto QC) {
                constexpr int q = 1 << decltype(QC)::value;
                if constexpr (q < TL) {
                    const uint32_t o = from_lane_above<q>(u[g]);
                    u[g] ^= (lane & q) == 0 ? o : 0u;
                }
            });
        }
#pragma unroll
        for (int d = 1; d < G; d <<= 1)
#pragma unroll
            for (int g = 0; g < G; ++g)
                if ((g & d) == 0) u[g] ^= u[g + d];
        if (valid) {
#pragma unroll
            for (int g = 0; g < G; ++g) store_bits<PPL, ALIGNED>(x_out + row + g * PPL * TL, u[g]);
        }
        wave_lds_sync();  // the next frames' bits go over these
    }
}

using EncodeFn = void (*)(CodeDev, const uint8_t*, int64_t, uint8_t*, uint8_t*, int);

struct EncodeEntry {
    EncodeFn aligned, any;
    int fpw;
};

template <int NLOG>
constexpr EncodeEntry encode_entry() {
    return EncodeEntry{&encode_kernel<NLOG, true>, &encode_kernel<NLOG, false>, EncGeom<NLOG>::FPW};
}

const EncodeEntry& encode_lookup(int n) {
    static const EncodeEntry table[10] = {encode_entry<3>(), encode_entry<4>(),  encode_entry<5>(),  encode_entry<6>(),
                                          encode_entry<7>(), encode_entry<8>(),  encode_entry<9>(),  encode_entry<10>(),
                                          encode_entry<11>(), encode_entry<12>()};
    return table[n - 3];
}

__device__ __forceinline__ float awgn_llr(uint32_t bit, float sd, float z, float s2) {
    const float y = (bit ? -1.0f : 1.0f) + sd * z;
    return 2.0f * y / s2;
}

__global__ __launch_bounds__(256) void channel_kernel(const uint8_t* __restrict__ x, const float* __restrict__ z,
                                                      const float* __restrict__ sigma2, int64_t total, int32_t N,
                                                      float* __restrict__ llr) {
    const int64_t idx = gid_x() * 256 + lid_x();
    if (idx >= total) return;
    const float s2 = sigma2[idx / N];
    llr[idx] = awgn_llr(x[idx], sqrtf(s2), z[idx], s2);
}

// Four elements of one row per thread (rows of 2^n >= 4 elements, buffers
// aligned to the loads: 4 bytes for x, 16 for z and llr): a quarter of the
// address arithmetic, a shift for the row instead of a 64-bit division, one
// square root for the four.  Bound by HBM (9 bytes per element): 67 M elements
// in 191 us one at a time, 105 us this way (5.8 TB/s).
__global__ __launch_bounds__(256) void channel4_kernel(const uint8_t* __restrict__ x, const float* __restrict__ z,
                                                       const float* __restrict__ sigma2, int64_t quads, int32_t rshift,
                                                       float* __restrict__ llr) {
    const int64_t q = gid_x() * 256 + lid_x();
    if (q >= quads) return;
    const float s2 = sigma2[q >> rshift];
    const uint32_t xb = reinterpret_cast<const uint32_t*>(x)[q];
    const float4 zv = reinterpret_cast<const float4*>(z)[q];
    const float sd = sqrtf(s2);
    float4 o;
    o.x = awgn_llr(xb & 0x000000FFu, sd, zv.x, s2);
    o.y = awgn_llr(xb & 0x0000FF00u, sd, zv.y, s2);
    o.z = awgn_llr(xb & 0x00FF0000u, sd, zv.z, s2);
    o.w = awgn_llr(xb & 0xFF000000u, sd, zv.w, s2);
    reinterpret_cast<float4*>(llr)[q] = o;
}

bool aligned_to(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

}  // namespace
}  // namespace polarhip

using namespace polarhip;

extern "C" polar_status polar_encode(const polar_code* code, const uint8_t* info, int64_t B,
                                     uint8_t* u_out, uint8_t* x_out, hipStream_t stream) {
    if (!code || !x_out || (B > 0 && !info)) return set_error(POLAR_ERR_INVALID_ARG, "polar_encode: null argument");
    if (B < 0 || B > (int64_t)INT32_MAX) return set_error(POLAR_ERR_INVALID_ARG, "polar_encode: bad batch size");
    if (B == 0) return ok_status();
    const EncodeEntry& e = encode_lookup(code->n);
    const int64_t per = (int64_t)ENC_WAVES * e.fpw;
    int64_t grid = (B + per - 1) / per;
    // the wavefronts that fit the chip, each walking the batch
    const int64_t cap = (int64_t)device_cu_count() * 8;
    if (grid > cap) grid = cap;
    // 16-byte stores need the outputs on such boundaries (any other pointer:
    // one byte at a time)
    const EncodeFn fn = aligned_to(x_out, 16) && (!u_out || aligned_to(u_out, 16)) ? e.aligned : e.any;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(ENC_THREADS), 0, stream, code->dev(), info, B, u_out, x_out,
                       (int)grid);
    return hip_check(hipGetLastError(), "encode_kernel launch") == POLAR_OK ? ok_status() : POLAR_ERR_DEVICE;
}

extern "C" polar_status polar_channel_awgn(const uint8_t* x, const float* z, const float* sigma2, int64_t B,
                                           int32_t N, float* llr, hipStream_t stream) {
    if (!x || !z || !sigma2 || !llr) return set_error(POLAR_ERR_INVALID_ARG, "polar_channel_awgn: null argument");
    if (B < 0 || N <= 0) return set_error(POLAR_ERR_INVALID_ARG, "polar_channel_awgn: bad sizes");
    int64_t total = B * (int64_t)N;
    if (total == 0) return ok_status();
    if (N >= 4 && (N & (N - 1)) == 0 && aligned_to(x, 4) && aligned_to(z, 16) && aligned_to(llr, 16)) {
        const int64_t quads = total / 4;
        hipLaunchKernelGGL(channel4_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, stream, x, z, sigma2,
                           quads, __builtin_ctz((unsigned)N) - 2, llr);
    } else {
        const unsigned blocks = (unsigned)((total + 255) / 256);
        hipLaunchKernelGGL(channel_kernel, dim3(blocks), dim3(256), 0, stream, x, z, sigma2, total, N, llr);
    }
    return hip_check(hipGetLastError(), "channel_kernel launch") == POLAR_OK ? ok_status() : POLAR_ERR_DEVICE;
}
