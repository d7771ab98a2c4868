// bp.hip -- batched min-sum belief-propagation decoder of polar codes
// (Sec. II-B, Fig. 2), plain and weighted, with early stopping by the
// re-encoding check or the CRC.
//
// Design (MI355X / gfx950).  Messages live in registers.  A frame of N = 2^n
// nodes per stage is spread over T = N / V threads, each holding V = 2^r nodes
// of every stage row.  Which r index bits a thread holds in registers changes
// along the sweep: window k keeps bits [b_k, b_k + r) in registers and handles
// the PE columns that pair those bits, so every butterfly is computed inside
// one thread without communication.  Between windows the single row on the
// boundary is re-laid out through LDS (one write and one read per value).
// The LDS address of an index is a sum of per-bit coefficients chosen at
// compile time so that, for both layouts of a boundary, the 32 lanes of a
// half-wavefront hit 32 different banks and the register part of the address
// is an immediate offset.  Boundaries whose layouts differ only inside one
// wavefront need no barrier; the others are separated by a workgroup barrier.
// When a frame needs fewer than 64 threads, one wavefront carries 64 / T
// frames, each leaving the iteration loop on its own.
//
// PE arithmetic (min-sum inference): a PE's two g terms share one operand a,
// and g(a, b) = sgn(a) clamp(b, -|a|, |a|), so the sign of a is moved once
// into the weight and each g is one clamp; with one weight per stage column
// and every weight within [-1, 1] a second copy of the decoder leaves out the
// first output's clip, which cannot act there.
//
// Early stop (Sec. II-B): after each iteration the hard decisions on LLR(u)
// and LLR(x) are stored as bits (eight-register layouts; bytes otherwise) and
// gathered into words of N / 64 bits per checker lane, u_hat is re-encoded
// with shifts inside words and lane exchanges across words, and compared with
// x_hat; the CRC test uses per-nibble syndrome tables.
#include "bp_common.hpp"

namespace polarhip {
namespace bp {

template <class G>
__device__ __forceinline__ uint64_t load_bits(const uint8_t* src) {
    // CB bytes (0/1) starting at src -> CB-bit word, bit j = byte j
    uint64_t w = 0;
    if constexpr (G::CB >= 4) {
#pragma unroll
        for (int q = 0; q < G::CB / 4; ++q) {
            uint32_t d = reinterpret_cast<const uint32_t*>(src)[q];
            uint32_t nib = ((d * 0x01020408u) >> 24) & 0xFu;
            w |= (uint64_t)nib << (4 * q);
        }
    } else {
#pragma unroll
        for (int q = 0; q < G::CB; ++q) w |= (uint64_t)(src[q] & 1u) << q;
    }
    return w;
}

// Packed decisions (V = 8 and a frame of at least one wavefront): bit j of
// the frame's bit array is node j.  Checker lane l's CB consecutive bits, read
// in one access.
template <class G>
__device__ __forceinline__ uint64_t read_bits(const uint8_t* bits, int lane) {
    if constexpr (G::CB == 8) return bits[lane];
    else if constexpr (G::CB == 16) return reinterpret_cast<const uint16_t*>(bits)[lane];
    else if constexpr (G::CB == 32) return reinterpret_cast<const uint32_t*>(bits)[lane];
    else return reinterpret_cast<const uint64_t*>(bits)[lane];
}

template <class G, bool PACKED>
__device__ __forceinline__ uint64_t lane_bits(const uint8_t* src, int lane) {
    if constexpr (PACKED) return read_bits<G>(src, lane);
    else return load_bits<G>(src + lane * G::CB);
}

// bits p of a 64-bit word with p & d == 0 (d a power of two)
constexpr uint64_t low_half_mask(int d) {
    uint64_t m = 0;
    for (int p = 0; p < 64; ++p)
        if ((p & d) == 0) m |= 1ull << p;
    return m;
}

// u G == x on the words of one frame's checker lanes; every one of them gets
// the answer
template <class G>
__device__ __forceinline__ bool reencode_words(uint64_t u, uint64_t x, int lane) {
    // butterflies inside a word: distances 1, 2, .. CB/2 (masks fixed at compile time)
    static_for<0, 6>([&](auto D) {
        constexpr int d = 1 << decltype(D)::value;
        if constexpr (d < G::CB) {
            constexpr uint64_t m = low_half_mask(d);
            u ^= (u >> d) & m;
        }
    });
    // butterflies across the checker lanes: lanes with bit q clear take lane + q
    static_for<0, 6>([&](auto QC) {
        constexpr int q = 1 << decltype(QC)::value;
        if constexpr (q < G::TL) {
            const uint32_t lo = from_lane_above<q>((uint32_t)u);
            const uint32_t hi = G::CB > 32 ? from_lane_above<q>((uint32_t)(u >> 32)) : 0u;
            if ((lane & q) == 0) u ^= ((uint64_t)hi << 32) | lo;
        }
    });
    uint64_t bad = __ballot(u != x);
    if constexpr (G::TL < 64) {
        const int grp = (__lane_id() / G::TL) * G::TL;
        bad = (bad >> grp) & ((1ull << G::TL) - 1ull);
    }
    return bad == 0;
}

// the same on decisions in LDS
template <class G, bool PACKED>
__device__ __forceinline__ bool reencode_check(const uint8_t* ub, const uint8_t* xb, int lane) {
    return reencode_words<G>(lane_bits<G, PACKED>(ub, lane), lane_bits<G, PACKED>(xb, lane), lane);
}

// Frames of at most one wavefront whose threads hold at least as many lanes as
// registers (T >= V, T >= 8): a checker lane's bits of u are its own thread's,
// nodes V t .. V t + V - 1 of window 0, so u never goes through LDS.  Its bits of
// x are V bits of one of the ballots taken in the last window, where lane t
// holds node t + (v << P) in register v.
template <class G>
constexpr bool own_bits() {
    return G::T <= 64 && G::T >= 8 && G::T >= G::V && (G::V == 4 || G::V == 8);
}

template <class G>
__device__ __forceinline__ uint32_t own_x_bits(const uint64_t* words, int t, int slot) {
    const int i = G::V * t;                               // first node
    const int b = slot * G::T + (i & (G::T - 1));         // its bit in the ballot of register i >> P
    const uint32_t byte = reinterpret_cast<const uint8_t*>(words)[((i >> G::P) << 3) + (b >> 3)];
    return (byte >> (b & 7)) & ((1u << G::V) - 1u);
}

template <class G>
__device__ __forceinline__ bool own_crc(const CodeDev& code, uint32_t bits, int t) {
    if (code.c == 0) return true;
    const uint32_t* tab = code.syn_nib + (size_t)t * (G::V / 4) * 16;
    uint32_t s = tab[bits & 15u];
    if constexpr (G::V == 8) s ^= tab[16 + (bits >> 4)];
    return group_xor<G::TL>(s) == 0;
}

template <class G, bool PACKED>
__device__ __forceinline__ bool crc_check(const CodeDev& code, const uint8_t* ub, int lane) {
    if (code.c == 0) return true;
    uint64_t u = lane_bits<G, PACKED>(ub, lane);
    uint32_t s = 0;
    const uint32_t* tab = code.syn_nib + (size_t)(lane * G::CB / 4) * 16;
    if constexpr (G::CB >= 4) {
#pragma unroll
        for (int g = 0; g < G::CB / 4; ++g) s ^= tab[g * 16 + ((u >> (4 * g)) & 0xF)];
    } else {
        // fewer than 4 bits per lane: take the nibble from the lanes of the group
        const int g = lane * G::CB / 4;
        const int sh = (lane * G::CB) & 3;
        uint32_t part = (uint32_t)(u << sh);
        uint32_t nib = part;
#pragma unroll
        for (int q = 1; q < 4 / G::CB; ++q) nib |= __shfl_xor(part, q, 64);
        s = (sh == 0) ? code.syn_nib[(size_t)g * 16 + (nib & 0xF)] : 0u;
    }
    return group_xor<G::TL>(s) == 0;
}

// LDS of one workgroup: transpose buffers, the packed-decision staging and
// the wavefronts' partial CRC syndromes (two sets, taken by iteration parity)
template <class G>
struct BpShared {
    float tb[G::TAB.words];
    __attribute__((aligned(16))) uint8_t ubytes[G::FPW * G::N];
    __attribute__((aligned(16))) uint8_t xbytes[G::FPW * G::N];
    uint32_t syn[2][G::NWAVES];
};

// CRC test of a frame of at least one wavefront whose thread t holds its own
// packed decisions, nodes 8t .. 8t + 7 (nibble positions 2t and 2t + 1): each
// thread XORs the syndromes of its two nibbles, each wavefront reduces its
// lanes, and the frame's wavefronts combine their words through LDS.  syn is
// one of two sets taken by iteration parity: a wavefront's next write goes to
// the other set, and the one after it follows the next test's barrier, which
// every wavefront reaches only after its reads.  Every thread of the frame gets
// the answer; ends with a frame-wide barrier.
template <class G>
__device__ __forceinline__ bool crc_check_own(const CodeDev& code, uint32_t bits, int t, uint32_t* syn) {
    static_assert(G::V == 8 && G::T >= 64, "packed decisions of whole wavefronts");
    uint32_t s = 0;
    if (code.c != 0) {
        // byte offsets of the two table entries (bits < 256) from the
        // table's uniform base: 32-bit lane offsets, no per-lane pointer
        const uint8_t* tab = reinterpret_cast<const uint8_t*>(code.syn_nib);
        const uint32_t row = (uint32_t)t << 7;
        const uint32_t o0 = row | ((bits & 15u) << 2);
        const uint32_t o1 = row | 64u | ((bits >> 2) & 0x3Cu);
        s = group_xor<64>(*reinterpret_cast<const uint32_t*>(tab + o0) ^
                          *reinterpret_cast<const uint32_t*>(tab + o1));
    }
    if constexpr (G::NWAVES == 1) {
        frame_sync<G>();
        return s == 0;
    } else {
        if ((t & 63) == 0) syn[t >> 6] = s;
        frame_sync<G>();
        uint32_t a = 0;
#pragma unroll
        for (int w = 0; w < G::NWAVES; ++w) a ^= syn[w];
        return a == 0;
    }
}

// Where one frame's data lives.  SAVE (training): every message a column
// produces is also written to sv[iteration][direction][column][node],
// direction 0 = R (row s+1 of column s), 1 = L (row s), for the adjoint kernel.
struct FrameIO {
    const float* llr;   // [N] channel LLRs
    uint8_t* u_hat;     // [N] or null
    uint8_t* info;      // [K] or null: information bits, written when the verdict is ok
    float* llr_u;       // [N] or null
    int32_t* iters;     // one value or null
    uint8_t* ok;        // one value or null
    float* saved;       // SAVE only
};

// Decode one frame: thread t of the frame's T threads, frame slot `slot` of
// its wavefront (T < 64) or workgroup.  Returns the verdict (for queues).
// NOCLIP (per-stage weights, every weight within [-1, 1]): the first output
// of a PE is w g with |w g| <= |g| <= lmax, so its clip would return its input
// and is left out.
template <class G, bool WEIGHTED, bool SAVE, int RULE = 0, bool WSTAGE = false, bool NOCLIP = false>
__device__ __forceinline__ bool bp_frame(const CodeDev& code, const FrameIO& io, int max_iter, int stop, float lmax,
                                         const float* __restrict__ W, BpShared<G>& sh, int t, int slot) {
    constexpr int n = G::n, N = G::N, V = G::V, KL = G::NWIN - 1;
    // min-sum inference takes the sign-transfer form of g; training (SAVE)
    // and the exact rule keep the direct form
    constexpr bool FAST = RULE == 0 && !SAVE;
    // decisions stored as bits instead of one byte each (u: one byte per
    // thread of window 0, its eight consecutive nodes; x: one ballot per
    // register and wavefront, since in the last window a wavefront's lanes
    // hold 64 consecutive nodes)
    // Frames of one wavefront keep u in registers (own_bits above): N = 128, 1000
    // frames of at most 100 iterations 104 us with both in LDS, 99 us this way.
    // Not for decoding with a weight per node: the compiler then holds fewer weights
    // ahead (N = 512, r = 3, 256 frames of at most 10 iterations 42 us with both in
    // LDS, 62 us without)
    constexpr bool OWN = own_bits<G>() && (!WEIGHTED || WSTAGE || SAVE);
    constexpr bool BITPACK = G::V == 8 && G::T >= 64 && !OWN;
    float* tb = sh.tb;
    const int lane = (G::T < 64) ? t : (lid_x() & 63);
    uint8_t* ub = sh.ubytes + slot * N;
    uint8_t* xb = sh.xbytes + slot * N;

    // LDS bases of this thread for each boundary, on both sides
    int bfrom[G::NB > 0 ? G::NB : 1], bto[G::NB > 0 ? G::NB : 1];
    static_for<0, G::NB>([&](auto J) {
        constexpr int j = decltype(J)::value;
        bfrom[j] = lds_base<G, j, j>(t, slot);
        bto[j] = lds_base<G, j, j + 1>(t, slot);
    });

    // messages: row rho of L / R, each V values in the layout of the window
    // that stores it
    float Lm[n + 1][V];
    float Rm[n + 1][V];
    float prior[V];
#pragma unroll
    for (int s = 0; s <= n; ++s)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            Lm[s][v] = 0.0f;
            Rm[s][v] = 0.0f;
        }
    const float* fl = io.llr;
    {
        const int ib = idx_base<G, KL>(t);
#pragma unroll
        for (int v = 0; v < V; ++v) Lm[n][v] = clipf(fl[ib + (v << G::wbase(KL))], lmax);
    }
    uint32_t fmask = 0;  // frozen flags of this thread's nodes in window 0
    {
        const int ib = idx_base<G, 0>(t);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            int i = ib + v;
            uint32_t f = (code.frozen_bits[i >> 5] >> (i & 31)) & 1u;
            fmask |= f << v;
            prior[v] = f ? lmax : 0.0f;
        }
    }

    int it = 0;
    bool gok = false, cok = false;
    uint32_t ubits = 0;  // packed decisions of this thread's nodes (BITPACK)
    while (true) {
        const float* Wit = WEIGHTED ? W + (size_t)it * 2 * n * (WSTAGE ? 1 : N) : nullptr;
        float* Sit = SAVE ? io.saved + (size_t)it * 2 * n * N : nullptr;
        // ---------------- R sweep: columns 0..n-1
        static_for<0, G::NWIN>([&](auto KC) {
            constexpr int k = decltype(KC)::value;
            const int ib = idx_base<G, k>(t);
            static_for<G::cbeg(k), G::cend(k)>([&](auto SC) {
                constexpr int s = decltype(SC)::value;
                constexpr int q = s - G::wbase(k);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (v & (1 << q)) continue;
                    const int v2 = v | (1 << q);
                    const float r1 = (s == 0) ? prior[v] : Rm[s][v];
                    const float r2 = (s == 0) ? prior[v2] : Rm[s][v2];
                    const float l1 = Lm[s + 1][v], l2 = Lm[s + 1][v2];
                    if constexpr (FAST) {
                        // both g terms share r1: its sign rides on the weight
                        const float x = l2 + r2;
                        if constexpr (WEIGHTED) {
                            float wi, wj;
                            if constexpr (WSTAGE) {
                                wi = wj = Wit[0 * n + s];
                            } else {
                                const float* w = Wit + (size_t)(0 * n + s) * N + ib;
                                wi = w[v << G::wbase(k)];
                                wj = w[v2 << G::wbase(k)];
                            }
                            // column 0: r1 is the prior, 0 or lmax > 0, whose
                            // sign leaves the weight as it is
                            const float si = (s == 0) ? wi : sign_to(wi, r1);
                            const float sj = WSTAGE ? si : ((s == 0) ? wj : sign_to(wj, r1));
                            const float yi = si * clamp_mag(x, r1);
                            Rm[s + 1][v] = NOCLIP ? yi : clipf(yi, lmax);
                            Rm[s + 1][v2] = clipf(__fmaf_rn(sj, clamp_mag(l1, r1), r2), lmax);
                        } else {
                            const float si = (s == 0) ? 1.0f : sign_to(1.0f, r1);
                            Rm[s + 1][v] = si * clamp_mag(x, r1);  // |g| <= |r1| <= lmax
                            Rm[s + 1][v2] = clipf(__fmaf_rn(si, clamp_mag(l1, r1), r2), lmax);
                        }
                        continue;
                    }
                    const float gi = g_rule<RULE>(r1, l2 + r2);
                    const float gj = g_rule<RULE>(r1, l1);
                    if constexpr (WEIGHTED) {
                        float wi, wj;
                        if constexpr (WSTAGE) {
                            wi = wj = Wit[0 * n + s];  // uniform: one scalar load
                        } else {
                            const float* w = Wit + (size_t)(0 * n + s) * N + ib;
                            wi = w[v << G::wbase(k)];
                            wj = w[v2 << G::wbase(k)];
                        }
                        Rm[s + 1][v] = clipf(wi * gi, lmax);
                        Rm[s + 1][v2] = clipf(__fmaf_rn(wj, gj, r2), lmax);
                        if constexpr (SAVE) {
                            float* sv = Sit + (size_t)(0 * n + s) * N + ib;
                            sv[v << G::wbase(k)] = Rm[s + 1][v];
                            sv[v2 << G::wbase(k)] = Rm[s + 1][v2];
                        }
                    } else {
                        // min-sum: |g| <= |r1| <= lmax, so the clip is exact
                        Rm[s + 1][v] = RULE == 0 ? gi : clipf(gi, lmax);
                        Rm[s + 1][v2] = clipf(gj + r2, lmax);
                    }
                }
            });
            if constexpr (k < G::NWIN - 1) {
                transpose_row<G, k, k, k + 1, true>(Rm[G::cend(k)], tb, bfrom[k], bto[k]);
            }
        });
        if (stop != 2) {
            if constexpr (OWN) {
                uint64_t m[V];
#pragma unroll
                for (int v = 0; v < V; ++v) m[v] = __ballot((Lm[n][v] + Rm[n][v]) < 0.0f);
                if (t == 0) {  // (every frame still running writes the same)
                    uint64_t* xw = reinterpret_cast<uint64_t*>(sh.xbytes);
#pragma unroll
                    for (int v = 0; v < V; ++v) xw[v] = m[v];
                }
            } else if constexpr (BITPACK) {
                // thread t holds node t + (v << P): the wavefront's ballot for
                // register v is 64-bit word (v << (P - 6)) + w of the array
                uint64_t m[V];
#pragma unroll
                for (int v = 0; v < V; ++v) m[v] = __ballot((Lm[n][v] + Rm[n][v]) < 0.0f);
                if (lane == 0) {
                    uint64_t* xw = reinterpret_cast<uint64_t*>(xb) + (t >> 6);
#pragma unroll
                    for (int v = 0; v < V; ++v) xw[v << (G::P - 6)] = m[v];
                }
            } else {
                const int ib = idx_base<G, KL>(t);
#pragma unroll
                for (int v = 0; v < V; ++v) xb[ib + (v << G::wbase(KL))] = (Lm[n][v] + Rm[n][v]) < 0.0f ? 1 : 0;
            }
        }
        // ---------------- L sweep: columns n-1..0
        static_for_rev<0, G::NWIN>([&](auto KC) {
            constexpr int k = decltype(KC)::value;
            const int ib = idx_base<G, k>(t);
            static_for_rev<G::cbeg(k), G::cend(k)>([&](auto SC) {
                constexpr int s = decltype(SC)::value;
                constexpr int q = s - G::wbase(k);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (v & (1 << q)) continue;
                    const int v2 = v | (1 << q);
                    const float r1 = (s == 0) ? prior[v] : Rm[s][v];
                    const float r2 = (s == 0) ? prior[v2] : Rm[s][v2];
                    const float l1 = Lm[s + 1][v], l2 = Lm[s + 1][v2];
                    if constexpr (FAST) {
                        // both g terms share l1
                        const float x = l2 + r2;
                        if constexpr (WEIGHTED) {
                            float wi, wj;
                            if constexpr (WSTAGE) {
                                wi = wj = Wit[1 * n + s];
                            } else {
                                const float* w = Wit + (size_t)(1 * n + s) * N + ib;
                                wi = w[v << G::wbase(k)];
                                wj = w[v2 << G::wbase(k)];
                            }
                            const float si = sign_to(wi, l1);
                            const float sj = WSTAGE ? si : sign_to(wj, l1);
                            const float yi = si * clamp_mag(x, l1);
                            Lm[s][v] = NOCLIP ? yi : clipf(yi, lmax);
                            Lm[s][v2] = clipf(__fmaf_rn(sj, clamp_mag(r1, l1), l2), lmax);
                        } else {
                            const float si = sign_to(1.0f, l1);
                            Lm[s][v] = si * clamp_mag(x, l1);  // |g| <= |l1| <= lmax
                            Lm[s][v2] = clipf(__fmaf_rn(si, clamp_mag(r1, l1), l2), lmax);
                        }
                        continue;
                    }
                    const float gi = g_rule<RULE>(l1, l2 + r2);
                    const float gj = g_rule<RULE>(r1, l1);
                    if constexpr (WEIGHTED) {
                        float wi, wj;
                        if constexpr (WSTAGE) {
                            wi = wj = Wit[1 * n + s];
                        } else {
                            const float* w = Wit + (size_t)(1 * n + s) * N + ib;
                            wi = w[v << G::wbase(k)];
                            wj = w[v2 << G::wbase(k)];
                        }
                        Lm[s][v] = clipf(wi * gi, lmax);
                        Lm[s][v2] = clipf(__fmaf_rn(wj, gj, l2), lmax);
                        if constexpr (SAVE) {
                            float* sv = Sit + (size_t)(1 * n + s) * N + ib;
                            sv[v << G::wbase(k)] = Lm[s][v];
                            sv[v2 << G::wbase(k)] = Lm[s][v2];
                        }
                    } else {
                        Lm[s][v] = RULE == 0 ? gi : clipf(gi, lmax);  // min-sum: |g| <= |l1| <= lmax
                        Lm[s][v2] = clipf(gj + l2, lmax);
                    }
                }
            });
            if constexpr (k > 0) {
                transpose_row<G, k - 1, k, k - 1, false>(Lm[G::cbeg(k)], tb, bto[k - 1], bfrom[k - 1]);
            }
        });
        // ---------------- decisions in window 0 (register bits are the low bits)
        if constexpr (BITPACK || OWN) {
            // nodes 8t .. 8t + 7: byte t of the bit array.  LLR(u) = L + prior
            // is never -0 (the prior is +0 or lmax > 0, and a sum of zeros of
            // opposite signs rounds to +0), so its sign bit is the test
            // LLR(u) < 0; each bit is shifted in from the sign (one funnel
            // shift), frozen nodes are cleared after
            ubits = 0;
#pragma unroll
            for (int v = V - 1; v >= 0; --v)
                ubits = __builtin_amdgcn_alignbit(ubits, __float_as_uint(Lm[0][v] + prior[v]), 31);
            ubits &= ~fmask;
            // the CRC stop tests every thread's own bits and stores them once,
            // after the loop
            if (BITPACK && stop != 2) ub[t] = (uint8_t)ubits;
        } else {
            uint64_t pack = 0;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float lu = Lm[0][v] + prior[v];
                const uint64_t bit = (((fmask >> v) & 1u) == 0 && lu < 0.0f) ? 1ull : 0ull;
                pack |= bit << (8 * v);
            }
            uint8_t* dst = ub + idx_base<G, 0>(t);
            if constexpr (V == 8) {
                *reinterpret_cast<uint64_t*>(dst) = pack;
            } else if constexpr (V == 4) {
                *reinterpret_cast<uint32_t*>(dst) = (uint32_t)pack;
            } else if constexpr (V == 2) {
                *reinterpret_cast<uint16_t*>(dst) = (uint16_t)pack;
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v) dst[v] = (uint8_t)(pack >> (8 * v));
            }
        }
        ++it;
        const bool last = it >= max_iter;
        if constexpr (OWN) {
            if (stop == 1 || (stop == 0 && last)) {
                frame_sync<G>();
                gok = reencode_words<G>(ubits, own_x_bits<G>(reinterpret_cast<const uint64_t*>(sh.xbytes), t, slot), lane);
                if (gok || last) {
                    cok = own_crc<G>(code, ubits, t);
                    break;
                }
            } else if (stop == 2) {
                cok = own_crc<G>(code, ubits, t);
                if (cok || last) break;
            }
        } else if (stop == 1) {
            frame_sync<G>();
            gok = reencode_check<G, BITPACK>(ub, xb, lane);
            if (gok || last) {
                cok = crc_check<G, BITPACK>(code, ub, lane);
                break;
            }
        } else if (stop == 2) {
            if constexpr (BITPACK) {
                cok = crc_check_own<G>(code, ubits, t, sh.syn[it & 1]);
            } else {
                frame_sync<G>();
                cok = crc_check<G, BITPACK>(code, ub, lane);
            }
            if (cok || last) break;
        } else if (last) {
            frame_sync<G>();
            gok = reencode_check<G, BITPACK>(ub, xb, lane);
            cok = crc_check<G, BITPACK>(code, ub, lane);
            break;
        }
    }

    // ---------------- outputs (window 0 layout: V consecutive nodes per thread)
    const bool okv = stop == 2 ? cok : (gok && cok);
    {
        const int ib = idx_base<G, 0>(t);
        if (io.u_hat) {
            uint8_t* uo = io.u_hat + ib;
            if constexpr (BITPACK) {
                // ubits: the last iteration's decisions
                uint64_t bytes = 0;
#pragma unroll
                for (int v = 0; v < V; ++v) bytes |= (uint64_t)((ubits >> v) & 1u) << (8 * v);
                *reinterpret_cast<uint64_t*>(uo) = bytes;
            } else if constexpr (OWN) {
#pragma unroll
                for (int v = 0; v < V; ++v) uo[v] = (uint8_t)((ubits >> v) & 1u);
            } else {
                const uint8_t* src = ub + ib;
#pragma unroll
                for (int v = 0; v < V; ++v) uo[v] = src[v];
            }
        }
        if (io.llr_u) {
            float* lo = io.llr_u + ib;
#pragma unroll
            // row 0 still holds the last iteration's L messages (the loop
            // leaves right after the decisions that read it)
            for (int v = 0; v < V; ++v) lo[v] = Lm[0][v] + prior[v];
        }
        if constexpr (OWN) {
            if (io.info && okv) {
                ub[t] = (uint8_t)ubits;  // V bits a byte
                frame_sync<G>();
            }
        }
        if constexpr (BITPACK) {
            if (stop == 2 && io.info && okv) {
                // the CRC stop left the bits in registers (frame-uniform branch)
                ub[t] = (uint8_t)ubits;
                frame_sync<G>();
            }
        }
        if (io.info && okv) {
            // the hybrid keeps BP's result: its information bits go out here
            for (int q = t; q < code.K; q += G::T) {
                const int pos = code.info_pos[q];
                io.info[q] = BITPACK ? (uint8_t)((ub[pos >> 3] >> (pos & 7)) & 1u)
                             : OWN   ? (uint8_t)((ub[pos / V] >> (pos % V)) & 1u)
                                     : ub[pos];
            }
        }
        if (t == 0) {
            if (io.iters) *io.iters = it;
            if (io.ok) *io.ok = (uint8_t)okv;
        }
    }
    return okv;
}

// PERSIST: a grid smaller than the batch walks it (frame slots advance by the
// grid size), so a capped grid leaves room on every CU for other kernels.
// DENSE (N >= 1024, eight nodes per thread, no weight per node, which needs
// more registers): held to 128 VGPRs (from 126 to 162), so that four waves share
// a SIMD instead of three, at N = 4096 two frames a CU instead of one; what the
// kernel spills (0 to 80 bytes per lane) is read outside the iteration loop or
// once per iteration.  Plain BP, re-encoding stop: N = 1024, 65536 frames
// 2509 -> 2402 us, N = 4096, 4096 frames 4619 -> 3689 us; exact rule, N = 4096:
// 5788 -> 5177 us.  For batches that fill the chip (dense_batch below).
template <int NLOG, int RLOG, bool WEIGHTED, bool SAVE, int RULE = 0, bool WSTAGE = false, bool PERSIST = false,
          bool DENSE = false>
__global__ __launch_bounds__((Geom<NLOG, RLOG>::WG))
__attribute__((amdgpu_waves_per_eu(DENSE ? 4 : 1))) void bp_kernel(
    CodeDev code, const float* __restrict__ llr, int64_t B, int max_iter, int stop, float lmax,
    const float* __restrict__ W, uint8_t* __restrict__ u_hat, uint8_t* __restrict__ info_out,
    float* __restrict__ llr_u, int32_t* __restrict__ iters_out, uint8_t* __restrict__ ok_out,
    float* __restrict__ saved, BpQueue queue, int grid) {
    using G = Geom<NLOG, RLOG>;
    constexpr int N = G::N;
    __shared__ BpShared<G> sh;
    const int tid = lid_x();
    const int t = (G::T < 64) ? (tid & (G::T - 1)) : tid;
    const int slot = (G::T < 64) ? (tid >> G::P) : 0;
    const int64_t stride = PERSIST ? (int64_t)grid * G::FPW : 0;
    // per-stage weights all within [-1, 1]: the clip-free form applies (every
    // wavefront reads the max_iter * 2n weights, which sit in the caches)
    bool unit = false;
    if constexpr (WEIGHTED && WSTAGE && RULE == 0 && !SAVE) {
        float m = 0.0f;
        for (int i = tid & 63; i < max_iter * 2 * G::n; i += 64) m = fmaxf(m, fabsf(W[i]));
        unit = wave_max(m) <= 1.0f;
    }
    for (int64_t f0 = gid_x() * G::FPW; f0 < B; f0 += stride) {
        const int64_t frame = f0 + slot;
        if (PERSIST && G::T >= 64 && f0 != gid_x() * G::FPW) __syncthreads();  // staging reuse
        if (G::T < 64 && frame >= B) return;  // lone wavefront: no barriers to honour
        FrameIO io;
        io.llr = llr + frame * N;
        io.u_hat = u_hat ? u_hat + frame * N : nullptr;
        io.info = info_out ? info_out + frame * code.K : nullptr;
        io.llr_u = llr_u ? llr_u + frame * N : nullptr;
        io.iters = iters_out ? iters_out + frame : nullptr;
        io.ok = ok_out ? ok_out + frame : nullptr;
        io.saved = SAVE ? saved + (size_t)frame * max_iter * 2 * G::n * N : nullptr;
        bool okv;
        if constexpr (WEIGHTED && WSTAGE && RULE == 0 && !SAVE) {
            if (unit) okv = bp_frame<G, true, false, 0, true, true>(code, io, max_iter, stop, lmax, W, sh, t, slot);
            else okv = bp_frame<G, true, false, 0, true, false>(code, io, max_iter, stop, lmax, W, sh, t, slot);
        } else {
            okv = bp_frame<G, WEIGHTED, SAVE, RULE, WSTAGE>(code, io, max_iter, stop, lmax, W, sh, t, slot);
        }
        if (!SAVE && queue.ids && t == 0) {
            if (queue.used_scl) queue.used_scl[frame] = okv ? 0 : 1;
            if (!okv) queue.ids[atomicAdd(queue.count, 1)] = (int32_t)frame;
        }
        if (!PERSIST) break;
    }
}

// Persistent form for ragged batches: workgroups walk the list ids[0..*count)
// (the count lives on the device), each taking its first frames by its number
// and the next ones as it gets there (a frame runs 5 iterations or 200, and a
// fixed share of the list kept some workgroups busy with two long frames after
// the others had ended); frame id's LLR row starts at element
// io->off[id] of io->llr, its information bits go to io->info + io->out_off[id];
// iters and ok are indexed by id; failed frames are appended to their code's queue (one atomic
// each).
// Frame id uses the code io->codes[io->code_of[id]] (all of the kernel's block
// length).
// The unweighted gather kernels from N = 512 on are held to four waves per SIMD
// too: their failing frames run every iteration, so more frames in flight
// shorten the mixed batch's longest chain (twelve codes, 4096 frames: 2692 ->
// 2498 us).
template <int NLOG, int RLOG, bool WEIGHTED>
constexpr int gather_waves_per_eu() { return (NLOG >= 9 && RLOG == 3 && !WEIGHTED) ? 4 : 1; }

template <int NLOG, int RLOG, bool WEIGHTED>
__global__ __launch_bounds__((Geom<NLOG, RLOG>::WG))
__attribute__((amdgpu_waves_per_eu(gather_waves_per_eu<NLOG, RLOG, WEIGHTED>()))) void bp_gather_kernel(
    const MixedIo* __restrict__ mio, const int32_t* __restrict__ ids, const int32_t* __restrict__ count,
    int32_t* __restrict__ ticket, int max_iter, int stop, float lmax, const float* __restrict__ W,
    int32_t* __restrict__ iters_out, uint8_t* __restrict__ ok_out, int32_t* __restrict__ fail_ids,
    int64_t fail_stride, int32_t* __restrict__ fail_count, int grid) {
    using G = Geom<NLOG, RLOG>;
    __shared__ BpShared<G> sh;
    const int tid = lid_x();
    const int t = (G::T < 64) ? (tid & (G::T - 1)) : tid;
    const int slot = (G::T < 64) ? (tid >> G::P) : 0;
    const int64_t cnt = *count;
    const float* llr = mio->llr;
    const int64_t* off = mio->off;
    __shared__ int next_first;
    for (int64_t q0 = gid_x() * G::FPW; q0 < cnt;) {
        const int64_t q = q0 + slot;
        if (G::T >= 64) __syncthreads();  // the previous frame's staging and next_first are read
        int ticket_now = 0;
        if (tid == 0) ticket_now = atomicAdd(ticket, G::FPW);  // not waited for before the frame is decoded
        if (q >= cnt) break;             // only when T < 64: this slot's wavefront lanes leave alone
        const int id = ids[q];
        const int cid = mio->code_of[id];
        const CodeDev cd = mio->codes[cid];
        FrameIO io;
        io.llr = llr + off[id];
        io.u_hat = nullptr;
        io.info = mio->info + mio->out_off[id];
        io.llr_u = nullptr;
        io.iters = iters_out + id;
        io.ok = ok_out + id;
        io.saved = nullptr;
        const bool okv = bp_frame<G, WEIGHTED, false>(cd, io, max_iter, stop, lmax, W, sh, t, slot);
        if (t == 0 && !okv) fail_ids[cid * fail_stride + atomicAdd(&fail_count[cid], 1)] = id;
        if (tid == 0) next_first = ticket_now;
        frame_sync<G>();
        q0 = (int64_t)grid * G::FPW + next_first;
    }
}

// ------------------------------------------------------------------ dispatch

using KernelFn = void (*)(CodeDev, const float*, int64_t, int, int, float, const float*, uint8_t*, uint8_t*,
                          float*, int32_t*, uint8_t*, float*, BpQueue, int);

using GatherFn = void (*)(const MixedIo*, const int32_t*, const int32_t*, int32_t*, int, int, float, const float*,
                          int32_t*, uint8_t*, int32_t*, int64_t, int32_t*, int);

struct Entry {
    KernelFn plain, weighted, weighted_save, exact, weighted_stage;
    KernelFn dense_plain, dense_exact, dense_weighted_stage;  // or the ones above
    KernelFn persist_plain, persist_weighted_stage;
    GatherFn gather_plain, gather_weighted;
    int wg, fpw;
};

template <int NL, int RL>
constexpr Entry make_entry() {
    constexpr bool D = NL >= 10 && RL == 3;
    return Entry{&bp_kernel<NL, RL, false, false>, &bp_kernel<NL, RL, true, false>, &bp_kernel<NL, RL, true, true>,
                 &bp_kernel<NL, RL, false, false, 1>, &bp_kernel<NL, RL, true, false, 0, true>,
                 &bp_kernel<NL, RL, false, false, 0, false, false, D>, &bp_kernel<NL, RL, false, false, 1, false, false, D>,
                 &bp_kernel<NL, RL, true, false, 0, true, false, D>,
                 &bp_kernel<NL, RL, false, false, 0, false, true>, &bp_kernel<NL, RL, true, false, 0, true, true>,
                 &bp_gather_kernel<NL, RL, false>, &bp_gather_kernel<NL, RL, true>, Geom<NL, RL>::WG,
                 Geom<NL, RL>::FPW};
}

// variants: register bits r = 2 or 3 (variant id = r)
constexpr int kMinN = 3, kMaxN = 12;

const Entry* lookup(int n, int r) {
    static const Entry table[kMaxN + 1][4] = {
        {},
        {},
        {},
        {{}, {}, make_entry<3, 2>(), make_entry<3, 3>()},
        {{}, {}, make_entry<4, 2>(), make_entry<4, 3>()},
        {{}, {}, make_entry<5, 2>(), make_entry<5, 3>()},
        {{}, {}, make_entry<6, 2>(), make_entry<6, 3>()},
        {{}, {}, make_entry<7, 2>(), make_entry<7, 3>()},
        {{}, {}, make_entry<8, 2>(), make_entry<8, 3>()},
        {{}, {}, make_entry<9, 2>(), make_entry<9, 3>()},
        {{}, {}, make_entry<10, 2>(), make_entry<10, 3>()},
        {{}, {}, make_entry<11, 2>(), make_entry<11, 3>()},
        {{}, {}, make_entry<12, 2>(), make_entry<12, 3>()},
    };
    if (n < kMinN || n > kMaxN || r < 2 || r > 3) return nullptr;
    return &table[n][r];
}

}  // namespace bp

bool bp_variant_supported(int n, int variant) { return bp::lookup(n, variant) != nullptr; }

int bp_default_variant(int n) { return n >= 9 ? 3 : 2; }

// The default layout of a batch.  Eight nodes per thread (r = 3) issue fewer
// instructions per frame; four (r = 2) spread a frame over twice the threads,
// which ends its iterations sooner as long as the chip holds all frames at once:
// N = 1024 up to three frames per CU (256 frames, at most 100 iterations: 160
// against 202 us; 768: 213 against 230; 8192: 674 both; 65536: 4253 against
// 4040), N = 2048 one (256: 133 against 135 us, with weights 48 against 52; 512:
// 185 against 156) unless the CRC stops it, whose test costs r = 2 an LDS round
// trip more (256: 181 against 137 us, with weights 63 against 51); never at N =
// 4096 (16 frames: 376 against 339 us).  With a weight per node the
// registers r = 3 holds weights in cost it wavefronts: N = 512 is faster with
// r = 2 at every size (16 frames 25 against 42 us, 65536: 699 against 876) and
// so is N = 4096 (768: 227 against 566 us), N = 1024 and, without the CRC stop,
// 2048 up to three frames per CU (768: 38 against 40, 77 against 87 us; with it
// N = 2048 takes 111 against 87).
static int bp_auto_variant(int n, int64_t B, const bp_params* p) {
    const int64_t cus = device_cu_count();
    if (p->rule == 0 && p->weights && p->weight_layout == 0) {
        if (n == 9 || n == 12) return 2;
        if ((n == 10 || (n == 11 && p->stop != 2)) && B <= 3 * cus) return 2;
    } else if (p->rule == 0) {
        if ((n == 10 && B <= 3 * cus) || (n == 11 && B <= cus && p->stop != 2)) return 2;
    }
    return bp_default_variant(n);
}

// Batches that the DENSE kernels serve: those that do not fit the chip at once
// with the registers the other kernels take -- more than three frames a CU at N =
// 2048, one at N = 4096.  Below, the spills only make every iteration longer (N =
// 4096, 256 frames of at most 60 iterations, re-encoding stop: 212 us DENSE, 181
// us not; N = 2048, 768 frames: 215 and 204); beyond, the frames in flight count
// (300 frames: 309 and 353 us; 1024: 264 and 290; at 3 dB, where a few frames
// run long after the others, the shorter iteration still wins up to 700 frames
// of N = 4096, 193 and 157 us).  At N = 1024 it is six a CU with weights (1536
// frames: 72 and 64 us; 2000: 88 and 106) or without an early stop (2000: 87 and
// 103), eight otherwise (2048: 231 and 218 us; 2600: 259 and 265; 16384: 1064
// and 1130).
static bool dense_batch(int n, int64_t B, const bp_params* p) {
    const int64_t per_cu = n == 10 ? (p->weights || p->stop == 0 ? 6 : 8) : n == 11 ? 3 : 1;
    return n >= 10 && B > per_cu * device_cu_count();
}

int bp_list_variants(int n, int32_t* ids, int cap) {
    int c = 0;
    for (int r = 2; r <= 3; ++r)
        if (bp::lookup(n, r)) {
            if (ids && c < cap) ids[c] = r;
            ++c;
        }
    return c;
}

polar_status launch_bp(const polar_code* code, const float* llr, int64_t B, const bp_params* p, uint8_t* u_hat,
                       float* llr_u, int32_t* iters, uint8_t* ok, hipStream_t stream, int wgs_per_cu,
                       uint8_t* info_out, BpQueue queue) {
    const int variant = p->variant ? p->variant : bp_auto_variant(code->n, B, p);
    const bp::Entry* e = bp::lookup(code->n, variant);
    if (!e) return set_error(POLAR_ERR_UNSUPPORTED, "bp: no kernel variant for this block length");
    if (B == 0) return POLAR_OK;
    const int64_t blocks = (B + e->fpw - 1) / e->fpw;
    if (blocks > (int64_t)INT32_MAX) return set_error(POLAR_ERR_INVALID_ARG, "bp: batch too large");
    const bool dense = dense_batch(code->n, B, p);
    bp::KernelFn fn = p->rule == 1       ? (dense ? e->dense_exact : e->exact)
                      : !p->weights      ? (dense ? e->dense_plain : e->plain)
                      : p->weight_layout ? (dense ? e->dense_weighted_stage : e->weighted_stage)
                                         : e->weighted;
    int64_t grid = blocks;
    if (wgs_per_cu > 0 && p->rule == 0 && (!p->weights || p->weight_layout == 1)) {
        // capped persistent grid: leaves room on every CU for concurrent kernels
        const int64_t cap = (int64_t)device_cu_count() * wgs_per_cu;
        if (cap < blocks) {
            fn = p->weights ? e->persist_weighted_stage : e->persist_plain;
            grid = cap;
        }
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(e->wg), 0, stream, code->dev(), llr, B, p->max_iter, p->stop,
                       p->llr_max, p->weights, u_hat, info_out, llr_u, iters, ok, (float*)nullptr, queue, (int)grid);
    return hip_check(hipGetLastError(), "bp_kernel launch");
}

polar_status bp_gather_grid(const polar_code* code, const bp_params* p, int64_t max_frames, int* grid) {
    const int variant = p->variant ? p->variant : bp_default_variant(code->n);
    const bp::Entry* e = bp::lookup(code->n, variant);
    if (!e) return set_error(POLAR_ERR_UNSUPPORTED, "bp: no kernel variant for this block length");
    bp::GatherFn fn = p->weights ? e->gather_weighted : e->gather_plain;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, e->wg, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    int64_t g = (int64_t)device_cu_count() * per_cu;
    const int64_t need = (max_frames + e->fpw - 1) / e->fpw;
    if (need < g) g = need;
    *grid = (int)(g < 1 ? 1 : g);
    return POLAR_OK;
}

polar_status launch_bp_gather(const polar_code* code, const MixedIo* io, const int32_t* ids, const int32_t* count,
                              int32_t* ticket, const bp_params* p, int32_t* iters, uint8_t* ok, int32_t* fail_ids,
                              int64_t fail_stride, int32_t* fail_count, int grid, hipStream_t stream) {
    const int variant = p->variant ? p->variant : bp_default_variant(code->n);
    const bp::Entry* e = bp::lookup(code->n, variant);
    if (!e) return set_error(POLAR_ERR_UNSUPPORTED, "bp: no kernel variant for this block length");
    bp::GatherFn fn = p->weights ? e->gather_weighted : e->gather_plain;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(e->wg), 0, stream, io, ids, count, ticket, p->max_iter,
                       p->stop, p->llr_max, p->weights, iters, ok, fail_ids, fail_stride, fail_count, grid);
    return hip_check(hipGetLastError(), "bp_gather_kernel launch");
}

polar_status launch_bp_save(const polar_code* code, const float* llr, int64_t B, int T, float llr_max,
                            const float* W, int variant, uint8_t* u_hat, float* llr_u, uint8_t* ok, float* saved,
                            hipStream_t stream) {
    // with the messages saved the pass is bound by its stores, and up to
    // N = 1024 r = 2, with more wavefronts in flight, issues them faster (saved
    // messages of 755 MB at N = 512: 207 against 285 us; 1.7 GB at N = 1024: 473
    // against 495; 923 MB at N = 2048: 365 against 262)
    const int v = variant ? variant : (saved && code->n <= 10) ? 2 : bp_default_variant(code->n);
    const bp::Entry* e = bp::lookup(code->n, v);
    if (!e) return set_error(POLAR_ERR_UNSUPPORTED, "wbp: no kernel variant for this block length");
    if (B == 0) return POLAR_OK;
    const int64_t blocks = (B + e->fpw - 1) / e->fpw;
    bp::KernelFn fn = saved ? e->weighted_save : e->weighted;
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(e->wg), 0, stream, code->dev(), llr, B, T, 0, llr_max, W,
                       u_hat, (uint8_t*)nullptr, llr_u, (int32_t*)nullptr, ok, saved, BpQueue(), (int)blocks);
    return hip_check(hipGetLastError(), "bp_kernel launch");
}

}  // namespace polarhip

using namespace polarhip;

extern "C" polar_status polar_bp_variants(int32_t N, int32_t* ids, int32_t cap, int32_t* count) {
    if (!count || cap < 0) return set_error(POLAR_ERR_INVALID_ARG, "polar_bp_variants: bad argument");
    int n = 0;
    while ((1 << n) < N) ++n;
    if ((1 << n) != N) return set_error(POLAR_ERR_INVALID_ARG, "polar_bp_variants: N not a power of two");
    *count = bp_list_variants(n, ids, cap);
    return ok_status();
}

extern "C" polar_status bp_decode_batch(const polar_code* code, const float* llr, int64_t B, const bp_params* p,
                                        uint8_t* u_hat, float* llr_u, int32_t* iters, uint8_t* ok,
                                        hipStream_t stream) {
    if (!code || !p) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: null code or params");
    if (B < 0) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: negative batch");
    if (B > 0 && (!llr || !u_hat || !ok)) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: null buffer");
    if (p->max_iter < 1) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: max_iter must be >= 1");
    if (p->stop < 0 || p->stop > 2) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: stop must be 0, 1 or 2");
    if (p->stop == 2 && code->c == 0)
        return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: CRC stop needs a code with a CRC");
    if (!(p->llr_max > 0.0f)) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: llr_max must be > 0");
    if (p->rule != 0 && p->rule != 1) return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: rule must be 0 or 1");
    if (p->rule == 1 && p->weights)
        return set_error(POLAR_ERR_UNSUPPORTED, "bp_decode_batch: the exact rule has no weighted form");
    if (p->weights && p->weight_iters < p->max_iter)
        return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: weight_iters < max_iter");
    if (p->weight_layout != 0 && p->weight_layout != 1)
        return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: weight_layout must be 0 or 1");
    if (p->variant != 0 && !bp_variant_supported(code->n, p->variant))
        return set_error(POLAR_ERR_INVALID_ARG, "bp_decode_batch: unknown variant");
    polar_status st = launch_bp(code, llr, B, p, u_hat, llr_u, iters, ok, stream);
    return st == POLAR_OK ? ok_status() : st;
}
