// wbp.hip -- weighted (learned) min-sum BP: loss, hand-written adjoint, weight
// gradient reduction and Adam.
//
// Forward: bp_kernel with weights and message saving (bp.hip): T iterations,
// no early stop, every produced row saved as saved[f][t][dir][s][node].
// Losses: binary cross-entropy of P(u_i = 1) = sigmoid(-lambda_i) over the
// non-frozen positions after the last iteration (or after every iteration),
// lambda = L_{i,1} + R_{i,1}; or the frame-failure surrogate, the probability
// (bits independent) that no iteration decides the whole frame right.
// Adjoint (reverse mode, by hand): iterations T..1; inside one, the L sweep is
// undone first (columns 0..n-1), then the R sweep (columns n-1..0), in the
// same register windows as the forward: adjoint rows cross window boundaries
// through the same LDS maps in the opposite direction.  Derivative rules:
// d clip(p)/dp = [|p| <= llr_max]; g(a,b) = a sgn(b) when |a| <= |b| (ties to
// a), else b sgn(a); the sign factor has zero derivative.  Every operation
// follows the CPU oracle's order, so a frame's gradient is bit-exact with the
// oracle's float build.  The per-frame weight gradient is written over the
// saved messages it no longer needs, and reduced over frames in double
// precision, in an order fixed by the sizes (deterministic).
#include "bp_common.hpp"

namespace polarhip {
namespace bp {

__device__ __forceinline__ void g_partials(float a, float b, float& da, float& db) {
    const float sb = (__float_as_uint(b) & 0x80000000u) ? -1.0f : 1.0f;
    const float sa = (__float_as_uint(a) & 0x80000000u) ? -1.0f : 1.0f;
    if (fabsf(a) <= fabsf(b)) {
        da = sb;
        db = 0.0f;
    } else {
        da = 0.0f;
        db = sa;
    }
}

// Bound by HBM: every saved message read and its slot written once (the other
// reads of a row come soon after the first, from the caches).  N = 1024, T = 20,
// 1024 frames, 3.36 GB: 1275 us with each column's operands loaded when it is
// reached, 855 us with the next column's in flight (3.9 TB/s); N = 256, T = 10,
// 4096 frames, 1.34 GB: 441 and 324 us; with the sum over frames, and the
// frames of a group added before they are written (below), 1803 -> 1181 -> 798
// and 2088 -> 489 -> 227 us.
// FG > 1: a workgroup takes FG frames through the columns in step and adds their
// weight gradients, column by column, in frame order and double precision,
// before anything is written: the double goes over the slots of the group's
// first two frames (low word, high word; a last group of one frame keeps its
// float), so instead of FG floats written here and read by the sum over frames
// it is two.  The frames' values of a column meet in LDS, one barrier per column
// (two buffers in turn), thread (g, t) adding registers g, g + FG, ...
template <class G, int FG>
struct BwdGeom {
    static constexpr int WG = FG == 1 ? G::WG : FG * G::T;
    static constexpr int FPG = FG == 1 ? G::FPW : FG;                 // frames per workgroup
    static constexpr int TBS = G::T < 64 ? WG / 64 : WG / G::T;       // transpose buffers
    static constexpr int XCH = FG == 1 ? 1 : 2 * FG * G::N;           // words of the exchange
};

template <int NLOG, int RLOG, int FG>
__global__ __launch_bounds__((BwdGeom<Geom<NLOG, RLOG>, FG>::WG)) void wbp_bwd_kernel(
    CodeDev code, const float* __restrict__ llr, int64_t B, int T, float lmax, const float* __restrict__ W,
    float* __restrict__ saved, const float* __restrict__ dlam, int dlam_iters, float* __restrict__ dllr) {
    using G = Geom<NLOG, RLOG>;
    using BG = BwdGeom<G, FG>;
    constexpr int n = G::n, N = G::N, V = G::V, KL = G::NWIN - 1;
    __shared__ float tb_all[BG::TBS * G::TAB.words];
    __shared__ float xch[BG::XCH];

    const int tid = lid_x();
    const int t = tid & (G::T - 1);
    // frame of the workgroup (the same for a whole wavefront where it has one)
    const int gf = G::T >= 64 ? __builtin_amdgcn_readfirstlane(tid >> G::P) : tid >> G::P;
    const int slot = (G::T < 64) ? ((tid & 63) >> G::P) : 0;  // and of the wavefront
    float* const tb = tb_all + (G::T < 64 ? tid >> 6 : gf) * G::TAB.words;
    const int64_t first = gid_x() * BG::FPG;
    const bool valid = first + gf < B;
    if (FG == 1 && G::T < 64 && !valid) return;
    // a group's missing frames go along on the last one and add nothing
    const int64_t frame = valid ? first + gf : B - 1;
    const int group = (int)(B - first < FG ? B - first : FG);  // frames of this group

    int bfrom[G::NB > 0 ? G::NB : 1], bto[G::NB > 0 ? G::NB : 1];
    static_for<0, G::NB>([&](auto J) {
        constexpr int j = decltype(J)::value;
        bfrom[j] = lds_base<G, j, j>(t, slot);
        bto[j] = lds_base<G, j, j + 1>(t, slot);
    });

    float aL[n + 1][V];
    float aR[n + 1][V];
#pragma unroll
    for (int s = 0; s <= n; ++s)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            aL[s][v] = 0.0f;
            aR[s][v] = 0.0f;
        }
    float prior[V], chanc[V], chraw[V];
    {
        const int ib = idx_base<G, 0>(t);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int i = ib + v;
            prior[v] = ((code.frozen_bits[i >> 5] >> (i & 31)) & 1u) ? lmax : 0.0f;
        }
    }
    {
        const int ib = idx_base<G, KL>(t);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            chraw[v] = llr[frame * N + ib + (v << G::wbase(KL))];
            chanc[v] = clipf(chraw[v], lmax);
        }
    }
    float* S = saved + (size_t)frame * T * 2 * n * N;

    // Operands of the next column, loaded before the present one is worked
    // on: a column's loads may not pass the stores of the one before it (one
    // buffer), so without this a wavefront waits for memory once per column.
    // x: L row s + 1 (of iteration it for the L sweep, it - 1 for the R sweep),
    // y: R row s, w: the column's weights, all in the layout of its window.
    float nx[V], ny[V], nw[V];
    auto fetch = [&](auto DC, auto SC, int it) {
        constexpr int dir = decltype(DC)::value, s = decltype(SC)::value;
        constexpr int k = s / G::r;
        int to = t;
        if constexpr (FG > 1) asm volatile("" : "+v"(to));
        const int ib = idx_base<G, k>(to);
        const float* Sy = S + (size_t)it * 2 * n * N;
        const int lt = dir == 1 ? it : it - 1;
        const float* Sx = S + (size_t)(lt > 0 ? lt : 0) * 2 * n * N;
        const float* Wc = W + (size_t)(it * 2 + dir) * n * N;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int off = ib + (v << G::wbase(k));
            if constexpr (s + 1 < n) nx[v] = Sx[(size_t)(1 * n + s + 1) * N + off];
            if constexpr (s > 0) ny[v] = Sy[(size_t)(0 * n + s - 1) * N + off];
            nw[v] = Wc[(size_t)s * N + off];
        }
    };
    fetch(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{}, T - 1);
    // the weight gradient of column s, direction dir, over the messages it no
    // longer needs
    auto put_gradient = [&](auto DC, auto SC, int it, const float (&dWv)[V]) {
        constexpr int dir = decltype(DC)::value, s = decltype(SC)::value;
        constexpr int wb = G::wbase(s / G::r);
        const size_t row = ((size_t)it * 2 + dir) * n * N + (size_t)s * N;
        if constexpr (FG == 1) {
            const int ib = idx_base<G, s / G::r>(t);
#pragma unroll
            for (int v = 0; v < V; ++v) S[row + ib + (v << wb)] = dWv[v];
        } else {
            // the thread index made opaque here, so that the addresses of all
            // columns are not computed ahead and held in registers
            int to = t;
            asm volatile("" : "+v"(to));
            const int ib = idx_base<G, s / G::r>(to);
            constexpr int buf = (dir == 1 ? s : s + 1) & 1;  // columns alternate: L 0 .. n - 1, R n - 1 .. 0
            float* xb = xch + buf * FG * N;
#pragma unroll
            for (int v = 0; v < V; ++v) xb[gf * N + v * G::T + to] = valid ? dWv[v] : 0.0f;
            __syncthreads();
            float* const S0 = saved + (size_t)first * T * 2 * n * N + row;
            float* const S1 = S0 + (size_t)T * 2 * n * N;
#pragma unroll
            for (int q = 0; q < (V + FG - 1) / FG; ++q) {
                const int v = gf + q * FG;
                if (v < V) {
                    double acc = 0.0;
#pragma unroll
                    for (int g = 0; g < FG; ++g) acc += (double)xb[g * N + v * G::T + to];
                    const uint64_t w = (uint64_t)__double_as_longlong(acc);
                    const int off = ib + (v << wb);
                    S0[off] = group > 1 ? __uint_as_float((uint32_t)w) : (float)acc;
                    if (group > 1) S1[off] = __uint_as_float((uint32_t)(w >> 32));
                }
            }
        }
    };

    for (int itc = T - 1; itc >= 0; --itc) {
        // the iteration made opaque, so that the loop carries one counter and
        // not an address for every row
        int it = itc;
        asm volatile("" : "+s"(it));
        // the loss reads LLR(u) after this iteration (every iteration, or only
        // the last); row 0 of L feeds nothing else, so its adjoint is d loss / d lambda
        if (dlam_iters == T || it == T - 1) {
            const int ib = idx_base<G, 0>(t);
            const float* dl = dlam + ((size_t)frame * dlam_iters + (dlam_iters == T ? it : 0)) * N;
#pragma unroll
            for (int v = 0; v < V; ++v) aL[0][v] = dl[ib + v];
        }
        // ---------------- undo the L sweep: columns 0..n-1
        static_for<0, G::NWIN>([&](auto KC) {
            constexpr int k = decltype(KC)::value;
            if constexpr (k > 0) {
                transpose_row<G, k - 1, k - 1, k, false>(aL[G::cbeg(k)], tb, bfrom[k - 1], bto[k - 1]);
            }
            static_for<G::cbeg(k), G::cend(k)>([&](auto SC) {
                constexpr int s = decltype(SC)::value;
                constexpr int q = s - G::wbase(k);
                float A[V], Rr[V], Wr[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    A[v] = (s + 1 == n) ? chanc[v] : nx[v];
                    Rr[v] = (s == 0) ? prior[v] : ny[v];
                    Wr[v] = nw[v];
                }
                if constexpr (s + 1 < n) fetch(std::integral_constant<int, 1>{}, std::integral_constant<int, s + 1>{}, it);
                else fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, n - 1>{}, it);
                float dWv[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (v & (1 << q)) continue;
                    const int v2 = v | (1 << q);
                    const float a1 = A[v], a2 = A[v2], r1 = Rr[v], r2 = Rr[v2];
                    const float wi = Wr[v], wj = Wr[v2];
                    const float bi = a2 + r2;
                    const float gi = g_ms(a1, bi), gj = g_ms(r1, a1);
                    const float pi = wi * gi, pj = __fmaf_rn(wj, gj, a2);
                    const float di = (fabsf(pi) <= lmax) ? aL[s][v] : 0.0f;
                    const float dj = (fabsf(pj) <= lmax) ? aL[s][v2] : 0.0f;
                    aL[s][v] = 0.0f;
                    aL[s][v2] = 0.0f;
                    dWv[v] = di * gi;
                    dWv[v2] = dj * gj;
                    float ga, gb;
                    g_partials(a1, bi, ga, gb);
                    const float ci = di * wi;
                    aL[s + 1][v] = aL[s + 1][v] + ci * ga;
                    aL[s + 1][v2] = aL[s + 1][v2] + ci * gb;
                    if (s > 0) aR[s][v2] = aR[s][v2] + ci * gb;
                    g_partials(r1, a1, ga, gb);
                    const float cj = dj * wj;
                    if (s > 0) aR[s][v] = aR[s][v] + cj * ga;
                    aL[s + 1][v] = aL[s + 1][v] + cj * gb;
                    aL[s + 1][v2] = aL[s + 1][v2] + dj;
                }
                // L^t_s is no longer read: its slot takes the weight gradient
                put_gradient(std::integral_constant<int, 1>{}, SC, it, dWv);
            });
        });
        // ---------------- undo the R sweep: columns n-1..0
        static_for_rev<0, G::NWIN>([&](auto KC) {
            constexpr int k = decltype(KC)::value;
            if constexpr (k < G::NWIN - 1) {
                transpose_row<G, k, k + 1, k, true>(aR[G::cend(k)], tb, bto[k], bfrom[k]);
            }
            static_for_rev<G::cbeg(k), G::cend(k)>([&](auto SC) {
                constexpr int s = decltype(SC)::value;
                constexpr int q = s - G::wbase(k);
                float Lp[V], Rr[V], Wr[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    Rr[v] = (s == 0) ? prior[v] : ny[v];
                    Lp[v] = (s + 1 == n) ? chanc[v] : (it == 0 ? 0.0f : nx[v]);
                    Wr[v] = nw[v];
                }
                if constexpr (s > 0) fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, s - 1>{}, it);
                else fetch(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{}, it > 0 ? it - 1 : 0);
                float dWv[V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (v & (1 << q)) continue;
                    const int v2 = v | (1 << q);
                    const float r1 = Rr[v], r2 = Rr[v2], l1 = Lp[v], l2 = Lp[v2];
                    const float wi = Wr[v], wj = Wr[v2];
                    const float bi = l2 + r2;
                    const float gi = g_ms(r1, bi), gj = g_ms(r1, l1);
                    const float pi = wi * gi, pj = __fmaf_rn(wj, gj, r2);
                    const float di = (fabsf(pi) <= lmax) ? aR[s + 1][v] : 0.0f;
                    const float dj = (fabsf(pj) <= lmax) ? aR[s + 1][v2] : 0.0f;
                    aR[s + 1][v] = 0.0f;
                    aR[s + 1][v2] = 0.0f;
                    dWv[v] = di * gi;
                    dWv[v2] = dj * gj;
                    float ga, gb;
                    g_partials(r1, bi, ga, gb);
                    const float ci = di * wi;
                    if (s > 0) aR[s][v] = aR[s][v] + ci * ga;
                    aL[s + 1][v2] = aL[s + 1][v2] + ci * gb;
                    if (s > 0) aR[s][v2] = aR[s][v2] + ci * gb;
                    g_partials(r1, l1, ga, gb);
                    const float cj = dj * wj;
                    if (s > 0) aR[s][v] = aR[s][v] + cj * ga;
                    aL[s + 1][v] = aL[s + 1][v] + cj * gb;
                    if (s > 0) aR[s][v2] = aR[s][v2] + dj;
                }
                // R^t_{s+1} is no longer read: its slot takes the weight gradient
                put_gradient(std::integral_constant<int, 0>{}, SC, it, dWv);
            });
        });
    }
    if (dllr && valid) {
        const int ib = idx_base<G, KL>(t);
#pragma unroll
        for (int v = 0; v < V; ++v)
            dllr[frame * N + ib + (v << G::wbase(KL))] = (fabsf(chraw[v]) <= lmax) ? aL[n][v] : 0.0f;
    }
}

using BwdFn = void (*)(CodeDev, const float*, int64_t, int, float, const float*, float*, const float*, int, float*);

struct BwdEntry {
    BwdFn fn;
    int wg, fpw;
    // the grouped form (or null)
    BwdFn group_fn;
    int group_wg, group;
};

// Frames per group where the grouped form exists: N = 128 to 1024, in the layout
// of r that leaves room for at least four frames in a workgroup of 512 threads with
// its registers (N = 2048 and 4096 have no such layout; shorter blocks would, but
// were not measured)
template <int NL, int RL>
constexpr int bwd_group() {
    return (NL == 7 || NL == 8) && RL == 2 ? 8 : NL == 9 && RL == 3 ? 8 : NL == 10 && RL == 3 ? 4 : 1;
}

template <int NL, int RL>
constexpr BwdEntry make_bwd() {
    using G = Geom<NL, RL>;
    constexpr int FG = bwd_group<NL, RL>();
    return BwdEntry{&wbp_bwd_kernel<NL, RL, 1>, G::WG, G::FPW, FG > 1 ? &wbp_bwd_kernel<NL, RL, FG> : nullptr,
                    BwdGeom<G, FG>::WG, FG};
}

const BwdEntry* lookup_bwd(int n, int r) {
    static const BwdEntry table[13][4] = {
        {}, {}, {},
        {{}, {}, make_bwd<3, 2>(), make_bwd<3, 3>()},
        {{}, {}, make_bwd<4, 2>(), make_bwd<4, 3>()},
        {{}, {}, make_bwd<5, 2>(), make_bwd<5, 3>()},
        {{}, {}, make_bwd<6, 2>(), make_bwd<6, 3>()},
        {{}, {}, make_bwd<7, 2>(), make_bwd<7, 3>()},
        {{}, {}, make_bwd<8, 2>(), make_bwd<8, 3>()},
        {{}, {}, make_bwd<9, 2>(), make_bwd<9, 3>()},
        {{}, {}, make_bwd<10, 2>(), make_bwd<10, 3>()},
        {{}, {}, make_bwd<11, 2>(), make_bwd<11, 3>()},
        {{}, {}, make_bwd<12, 2>(), make_bwd<12, 3>()},
    };
    if (n < 3 || n > 12 || r < 2 || r > 3) return nullptr;
    return &table[n][r];
}

}  // namespace bp

namespace {

// Register layout of the adjoint (nodes per thread 2^r): r = 2 keeps more
// wavefronts in flight, which the adjoint, bound by its memory accesses, needs
// where frames are few (N = 1024, T = 20: 287 against 324 us for 200 frames,
// 1183 against 1176 us for 1024, with the sum over frames; N = 2048, T = 10,
// 512 frames: 637 against 669 us); at N = 4096 its 1024 threads per frame leave
// 128 registers and spill more than r = 3 (865 against 818 us for 256 frames).
int bwd_default_variant(int n) { return n <= 11 ? 2 : 3; }

// The grouped adjoint: its layout, and the batches it serves -- those whose
// groups fill enough of the places for them on the chip (workgroups of 256 or
// 512 threads: this many per CU by registers), over all rounds: half up to N =
// 512, where the adjoint and the sum over frames take less than half the time
// when all places are filled (4096 frames of N = 256, T = 10: 227 against 531
// us; 2048 of N = 512: 271 against 545), seven tenths at N = 1024 (1024 frames,
// T = 20: 798 against 1182 us); with fewer groups the frames one by one spread
// better.  All frames of a batch take one form, so a batch a little over whole
// rounds goes back to single frames (N = 1024, T = 5: 1024 frames 208 us, 1100 frames
// 346, 1500, whose groups fill seven tenths of two rounds again, 369).
int bwd_group_variant(int n) { return n <= 8 ? 2 : 3; }
bool bwd_grouped(int n, int64_t B) {
    if (n < 7 || n > 10) return false;
    const int64_t group = n == 10 ? 4 : 8, per_cu = n == 7 ? 3 : n == 8 ? 2 : 1;
    const int64_t groups = B / group, places = (int64_t)device_cu_count() * per_cu;
    const int64_t rounds = (groups + places - 1) / places;
    return groups > 0 && (n == 10 ? 10 * groups >= 7 * rounds * places : 2 * groups >= rounds * places);
}

// Sum of the per-frame gradients part[f][q] over the frames, in double.  One
// thread per VEC columns q would leave the chip idle (P / 256 workgroups, a
// serial chain of B loads each), so the frames are split into segments of
// equal length: workgroup (x, s) sums the rows of segment s in frame order and
// leaves the double in that segment's first two rows of its own columns (low
// word, high word -- entries that no other thread reads), and a second kernel
// adds the segments in order.  The order of additions depends on B, P and the
// number of CUs.  Bound by HBM: the B P floats are read once; the partial sums, two floats
// written and read again per segment and column, add at most an eighth with 32
// rows a segment, at most a quarter with eight grouped rows of two floats (below).
// Measured, ungrouped: T = 10, N = 256,
// B = 4096 (671 MB) 1647 us with one thread per column, 165 us; T = 20,
// N = 1024, B = 1024 (1.7 GB) 528 us, 326 us.
// Grouped rows (group > 1, the adjoint's sums over `group` frames): row g is
// the double in rows group g and group g + 1, the last a float where its group
// has one frame.
constexpr int kReduceUnroll = 8;
constexpr int64_t kReduceMinRows = 32;

template <int VEC>
struct alignas(4 * VEC) FloatVec {
    float v[VEC];
};

// VEC doubles kept as low and high words in two rows
template <int VEC>
__device__ __forceinline__ void load_pair(const float* lo, const float* hi, double (&d)[VEC]) {
    using Vec = FloatVec<VEC>;
    const Vec l = *reinterpret_cast<const Vec*>(lo), h = *reinterpret_cast<const Vec*>(hi);
#pragma unroll
    for (int j = 0; j < VEC; ++j)
        d[j] = __longlong_as_double((long long)(((uint64_t)__float_as_uint(h.v[j]) << 32) | __float_as_uint(l.v[j])));
}
template <int VEC>
__device__ __forceinline__ void store_pair(float* lo, float* hi, const double (&d)[VEC]) {
    using Vec = FloatVec<VEC>;
    Vec l, h;
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const uint64_t w = (uint64_t)__double_as_longlong(d[j]);
        l.v[j] = __uint_as_float((uint32_t)w);
        h.v[j] = __uint_as_float((uint32_t)(w >> 32));
    }
    *reinterpret_cast<Vec*>(lo) = l;
    *reinterpret_cast<Vec*>(hi) = h;
}
template <int VEC>
__device__ __forceinline__ void store_float(float* p, const double (&d)[VEC]) {
    FloatVec<VEC> o;
#pragma unroll
    for (int j = 0; j < VEC; ++j) o.v[j] = (float)d[j];
    *reinterpret_cast<FloatVec<VEC>*>(p) = o;
}

// rows: frames (group = 1) or groups of frames
template <int VEC, bool PARTIAL, bool GROUPED>
__global__ __launch_bounds__(256) void wbp_reduce_kernel(float* part, int64_t B, int group, int64_t P, int segments,
                                                         float* __restrict__ dW) {
    const int64_t q = (gid_x() * 256 + lid_x()) * VEC;
    if (q >= P) return;
    const int64_t rows = GROUPED ? (B + group - 1) / group : B;
    const int64_t s = PARTIAL ? gid_y() : 0;
    const int64_t r0 = PARTIAL ? rows * s / segments : 0, r1 = PARTIAL ? rows * (s + 1) / segments : rows;
    const int64_t stride = (GROUPED ? group : 1) * P;
    double acc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = 0.0;
    using Vec = FloatVec<VEC>;
    constexpr int U = GROUPED ? kReduceUnroll / 2 : kReduceUnroll;
    // the last group of a single frame is a float
    const int64_t pairs = GROUPED && r1 == rows && (B - 1) % group == 0 ? r1 - 1 : r1;
    int64_t f = r0;
    for (; f + U <= pairs; f += U) {
        double x[U][VEC];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const float* p = part + (f + k) * stride + q;
            if constexpr (GROUPED) {
                load_pair<VEC>(p, p + P, x[k]);
            } else {
                const Vec v = *reinterpret_cast<const Vec*>(p);
#pragma unroll
                for (int j = 0; j < VEC; ++j) x[k][j] = (double)v.v[j];
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] += x[k][j];
    }
    for (; f < r1; ++f) {
        const float* p = part + f * stride + q;
        if (GROUPED && f < pairs) {
            double x[VEC];
            load_pair<VEC>(p, p + P, x);
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] += x[j];
        } else {
            const Vec v = *reinterpret_cast<const Vec*>(p);
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] += (double)v.v[j];
        }
    }
    if constexpr (PARTIAL) store_pair<VEC>(part + r0 * stride + q, part + r0 * stride + P + q, acc);
    else store_float<VEC>(dW + q, acc);
}

template <int VEC>
__global__ __launch_bounds__(256) void wbp_reduce_segments_kernel(const float* __restrict__ part, int64_t rows,
                                                                  int64_t stride, int64_t P, int segments,
                                                                  float* __restrict__ dW) {
    const int64_t q = (gid_x() * 256 + lid_x()) * VEC;
    if (q >= P) return;
    double acc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = 0.0;
#pragma unroll 4
    for (int s = 0; s < segments; ++s) {
        const float* p = part + rows * s / segments * stride + q;
        double x[VEC];
        load_pair<VEC>(p, p + P, x);
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[j] += x[j];
    }
    store_float<VEC>(dW + q, acc);
}

// group: frames summed by the adjoint (1: none)
template <int VEC>
polar_status launch_reduce(float* part, int64_t B, int group, int64_t P, float* dW, hipStream_t stream) {
    const int64_t bx = (P / VEC + 255) / 256;
    const int64_t rows = (B + group - 1) / group;
    // about eight workgroups per CU (of four columns a thread, also where the
    // buffers' alignment allows one: it shall not change the order of the sum); a
    // segment's first row is never a last group of one frame, since it has more rows
    // than that
    int64_t segments = (int64_t)device_cu_count() * 8 / ((P / 4 + 255) / 256);
    const int64_t most = rows / (group > 1 ? kReduceMinRows / 4 : kReduceMinRows);
    if (segments > most) segments = most;
    const dim3 one((unsigned)bx), many((unsigned)bx, (unsigned)(segments > 1 ? segments : 1));
    if (segments > 1) {
        if (group > 1)
            hipLaunchKernelGGL((wbp_reduce_kernel<VEC, true, true>), many, dim3(256), 0, stream, part, B, group, P,
                               (int)segments, dW);
        else
            hipLaunchKernelGGL((wbp_reduce_kernel<VEC, true, false>), many, dim3(256), 0, stream, part, B, group, P,
                               (int)segments, dW);
        hipLaunchKernelGGL(wbp_reduce_segments_kernel<VEC>, one, dim3(256), 0, stream, part, rows, group * P, P,
                           (int)segments, dW);
    } else if (group > 1) {
        hipLaunchKernelGGL((wbp_reduce_kernel<VEC, false, true>), one, dim3(256), 0, stream, part, B, group, P, 1, dW);
    } else {
        hipLaunchKernelGGL((wbp_reduce_kernel<VEC, false, false>), one, dim3(256), 0, stream, part, B, group, P, 1, dW);
    }
    return hip_check(hipGetLastError(), "wbp_reduce launch");
}

// ------------------------------------------------------------------ losses
// Bound by double-precision arithmetic (one exponential and one log1p per
// non-frozen position and iteration; the gradient of the frame-level losses
// one exponential and one division more).  A workgroup takes one frame, its
// wavefronts the iterations in turn, so an iteration's sum needs no workgroup
// barrier, and the lanes walk the non-frozen positions alone, staged in LDS
// with the frame's bits: walking all positions leaves the frozen lanes idle.
constexpr int kLossThreads = 256;
constexpr int kLossWaves = kLossThreads / 64;
constexpr int kLossMaxN = 4096;

// positions of the non-frozen nodes, the true bit in the top bit
__device__ __forceinline__ void stage_positions(const CodeDev& code, const uint8_t* u, uint16_t* pos) {
    for (int q = lid_x(); q < code.k; q += kLossThreads) {
        const int i = code.info_pos[q];
        pos[q] = (uint16_t)(i | (u[i] ? 0x8000 : 0));
    }
    __syncthreads();
}

// softplus(z) and sigmoid(z) from one exponential
__device__ __forceinline__ double softplus_of(double z, double e) { return fmax(z, 0.0) + log1p(e); }
__device__ __forceinline__ double sigmoid_of(double z, double e) { return (z > 0.0 ? 1.0 : e) / (1.0 + e); }

// sum over the wavefront, in every lane
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// zeros at the frozen nodes first, first + step, .. of a gradient row
__device__ __forceinline__ void zero_frozen(const CodeDev& code, float* row, int first, int step) {
    for (int i = first; i < code.N; i += step)
        if ((code.frozen_bits[i >> 5] >> (i & 31)) & 1u) row[i] = 0.0f;
}

// Cross-entropy losses: sum over `rows` LLR rows of the frame (LLR(u) after
// the last iteration, or L row 0 of every iteration in `saved`: the frozen
// prior is 0 where the loss reads) and the non-frozen i of softplus((2u_i - 1)
// lambda_i), times scale; d loss / d lambda_i = scale (2u_i - 1)
// sigmoid((2u_i - 1) lambda_i); in double.  Row r of frame f starts at lam +
// f * lam_frame + r * lam_row.
__global__ __launch_bounds__(kLossThreads) void wbp_bce_kernel(CodeDev code, const float* __restrict__ lam,
                                                               int64_t lam_frame, int64_t lam_row,
                                                               const uint8_t* __restrict__ u, int rows, double scale,
                                                               float* __restrict__ loss, float* __restrict__ dlam) {
    __shared__ uint16_t pos[kLossMaxN];
    __shared__ double red[kLossWaves];
    const int64_t f = gid_x();
    const int N = code.N, k = code.k, lane = lid_x() & 63, wave = lid_x() >> 6;
    stage_positions(code, u + f * N, pos);
    // several rows: a wavefront takes whole rows; one row: all wavefronts share it
    const int r_first = rows > 1 ? wave : 0, r_step = rows > 1 ? kLossWaves : 1;
    const int q_first = rows > 1 ? lane : lid_x(), q_step = rows > 1 ? 64 : kLossThreads;
    double acc = 0.0;
    for (int r = r_first; r < rows; r += r_step) {
        const float* lrow = lam + f * lam_frame + r * lam_row;
        float* drow = dlam + (f * rows + r) * N;
        for (int q = q_first; q < k; q += q_step) {
            const int i = pos[q] & 0x7FFF;
            const double s = (pos[q] & 0x8000) ? 1.0 : -1.0;
            const double z = s * (double)lrow[i];
            const double e = exp(-fabs(z));
            acc += softplus_of(z, e);
            drow[i] = (float)(scale * s * sigmoid_of(z, e));
        }
        zero_frozen(code, drow, q_first, q_step);
    }
    if (loss) {
        acc = wave_sum(acc);
        if (lane == 0) red[wave] = acc;
        __syncthreads();
        if (lid_x() == 0) {
            double tot = 0.0;
            for (int w = 0; w < kLossWaves; ++w) tot += red[w];
            loss[f] = (float)(tot * scale);
        }
    }
}

constexpr int kFrameLossMaxT = 256;

// Frame-level losses of frame f (one workgroup), from S_t = sum over the
// non-frozen i of softplus((2u_i - 1) lambda_{t,i}), lambda_{t,i} = saved L row
// 0 of iteration t plus the frozen prior (0 where the loss reads).  With the
// bits taken as independent, q_t = 1 - e^{-S_t} is the probability that some
// decision after iteration t is wrong, and P_u = prod_{t<=u} q_t that the frame
// is still undecided after iteration u.
//   ITER = false: loss = P_T, the probability that no iteration gets the
//     frame right (a smooth stand-in for a BP failure within T iterations);
//   ITER = true:  loss = sum_{u<T} P_u + c P_T, the expected number of
//     iterations beyond the first of an early-stopping decoder plus c per
//     frame still undecided after T (c = fail_weight).
// d loss / d lambda_{t,i} = scale * d loss / d S_t * (2u_i - 1)
// sigmoid((2u_i - 1) lambda_{t,i}), where d loss / d S_t = e^{-S_t} times the
// sum of the products that hold q_t, with q_t taken out: the product of the
// q before t times H_t, H_{T-1} = 1 (c with ITER), H_t = q_{t+1} H_{t+1}
// (+ 1 with ITER) -- one pass each way, no division.  All in double.
// T = 20, N = 1024, K + c = 536, 1024 frames: 436 us with every thread
// building each of those products anew, 148 us.
template <bool ITER>
__global__ __launch_bounds__(kLossThreads) void wbp_frame_loss_kernel(CodeDev code, const float* __restrict__ saved,
                                                                      const uint8_t* __restrict__ u, int T,
                                                                      double scale, double fail_weight,
                                                                      float* __restrict__ loss,
                                                                      float* __restrict__ dlam) {
    __shared__ uint16_t pos[kLossMaxN];
    __shared__ double S[kFrameLossMaxT];
    __shared__ double dS[kFrameLossMaxT];
    const int64_t f = gid_x();
    const int N = code.N, n = code.n, k = code.k, lane = lid_x() & 63, wave = lid_x() >> 6;
    stage_positions(code, u + f * N, pos);
    // one or two iterations of more than a wavefront's width: all wavefronts share
    // each (T = 1, one frame of N = 4096: 40 us with one wavefront, 14 us with all;
    // T = 3, 2048 frames of N = 256: 17 us by wavefronts, 19 us shared)
    const bool share = 2 * T <= kLossWaves && k > 64;
    const int t_first = share ? 0 : wave, t_step = share ? 1 : kLossWaves;
    const int q_first = share ? lid_x() : lane, q_step = share ? kLossThreads : 64;
    for (int t = t_first; t < T; t += t_step) {
        const float* lrow = saved + (((size_t)f * T + t) * 2 * n + n) * N;
        double acc = 0.0;
        for (int q = q_first; q < k; q += q_step) {
            const double z = ((pos[q] & 0x8000) ? 1.0 : -1.0) * (double)lrow[pos[q] & 0x7FFF];
            acc += softplus_of(z, exp(-fabs(z)));
        }
        acc = wave_sum(acc);
        if (lane == 0) {
            if (share) dS[t * kLossWaves + wave] = acc;  // added below
            else S[t] = acc;
        }
    }
    __syncthreads();
    if (lid_x() == 0) {
        if (share)
            for (int t = 0; t < T; ++t) {
                double s = 0.0;
                for (int w = 0; w < kLossWaves; ++w) s += dS[t * kLossWaves + w];
                S[t] = s;
            }
        double P = 1.0, L = 0.0;
        for (int t = 0; t < T; ++t) {
            dS[t] = P;  // the product of the q before t
            P *= -expm1(-S[t]);
            if (ITER && t < T - 1) L += P;
        }
        L = ITER ? L + fail_weight * P : P;
        if (loss) loss[f] = (float)(L * scale);
        double H = ITER ? fail_weight : 1.0;
        for (int t = T - 1; t >= 0; --t) {
            dS[t] *= exp(-S[t]) * H;
            H = (ITER ? 1.0 : 0.0) - expm1(-S[t]) * H;
        }
    }
    __syncthreads();
    for (int t = t_first; t < T; t += t_step) {
        const float* lrow = saved + (((size_t)f * T + t) * 2 * n + n) * N;
        float* drow = dlam + ((size_t)f * T + t) * N;
        const double g = scale * dS[t];
        for (int q = q_first; q < k; q += q_step) {
            const int i = pos[q] & 0x7FFF;
            const double sg = (pos[q] & 0x8000) ? 1.0 : -1.0;
            const double z = sg * (double)lrow[i];
            drow[i] = (float)(g * sg * sigmoid_of(z, exp(-fabs(z))));
        }
        zero_frozen(code, drow, q_first, q_step);
    }
}

// W[t][d][s][i] = Wc[t][d][s]: one weight per stage column spread over its
// nodes (2^n), VEC nodes per thread
template <int VEC>
__global__ __launch_bounds__(256) void wbp_expand_columns_kernel(const float* __restrict__ wc, int64_t total, int n,
                                                                 float* __restrict__ w) {
    const int64_t q = (gid_x() * 256 + lid_x()) * VEC;
    if (q >= total) return;
    const float x = wc[q >> n];
    FloatVec<VEC> o;
#pragma unroll
    for (int j = 0; j < VEC; ++j) o.v[j] = x;
    *reinterpret_cast<FloatVec<VEC>*>(w + q) = o;
}

// dWc[c] = sum over the N nodes of column c in double, one wavefront per
// column (one thread per column: a chain of N loads, 123 us for 400 columns of
// 1024): the gradient of a weight shared by the whole column
__global__ __launch_bounds__(256) void wbp_sum_columns_kernel(const float* __restrict__ dw, int64_t cols, int N,
                                                              float* __restrict__ dwc) {
    const int64_t c = gid_x() * 4 + (lid_x() >> 6);
    if (c >= cols) return;
    const int lane = lid_x() & 63;
    double acc = 0.0;
    for (int i = lane; i < N; i += 64) acc += (double)dw[c * N + i];
    acc = wave_sum(acc);
    if (lane == 0) dwc[c] = (float)acc;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ w, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, int64_t count,
                                                   float lr, float b1, float b2, float eps, float c1, float c2,
                                                   float lo, float hi) {
    const int64_t q = gid_x() * 256 + lid_x();
    if (q >= count) return;
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.0f - b1) * gq;
    const float vq = b2 * v[q] + (1.0f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    const float mh = mq / c1, vh = vq / c2;
    w[q] = fminf(fmaxf(w[q] - lr * mh / (sqrtf(vh) + eps), lo), hi);
}

}  // namespace
}  // namespace polarhip

using namespace polarhip;

extern "C" polar_status wbp_forward(const polar_code* code, const float* llr, int64_t B, const float* W, int32_t T,
                                    float llr_max, int32_t variant, float* llr_u, uint8_t* u_hat, float* saved,
                                    hipStream_t stream) {
    if (!code || (B > 0 && (!llr || !W || !llr_u || !u_hat)))
        return set_error(POLAR_ERR_INVALID_ARG, "wbp_forward: null argument");
    if (B < 0 || T < 1 || !(llr_max > 0.0f)) return set_error(POLAR_ERR_INVALID_ARG, "wbp_forward: bad sizes");
    if (variant != 0 && !bp_variant_supported(code->n, variant))
        return set_error(POLAR_ERR_INVALID_ARG, "wbp_forward: unknown variant");
    polar_status st = launch_bp_save(code, llr, B, T, llr_max, W, variant, u_hat, llr_u, nullptr, saved, stream);
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status wbp_bce(const polar_code* code, const float* llr_u, const uint8_t* u_true, int64_t B,
                                double scale, float* loss, float* dlam, hipStream_t stream) {
    if (!code || (B > 0 && (!llr_u || !u_true || !dlam))) return set_error(POLAR_ERR_INVALID_ARG, "wbp_bce: null argument");
    if (B < 0) return set_error(POLAR_ERR_INVALID_ARG, "wbp_bce: bad batch");
    if (B == 0) return ok_status();
    hipLaunchKernelGGL(wbp_bce_kernel, dim3((unsigned)B), dim3(kLossThreads), 0, stream, code->dev(), llr_u,
                       (int64_t)code->N, (int64_t)0, u_true, 1, scale, loss, dlam);
    polar_status st = hip_check(hipGetLastError(), "wbp_bce launch");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status wbp_bce_multi(const polar_code* code, const float* saved, const uint8_t* u_true, int64_t B,
                                      int32_t T, double scale, float* loss, float* dlam, hipStream_t stream) {
    if (!code || (B > 0 && (!saved || !u_true || !dlam)))
        return set_error(POLAR_ERR_INVALID_ARG, "wbp_bce_multi: null argument");
    if (B < 0 || T < 1 || B > (int64_t)INT32_MAX) return set_error(POLAR_ERR_INVALID_ARG, "wbp_bce_multi: bad sizes");
    if (B == 0) return ok_status();
    const int64_t iter = (int64_t)2 * code->n * code->N;  // L row 0 of an iteration: after its n R rows
    hipLaunchKernelGGL(wbp_bce_kernel, dim3((unsigned)B), dim3(kLossThreads), 0, stream, code->dev(), saved + iter / 2,
                       T * iter, iter, u_true, T, scale, loss, dlam);
    polar_status st = hip_check(hipGetLastError(), "wbp_bce_multi launch");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status wbp_backward(const polar_code* code, const float* llr, int64_t B, const float* W, int32_t T,
                                     float llr_max, int32_t variant, float* saved, const float* dlam,
                                     int32_t dlam_iters, float* dW, float* dllr, hipStream_t stream) {
    if (!code || !W || !dW || (B > 0 && (!llr || !saved || !dlam)))
        return set_error(POLAR_ERR_INVALID_ARG, "wbp_backward: null argument");
    if (B < 0 || T < 1 || !(llr_max > 0.0f)) return set_error(POLAR_ERR_INVALID_ARG, "wbp_backward: bad sizes");
    if (dlam_iters != 1 && dlam_iters != T)
        return set_error(POLAR_ERR_INVALID_ARG, "wbp_backward: dlam_iters must be 1 or T");
    const bool grouped = variant == 0 && bwd_grouped(code->n, B);
    const int v = variant ? variant : grouped ? bwd_group_variant(code->n) : bwd_default_variant(code->n);
    const bp::BwdEntry* e = bp::lookup_bwd(code->n, v);
    if (!e) return set_error(POLAR_ERR_UNSUPPORTED, "wbp_backward: no kernel variant for this block length");
    const int64_t P = (int64_t)T * 2 * code->n * code->N;
    if (B > 0) {
        const int64_t per = grouped ? e->group : e->fpw;
        hipLaunchKernelGGL((grouped ? e->group_fn : e->fn), dim3((unsigned)((B + per - 1) / per)),
                           dim3(grouped ? e->group_wg : e->wg), 0, stream, code->dev(), llr, B, T, llr_max, W, saved,
                           dlam, dlam_iters, dllr);
        polar_status st = hip_check(hipGetLastError(), "wbp_bwd launch");
        if (st != POLAR_OK) return st;
    }
    const int group = grouped ? e->group : 1;
    // 16-byte accesses where both buffers allow them (P is a multiple of 4)
    polar_status st = aligned16(saved) && aligned16(dW) ? launch_reduce<4>(saved, B, group, P, dW, stream)
                                                        : launch_reduce<1>(saved, B, group, P, dW, stream);
    return st == POLAR_OK ? ok_status() : st;
}

static polar_status adam_launch(float* w, const float* g, float* m, float* v, int64_t count, int32_t step, float lr,
                                float beta1, float beta2, float eps, float lo, float hi, hipStream_t stream) {
    if (!w || !g || !m || !v || count < 0 || step < 1) return set_error(POLAR_ERR_INVALID_ARG, "polar_adam_step: bad argument");
    if (!(lo <= hi)) return set_error(POLAR_ERR_INVALID_ARG, "polar_adam_step_bounded: need lo <= hi");
    if (count == 0) return ok_status();
    const float c1 = (float)(1.0 - std::pow((double)beta1, step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, step));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, w, g, m, v, count, lr,
                       beta1, beta2, eps, c1, c2, lo, hi);
    polar_status st = hip_check(hipGetLastError(), "adam launch");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status polar_adam_step(float* w, const float* g, float* m, float* v, int64_t count, int32_t step,
                                        float lr, float beta1, float beta2, float eps, hipStream_t stream) {
    return adam_launch(w, g, m, v, count, step, lr, beta1, beta2, eps, -INFINITY, INFINITY, stream);
}

extern "C" polar_status polar_adam_step_bounded(float* w, const float* g, float* m, float* v, int64_t count,
                                                int32_t step, float lr, float beta1, float beta2, float eps, float lo,
                                                float hi, hipStream_t stream) {
    return adam_launch(w, g, m, v, count, step, lr, beta1, beta2, eps, lo, hi, stream);
}

static polar_status frame_loss_launch(const char* who, bool iter, const polar_code* code, const float* saved,
                                      const uint8_t* u_true, int64_t B, int32_t T, double fail_weight, double scale,
                                      float* loss, float* dlam, hipStream_t stream) {
    if (!code || (B > 0 && (!saved || !u_true || !dlam)))
        return set_error(POLAR_ERR_INVALID_ARG, std::string(who) + ": null argument");
    if (B < 0 || T < 1 || T > kFrameLossMaxT || B > (int64_t)INT32_MAX)
        return set_error(POLAR_ERR_INVALID_ARG, std::string(who) + ": bad sizes (1 <= T <= 256)");
    if (!(fail_weight >= 0.0)) return set_error(POLAR_ERR_INVALID_ARG, std::string(who) + ": fail_weight < 0");
    if (B == 0) return ok_status();
    if (iter)
        hipLaunchKernelGGL(wbp_frame_loss_kernel<true>, dim3((unsigned)B), dim3(kLossThreads), 0, stream, code->dev(), saved,
                           u_true, T, scale, fail_weight, loss, dlam);
    else
        hipLaunchKernelGGL(wbp_frame_loss_kernel<false>, dim3((unsigned)B), dim3(kLossThreads), 0, stream, code->dev(), saved,
                           u_true, T, scale, fail_weight, loss, dlam);
    polar_status st = hip_check(hipGetLastError(), "frame loss launch");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status wbp_frame_loss(const polar_code* code, const float* saved, const uint8_t* u_true, int64_t B,
                                       int32_t T, double scale, float* loss, float* dlam, hipStream_t stream) {
    return frame_loss_launch("wbp_frame_loss", false, code, saved, u_true, B, T, 0.0, scale, loss, dlam, stream);
}

extern "C" polar_status wbp_iteration_loss(const polar_code* code, const float* saved, const uint8_t* u_true,
                                           int64_t B, int32_t T, double fail_weight, double scale, float* loss,
                                           float* dlam, hipStream_t stream) {
    return frame_loss_launch("wbp_iteration_loss", true, code, saved, u_true, B, T, fail_weight, scale, loss, dlam,
                             stream);
}

extern "C" polar_status wbp_column_weights(const polar_code* code, const float* Wc, int32_t T, float* W,
                                           hipStream_t stream) {
    if (!code || !Wc || !W) return set_error(POLAR_ERR_INVALID_ARG, "wbp_column_weights: null argument");
    if (T < 1) return set_error(POLAR_ERR_INVALID_ARG, "wbp_column_weights: T < 1");
    const int64_t cols = (int64_t)T * 2 * code->n, tot = cols * code->N;
    const unsigned blocks = (unsigned)((tot + 1023) / 1024);
    if (aligned16(W))
        hipLaunchKernelGGL(wbp_expand_columns_kernel<4>, dim3(blocks), dim3(256), 0, stream, Wc, tot, code->n, W);
    else
        hipLaunchKernelGGL(wbp_expand_columns_kernel<1>, dim3(4 * blocks), dim3(256), 0, stream, Wc, tot, code->n, W);
    polar_status st = hip_check(hipGetLastError(), "wbp_column_weights launch");
    return st == POLAR_OK ? ok_status() : st;
}

extern "C" polar_status wbp_column_grad(const polar_code* code, const float* dW, int32_t T, float* dWc,
                                        hipStream_t stream) {
    if (!code || !dW || !dWc) return set_error(POLAR_ERR_INVALID_ARG, "wbp_column_grad: null argument");
    if (T < 1) return set_error(POLAR_ERR_INVALID_ARG, "wbp_column_grad: T < 1");
    const int64_t cols = (int64_t)T * 2 * code->n;
    hipLaunchKernelGGL(wbp_sum_columns_kernel, dim3((unsigned)((cols + 3) / 4)), dim3(256), 0, stream, dW, cols,
                       code->N, dWc);
    polar_status st = hip_check(hipGetLastError(), "wbp_column_grad launch");
    return st == POLAR_OK ? ok_status() : st;
}
