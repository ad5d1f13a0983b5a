// Propagator pass over neighbouring partitions of a line, or over a batch of
// segments of any sizes and rates (f32), for gfx950:
// the form of hx_prop1d.hip's block walk for lines of any length, alignment
// and boundary, at depths up to 256 steps, with nothing laid out beforehand.
//
// D steps are one convolution with the D-step propagator, whose taps fall off
// like a Gaussian of variance 2 r D: at r = 1/4 the taps beyond 64 cells sum to
// less than 2^-32 even after 200 steps, so a window of 64 cells on each side
// serves every depth with 2 r D up to about 100.  A wave advances one block of
// 1024 cells, four waves of consecutive blocks to a workgroup.  Loads, scale,
// two-term fp16 split, products, accuracy check and stores are the block
// walk's.  What differs:
//   * Taps.  The host sends one copy of the split taps with the launch (up to
//     192 fp16 pairs); each workgroup lays out its eight shifted copies.
//   * Reach.  A block's outputs depend on D cells on each side.  Past the
//     window (D > 64) those cells meet omitted taps only; the check bounds
//     everything omitted by E times the largest |x| of the neighbouring blocks
//     (or of 256 cells read beside the workgroup), and a non-finite cell there
//     fails it.
//   * A block that fails is stepped in registers (24 cells per lane, the
//     direct form's arithmetic), 2 instructions per cell and step.
//   * Boundaries.  Blocks near an end take what lies past it from the
//     neighbour's cells, or, past a zero-Dirichlet end, from the odd reflection
//     of the line about the ghost cell (u_{-1} = 0, u_{-2-k} = -u_k), which the
//     steps preserve exactly: four cells in one load, cell by cell only where
//     four straddle an end or the far end of a halo (line_cells4).
//   * Blocks start at the run's first cell whatever its address, so the bits do
//     not depend on where a run lies in memory, nor on who launches the pass (a
//     node of a graph, or all partitions in one).  (Blocks that start where `out`
//     is 128-byte aligned store whole lines: 1 to 5 % faster on misaligned runs
//     of 2^25 cells and more, 820 us against 834 for a batch of 622 million, and
//     up to 2 % slower on short ones.)
// Bound: HBM (or the last-level cache) for long lines, launch and one block's
// latency for short ones.  Measured, a pass of 20 / 50 / 200 steps: 2^20 cells
// 5.3 / 5.6 / 6.5 us, 2^22 9.1 / 9.7 / 10.7 us, 2^24 26 / 27 / 33 us, 2^26
// 98 / 104 / 134 us (5.5 / 5.2 / 4.0 TB/s); the direct form needs 110 us for
// 200 steps of 12345679 cells, this one 26 us.  80 VGPRs (6 waves per
// SIMD; the stepping path spills 32 to 34, the others none: one value spilled
// ahead of the products and reloaded among them cost a batch of 622 million
// cells 8 %): with 128 (4 waves) 2^24 cells and 50 steps took 12 % longer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>

#include "hx_internal.h"
#include "hx_line.hpp"

namespace hx {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kPlane = 36 * 64;   // bytes of one fp16 plane of the 1152-cell window
constexpr int kReach = 256;       // deepest pass
// The shallowest pass the library takes in this form.  From here on its error
// against 64 bits is the smaller one on positive noise and on smooth fields at
// every rate measured (r = 1/20 .. 1/4, 12 to 200 steps: 0.46-0.64e-7 against
// 0.56-10e-7), per cell also on noise of both signs.  The worst cell of combs of
// lone values, of spikes in noise and of log-normal noise, 300 rates from 1/1000
// to 1/4 and depths from 20 to 256 worked out in the products' own arithmetic:
// 4.9e-7, and no larger than stepping's of the same field but for 4 in 8474
// (by at most an eighth).
constexpr int kPropMinDepth = 20;
constexpr int kEdge = 320;        // cells a block may read on each side (the window and 256)
constexpr float kMaxF = 3.402823466e38f;

constexpr int units_of(int NC) { return 2 * NC + 3; }

__device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Byte offset of 16-byte unit `unit` of window row `row` (32 cells) in a plane.
__device__ __forceinline__ int swz(int row, int unit) {
    return row * 64 + ((unit ^ ((row >> 1) & 3)) << 4);
}

// x 2^e for two values, split into packed fp16 pairs hi + lo, each rounded to
// nearest.
__device__ __forceinline__ void split16(float x0, float x1, int e, uint32_t& h, uint32_t& l) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 s = {ldexpf(x0, e), ldexpf(x1, e)};
    const h2 hi = __builtin_convertvector(s, h2);
    const f2 rem = s - __builtin_convertvector(hi, f2);
    h = __builtin_bit_cast(uint32_t, hi);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(rem, h2));
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = __builtin_elementwise_maximum(x, __shfl_xor(x, o));
    return x;
}

typedef __attribute__((address_space(1))) const float GF;

// One run of cells as a block sees it: a partition or a segment.
struct Part {
    const float* in;
    float* out;
    int64_t n;
    const float* lo;  // hw cells before the first, or null: a zero-Dirichlet end
    const float* hi;  // hw cells after the last, or null
    int hw;
};

// Cell c of the line: the run's own, its neighbours' or the reflection.  Cells
// further out than D meet no tap and no check; their index is clamped to what
// is there.
__device__ __forceinline__ float line_cell(const Part& s, int64_t c) {
    if (c >= 0 && c < s.n) return ((GF*)s.in)[c];
    if (c < 0) {
        if (s.lo) return ((GF*)s.lo)[s.hw + c < 0 ? 0 : s.hw + c];
        return c == -1 ? 0.f : -((GF*)s.in)[-c - 2 < s.n ? -c - 2 : s.n - 1];
    }
    const int64_t k = c - s.n;
    if (s.hi) return ((GF*)s.hi)[k >= s.hw ? s.hw - 1 : k];
    return k == 0 ? 0.f : -((GF*)s.in)[k <= s.n ? s.n - k : 0];
}

// Cells c .. c + 3.  Four cells on one side of both ends are one load (of the
// reflection, reversed); only a group that straddles an end, or the far end of
// a halo, takes its cells one by one (each a round trip to memory: with all
// groups of an end's block taken so, a batch of 4096 short segments ran at half
// speed).  A group wholly past a halo loads the halo's last four cells.
// (Reflected cells are in reach up to D <= n from the end, so the clamp to the
// run meets none that a tap of the window does: those are at most 95 cells
// away, and the run has at least 256.)
__device__ __forceinline__ f32x4 line_cells4(const Part& s, int64_t c, bool inside) {
    typedef __attribute__((address_space(1))) const f32x4u G;
    if (inside) return *(G*)(s.in + c);
    const float* base = s.in;
    int64_t at = c;
    bool whole = true, flip = false;
    if (c + 4 <= 0) {
        if (s.lo) {
            base = s.lo;
            at = s.hw + c < 0 ? 0 : s.hw + c;
            whole = s.hw + c >= 0 || (s.hw + c <= -4 && s.hw >= 4);
        } else {
            flip = true;
            at = -c - 5 < s.n - 4 ? -c - 5 : s.n - 4;
            whole = c < -4;
        }
    } else if (c >= s.n) {
        const int64_t k = c - s.n;
        if (s.hi) {
            base = s.hi;
            at = k < s.hw - 4 ? k : s.hw - 4;
            whole = k + 4 <= s.hw || (k >= s.hw && s.hw >= 4);
        } else {
            flip = true;
            at = s.n - 3 - k > 0 ? s.n - 3 - k : 0;
            whole = k > 0;
        }
    } else {
        whole = c >= 0 && c + 4 <= s.n;
    }
    f32x4 v = {};
    if (whole) {
        v = *(G*)(base + at);
        if (flip) v = f32x4{-v[3], -v[2], -v[1], -v[0]};
    } else {
#pragma unroll 1
        for (int e = 0; e < 4; ++e) v[e] = line_cell(s, c + e);
    }
    return v;
}

// This lane's number, worked out where it is asked for (opaque to the compiler,
// which otherwise keeps what follows from it in registers across the kernel).
__device__ __forceinline__ int lane_here() {
    int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}

__device__ __forceinline__ float far4(const f32x4& x) {
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) m = __builtin_elementwise_maximum(m, fabsf(x[e]));
    return m;
}

// The stepping path of one block: its cells c0 .. c0 + 1023 advanced D steps
// over the window of 256 cells on each side, 24 consecutive cells per lane, in
// the rescaled direct form.  Past a zero-Dirichlet end the cells are 0 and reset
// after every step, as there (the reflection's ghost cell, the sum of opposite
// cells, would be NaN beside an infinity).
__device__ __forceinline__ void step_line(const Part& s, const PropLine& pl, int64_t c0) {
    constexpr int K = 24;
    const int l = lane_here();
    const int64_t b = c0 - kReach + (int64_t)K * l;
    float a[K];
    // the lane's cells from `lo` on and before `hi` lie inside the line (32-bit
    // indices: with the 64-bit comparisons of step_tile_scaled the whole kernel
    // was scheduled worse, a batch of 622 million cells, of which next to none
    // are stepped, took 1045 us in place of 831)
    const int64_t before = s.lo ? 0 : -b, inside = s.hi ? K : s.n - b;
    const int lo = before < 0 ? 0 : (before > K ? K : (int)before);
    const int hi = inside < 0 ? 0 : (inside > K ? K : (int)inside);
    const bool ends = __ballot(lo > 0 || hi < K) != 0;
#pragma unroll
    for (int t = 0; t < K; ++t) a[t] = t < lo || t >= hi ? 0.f : line_cell(s, b + t);
    const float beta = pl.beta, ap = pl.ap;
    const int D = pl.D, period = pl.period;
    int since = 0;
    for (int k = 0; k < D; ++k) {
        step_tile_scaled<float, K>(a, beta, false, false, 0, 0);
        if (ends) {
#pragma unroll
            for (int t = 0; t < K; ++t) a[t] = t < lo || t >= hi ? 0.f : a[t];
        }
        if (++since == period) {
            since = 0;
            scale_tile<float, K>(a, ap);
        }
    }
    if (since) scale_tile<float, K>(a, pl.ar);
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const int64_t c = b + t;
        if (c >= c0 && c < c0 + 1024 && c < s.n) s.out[c] = a[t];
    }
}

// The blocks 4 wg .. 4 wg + 3 of one run, a wave each.  NT: nontemporal loads
// of the block's own cells and stores (arrays that do not stay in the caches
// between passes).
template <int NC, bool NT>
__device__ __forceinline__ void line_blocks(const Part& s, const PropLine& a, uint32_t wg,
                                            char* lds_all, float* wmax) {
    constexpr int U = units_of(NC);
    constexpr int kUnits = 16 * U;
    char* const tl = lds_all + 4 * 2 * kPlane;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const lds = lds_all + wv * 2 * kPlane;
    const int l = threadIdx.x & 63;
    const int64_t c0 = 1024 * (4 * (int64_t)wg + wv);
    const bool live = c0 < s.n;
    const bool inside = c0 >= kEdge && c0 + 1024 + kEdge <= s.n;
    // the window, as in the block walk: cells 256 j + 4 l of the block and 64
    // context cells on each side; then, past them, what else is within reach
    const int q = l & 15;
    const bool left = (l & 31) < 16;
    f32x4 v[5] = {};
    float far = 0.f;  // the largest |x| beside the workgroup
    if (live) {
        typedef __attribute__((address_space(1))) const f32x4u G;
        const int64_t cx = (left ? c0 - 64 : c0 + 1024) + 4 * q;
        if (inside) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = NT ? (f32x4)__builtin_nontemporal_load((G*)(s.in + c0 + 256 * j + 4 * l))
                          : (f32x4)*(G*)(s.in + c0 + 256 * j + 4 * l);
            v[4] = *(G*)(s.in + cx);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = line_cells4(s, c0 + 256 * j + 4 * l, false);
            v[4] = line_cells4(s, cx, false);
        }
        // past the window a wave's neighbours in the workgroup know their own
        // maxima; the outer waves read 256 cells
        if (a.D > 64) {
            if (wv == 0) far = far4(line_cells4(s, c0 - 320 + 4 * l, inside));
            if (wv == 3 || c0 + 1024 >= s.n)
                far = __builtin_elementwise_maximum(
                    far, far4(line_cells4(s, c0 + 1088 + 4 * l, inside)));
        }
    }
    // eight shifted copies of the split taps: unit u of copy c of a level holds
    // its taps c + 8 u .. + 7
    for (int k = (int)threadIdx.x; k < kUnits; k += 256) {
        const int lv = k / (8 * U), c = (k - lv * 8 * U) / U, u = k % U;
        const int b = c + 8 * u;
        const uint32_t* w = reinterpret_cast<const uint32_t*>(a.tap[lv]) + (b >> 1);
        u32x4 x;
        if (b & 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = __builtin_amdgcn_alignbit(w[e + 1], w[e], 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = w[e];
        }
        *reinterpret_cast<u32x4*>(tl + 16 * k) = x;
    }
    // the window's scale: its largest |x| (fails the block below if non-finite)
    float mx = 0.f;
#pragma unroll
    for (int j = 0; j < 5; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = __builtin_elementwise_maximum(mx, fabsf(v[j][e]));
    mx = wave_max(mx);
    const bool outer = wv == 0 || wv == 3 || c0 + 1024 >= s.n;
    if (a.D > 64) {
        if (l == 0) wmax[wv] = mx;
        if (outer) far = wave_max(far);
    }
    const bool finite = mx <= kMaxF;
    const int ex = __builtin_amdgcn_readfirstlane(
        finite && mx > 0.f ? 15 - __builtin_amdgcn_frexp_expf(mx) : 0);
    {
        int woff[5];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            woff[j] = swz(2 + 8 * j + (l >> 3), (l & 7) >> 1) + 8 * (l & 1);
        woff[4] = swz((left ? 0 : 34) + (q >> 3), (q & 7) >> 1) + 8 * (q & 1);
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            uint32_t h0, l0, h1, l1;
            split16(v[j][0], v[j][1], ex, h0, l0);
            split16(v[j][2], v[j][3], ex, h1, l1);
            char* d = lds + woff[j];
            *reinterpret_cast<u32x2*>(d) = u32x2{h0, h1};
            *reinterpret_cast<u32x2*>(d + kPlane) = u32x2{l0, l1};
        }
    }
    __syncthreads();
    if (!live) return;
    float M = mx;  // the largest |x| within reach, or more
    if (a.D > 64) {
        if (outer) M = __builtin_elementwise_maximum(M, far);
        if (wv > 0) M = __builtin_elementwise_maximum(M, wmax[wv - 1]);
        if (wv < 3) M = __builtin_elementwise_maximum(M, wmax[wv + 1]);
    }
    // products: the terms of the cells' and the taps' leading halves from the
    // outer chunks inwards, the cross terms (2^-11 of them) apart, so that few
    // of the sums round at the output's own scale (relative error 5.1e-8 after
    // 50 steps of noise at r = 1/4; all in one sum 8.8e-8, stepping 8.3e-8).
    // Narrow windows serve shallow passes, whose stepped error is smaller, and
    // take the product of the two lower halves too.
    const int ln = lane_here(), i = ln & 31, g = ln >> 5;
    const int d0 = 8 * g + 31 - i;
    const char* ta = tl + 16 * ((d0 & 7) * U + (d0 >> 3));
    f32x16 acc = {}, low = {};
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const int c = k & 1 ? NC - 1 - k / 2 : k / 2;
        const int X = 16 * c + 8 * g - 8 * (NC - 2);
        const char* w = lds + swz(2 + i + (X >> 5), (X & 31) >> 3);
        const int L = (a.levels >> (2 * c)) & 3;
        const u32x4 bh = *reinterpret_cast<const u32x4*>(w);
        const u32x4 bl = *reinterpret_cast<const u32x4*>(w + kPlane);
        const u32x4 ah = *reinterpret_cast<const u32x4*>(ta + 32 * c);
        const u32x4 al = *reinterpret_cast<const u32x4*>(ta + 32 * c + 16 * 8 * U);
        if (L >= 1) acc = mfma16(ah, bh, acc);
        if (L >= 2) {
            low = mfma16(ah, bl, low);
            low = mfma16(al, bh, low);
            if (NC <= 6) low = mfma16(al, bl, low);
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] += low[e];
    __builtin_amdgcn_sched_barrier(0);
    // the accuracy check, in the products' scale: what was omitted, at most E M,
    // is within 2^-21 of every output, or else of the sum of |p_j u_{i+j}| the
    // output cancelled from (the scale of stepping's own rounding), which one
    // more product per chunk, of the taps and the cells' magnitudes, gives
    float mn = fabsf(acc[0]), mo = mn;
#pragma unroll
    for (int e = 1; e < 16; ++e) {
        mn = __builtin_elementwise_minimum(mn, fabsf(acc[e]));
        mo = __builtin_elementwise_maximum(mo, fabsf(acc[e]));
    }
    const float thr = a.chk * ldexpf(M, ex);
    const bool bad = __ballot(!(M <= kMaxF) || !(mo <= kMaxF)) != 0;
    if (bad || __ballot(!(mn >= thr)) != 0) {
        bool fail = bad;
        if (!bad) {
            f32x16 sum = {};
#pragma unroll 1
            for (int c = 0; c < NC; ++c) {
                const int X = 16 * c + 8 * g - 8 * (NC - 2);
                u32x4 bh =
                    *reinterpret_cast<const u32x4*>(lds + swz(2 + i + (X >> 5), (X & 31) >> 3));
                bh &= 0x7fff7fffu;
                sum = mfma16(*reinterpret_cast<const u32x4*>(ta + 32 * c), bh, sum);
            }
            mn = sum[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mn = __builtin_elementwise_minimum(mn, sum[e]);
            fail = __ballot(!(mn >= thr)) != 0;
        }
        if (fail) {
            step_line(s, a, c0);
            return;
        }
    }
    // the outputs, scaled back and transposed through the window's planes
    auto tpos = [](int row, int unit) {
        return (row < 16 ? 0 : kPlane) + (row & 15) * 128 + ((unit ^ (row & 7)) << 4);
    };
    const int sc = -(ex + a.texp);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4*>(lds + tpos(i, 2 * e + g)) =
            f32x4{ldexpf(acc[4 * e], sc), ldexpf(acc[4 * e + 1], sc), ldexpf(acc[4 * e + 2], sc),
                  ldexpf(acc[4 * e + 3], sc)};
    f32x4 o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o[j] = *reinterpret_cast<const f32x4*>(lds + tpos(8 * j + (ln >> 3), ln & 7));
    const int64_t oc = c0 + 4 * ln;
    if (c0 + 1024 <= s.n) {
        typedef __attribute__((address_space(1))) f32x4u GO;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (NT)
                __builtin_nontemporal_store(o[j], (GO*)(s.out + oc + 256 * j));
            else
                *(GO*)(s.out + oc + 256 * j) = o[j];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t c = oc + 256 * j + e;
                if (c < s.n) s.out[c] = o[j][e];
            }
    }
}

// The workgroup's place in the line: workgroups go round the 8 XCDs in turn;
// in each 128 of them an XCD takes 16 consecutive ones, whose edges (and, in a
// batch, taps) then meet in its L2.  2^24 cells, 50 / 200 steps: 27.3 / 32.8 us
// against 27.5 / 34.5 in launch order; 622 million cells, 20 steps: 833
// against 858 (runs of 4: 889, of 64: 846, of 1024: 862).
__device__ __forceinline__ uint32_t local_group() {
    constexpr uint32_t C = 16, G = 8 * C;
    const uint32_t b = blockIdx.x, k = b % G;
    return b - k + G <= gridDim.x ? b - k + (k % 8) * C + k / 8 : b;
}

template <int NC>
constexpr int kLineLds = 4 * 2 * kPlane + 16 * 16 * units_of(NC);

// Neighbouring partitions: workgroups before partition p, and the most that a
// partition has.
struct LineGrid {
    uint32_t first[kMaxParts + 1];
    uint32_t per;
};

template <int NC, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8)))
void k_prop1d_line(PartSet1D ps, PropLine a, LineGrid f) {
    __shared__ __attribute__((aligned(16))) char lds[kLineLds<NC>];
    __shared__ float wmax[4];
    const uint32_t w = local_group();
    int p = (int)(w / f.per);
    while (w >= f.first[p + 1]) ++p;
    Part s;
    s.in = static_cast<const float*>(ps.in[p]);
    s.out = static_cast<float*>(ps.out[p]);
    s.n = ps.n[p];
    s.hw = a.D;
    s.lo = p > 0 ? static_cast<const float*>(ps.in[p - 1]) + (ps.n[p - 1] - a.D)
                 : static_cast<const float*>(ps.halo_lo);
    s.hi = static_cast<const float*>(p + 1 < ps.count ? ps.in[p + 1] : ps.halo_hi);
    line_blocks<NC, NT>(s, a, w - f.first[p], lds, wmax);
}

template <int NC, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8)))
void k_prop1d_segs(const LineSeg* __restrict__ segs, const uint32_t* __restrict__ wg_seg) {
    __shared__ __attribute__((aligned(16))) char lds[kLineLds<NC>];
    __shared__ float wmax[4];
    const uint32_t w = local_group();
    const LineSeg& q = segs[__builtin_amdgcn_readfirstlane(wg_seg[w])];
    Part s;
    s.in = q.in;
    s.out = q.out;
    s.n = q.n;
    s.lo = q.lo;
    s.hi = q.hi;
    s.hw = q.hw;
    line_blocks<NC, NT>(s, q.pl, w - q.first, lds, wmax);
}

// From this many cells on, a pass's arrays (8 bytes per cell) outgrow the
// 256 MB last-level cache and are better streamed past it.
constexpr int64_t kNtCells = int64_t(1) << 25;

// The taps p_j, 0 <= j <= K, of the D-step propagator (p_{-j} = p_j), by the
// downward recurrence (D - j + 1) p_{j-1} = (D + j + 1) p_{j+1} + (a/r) j p_j
// of the coefficients of (r/x + a + r x)^D, a = 1 - 2r, whose terms are all
// positive (no cancellation), normalised to sum 1; K = D, or where the taps
// have fallen below 1e-40 of the largest.
int line_taps(double r, int D, double (&p)[kReach + 2]) {
    const double sigma = std::sqrt(2.0 * r * D);
    const int K = std::min(D, (int)(14.0 * sigma) + 20);
    p[K + 1] = 0.0;
    p[K] = 1e-280;
    const double q = (1.0 - 2.0 * r) / r;
    // (the divisions ahead of the recurrence, out of its chain: a batch of 4096
    // rates pays for as many)
    double a[kReach + 2], b[kReach + 2];
    for (int j = 1; j <= K; ++j) {
        a[j] = (double)(D + j + 1) / (D - j + 1);
        b[j] = q * j / (D - j + 1);
    }
    for (int j = K; j >= 1; --j) p[j - 1] = a[j] * p[j + 1] + b[j] * p[j];
    double sum = p[0];
    for (int j = 1; j <= K; ++j) sum += 2.0 * p[j];
    for (int j = 0; j <= K; ++j) p[j] /= sum;
    return K;
}

// x rounded to the nearest fp16 (|x| < 65504, ties to even): its bits in *h, its
// value returned.
float to_half(float x, uint16_t* h) {
    const uint32_t b = __builtin_bit_cast(uint32_t, x), sign = b & 0x80000000u;
    const float a = __builtin_bit_cast(float, b & 0x7fffffffu);
    if (a < 6.103515625e-05f) {  // below 2^-14: multiples of 2^-24
        volatile float q = a * 16777216.0f + 8388608.0f;
        const float n = q - 8388608.0f;
        *h = (uint16_t)((sign >> 16) | (uint32_t)n);
        return sign ? -n / 16777216.0f : n / 16777216.0f;
    }
    const uint32_t m = b & 0x7fffffffu;
    const uint32_t r = (m + 0xfffu + ((m >> 13) & 1u)) & ~0x1fffu;
    *h = (uint16_t)((sign >> 16) | ((r - 0x38000000u) >> 13));
    return __builtin_bit_cast(float, sign | r);
}

}  // namespace

bool propline_setup(double r, int D, PropLine* out, int min_H) {
    // (up to r = 1/4 the taps fall monotonically from p_0)
    if (!(r >= 1e-3 && r <= 0.25) || D < 1 || D > kReach) return false;
    double p[kReach + 2];
    const int K = line_taps(r, D, p);
    auto tap = [&](int j) { return std::abs(j) <= K ? p[std::abs(j)] : 0.0; };
    // Everything omitted is kept near the fp16 split's own floors (2^-39 of the
    // window's largest), so that only outputs some 2^-15 of their surroundings
    // or smaller fail the check: the zero crossings of a smooth field mostly
    // pass.  The half window: the least multiple of 8 cells whose outer taps
    // sum to less than 2^-39 (all sum to 1), at most 64.
    double tail[kReach + 2];  // tail[j] = sum of p_k, k >= j
    tail[K + 1] = 0.0;
    for (int j = K; j >= 0; --j) tail[j] = tail[j + 1] + p[j];
    auto past = [&](int j) { return tail[std::min(std::max(j, 0), K + 1)]; };
    int H = std::max(8, min_H);
    while (H < 64 && 2.0 * past(H + 1) > 1.8e-12) H += 8;
    const int NC = (32 + 2 * H) / 16;
    // products per chunk (prop1d_levels16's rule at 2^-40)
    const double eps = std::ldexp(1.0, -40);
    uint32_t levels = 0;
    for (int c = 0; c < NC; ++c) {
        const int j0 = 16 * c - H - 31, j1 = 16 * c - H + 15;
        const double t = j0 <= 0 && j1 >= 0 ? p[0] : tap(std::min(std::abs(j0), std::abs(j1)));
        const uint32_t L = 16.0 * t <= eps ? 0 : (32.0 * t / 2048.0 <= eps ? 1 : 2);
        levels |= L << (2 * c);
    }
    int texp = 0;
    std::frexp(p[0], &texp);
    texp = 15 - texp;  // p_0 2^texp in [2^14, 2^15)
    // E as prop1d_err_bound, with the taps outside the window of each row
    auto range = [&](int j0, int j1) {  // sum of p_j, j0 <= j <= j1
        if (j1 < j0) return 0.0;
        if (j0 >= 0) return past(j0) - past(j1 + 1);
        if (j1 < 0) return past(-j1) - past(-j0 + 1);
        return past(0) + past(1) - past(j1 + 1) - past(-j0 + 1);
    };
    double E = 0.0;
    for (int m = 0; m < 16; ++m) {  // (row 31 - m mirrors row m)
        double e = past(H + m + 1) + past(H + 32 - m);
        for (int c = 0; c < NC; ++c) {
            const uint32_t L = (levels >> (2 * c)) & 3;
            if (L == 2) continue;
            const int j0 = 16 * c - H - m;
            e += (L == 0 ? 1.0 : 1.0 / 1024.0) * range(j0, j0 + 15);
        }
        E = std::max(E, e);
    }
    E += std::ldexp(1.0, -39) + (2 * H + 32) * std::ldexp(1.0, -25 - texp);
    if (E > std::ldexp(1.0, -30)) return false;  // 2 r D beyond what the window holds
    out->D = D;
    out->H = H;
    out->levels = levels;
    out->texp = texp;
    out->chk = (float)std::ldexp(E, 21 + texp);
    std::memset(out->tap, 0, sizeof out->tap);
    // (each tap is rounded by itself: its two halves are within 2^-23 of it.
    // Handing the roundings on to the next tap out, so that the rounded taps sum
    // to 1, gave a smooth field 10 % less error at r = 1/20, and cells that only
    // the next, far smaller tap reaches up to 3.9e-6)
    const double scale = std::ldexp(1.0, texp);
    for (int j = 0; j <= std::min(K, H + 31); ++j) {
        const double x = p[j] * scale;
        uint16_t hi, lo;
        const float xh = to_half((float)x, &hi);
        to_half((float)(x - xh), &lo);
        for (int k : {H + 31 + j, H + 31 - j}) {
            if (k >= 8 * units_of(NC) + 8) continue;
            out->tap[0][k] = hi;
            out->tap[1][k] = lo;
        }
    }
    Seg1D rate{};
    rate.r = r;
    set_rate_1d(rate, D);
    out->beta = (float)rate.beta;
    out->ap = (float)rate.alpha_p;
    out->ar = (float)rate.alpha_rem;
    out->period = rate.period;
    return true;
}

// Fitted to passes of 20 to 200 steps over lines from 2^18 to 2^28 cells
// (deviation at most 6 %).
double propline_us(double r, int64_t cells, int D, bool setup) {
    const double v = 2.0 * r * D;
    if (!(r >= 1e-3 && r <= 0.25) || D < kPropMinDepth || D > kReach || v > 104.0 ||
        cells < kPropLineMin)
        return std::numeric_limits<double>::infinity();
    const int H = std::min(64, ((int)(7.05 * std::sqrt(v)) + 8) / 8 * 8), NC = 2 + H / 8;
    const double m = 1e-6 * (double)cells;
    return (setup ? 0.5 + std::min(4.5, 0.028 * D) : 0.0) + 5.2 + 0.1 * NC +
           (D > 64 ? 0.4 : 0.0) + (0.75 + 0.02 * NC) * std::min(m, 4.0) +
           (1.13 + 0.04 * NC + (D > 64 ? 0.34 : 0.0)) * std::max(0.0, m - 4.0);
}

#define HX_LINE_SWITCH(H, nt, ...)  \
    switch ((32 + 2 * (H)) / 16) {  \
        HX_LINE_CASE(3, nt, __VA_ARGS__)  \
        HX_LINE_CASE(4, nt, __VA_ARGS__)  \
        HX_LINE_CASE(5, nt, __VA_ARGS__)  \
        HX_LINE_CASE(6, nt, __VA_ARGS__)  \
        HX_LINE_CASE(7, nt, __VA_ARGS__)  \
        HX_LINE_CASE(8, nt, __VA_ARGS__)  \
        HX_LINE_CASE(9, nt, __VA_ARGS__)  \
        HX_LINE_CASE(10, nt, __VA_ARGS__) \
    default: return hipErrorInvalidValue; \
    }

hipError_t launch_propline(const PartSet1D& set, const PropLine& pl, hipStream_t stream) {
    if (set.count < 1 || set.count > kMaxParts) return hipErrorInvalidValue;
    LineGrid f{};
    int64_t cells = 0;
    for (int p = 0; p < set.count; ++p) {
        if (set.n[p] < kPropLineMin) return hipErrorInvalidValue;
        const int64_t wg = propline_wgs(set.n[p]);
        if (f.first[p] + wg >= (int64_t(1) << 24)) return hipErrorInvalidValue;
        f.first[p + 1] = f.first[p] + (uint32_t)wg;
        f.per = std::max(f.per, (uint32_t)wg);
        cells += set.n[p];
    }
    const dim3 grid(f.first[set.count]), block(256);
#define HX_LINE_CASE(N, nt, ...)                                                              \
    case N:                                                                                   \
        if (nt) hipLaunchKernelGGL((k_prop1d_line<N, true>), grid, block, 0, stream, __VA_ARGS__); \
        else hipLaunchKernelGGL((k_prop1d_line<N, false>), grid, block, 0, stream, __VA_ARGS__);   \
        break;
    HX_LINE_SWITCH(pl.H, cells >= kNtCells, set, pl, f)
#undef HX_LINE_CASE
    return hipGetLastError();
}

hipError_t launch_propline_batch(const LineSeg* segs_dev, const uint32_t* wg_seg_dev, int64_t nwg,
                                 int64_t cells, int H, hipStream_t stream) {
    if (nwg < 1 || nwg >= (int64_t(1) << 24)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg), block(256);
#define HX_LINE_CASE(N, nt, ...)                                                              \
    case N:                                                                                   \
        if (nt) hipLaunchKernelGGL((k_prop1d_segs<N, true>), grid, block, 0, stream, __VA_ARGS__); \
        else hipLaunchKernelGGL((k_prop1d_segs<N, false>), grid, block, 0, stream, __VA_ARGS__);   \
        break;
    HX_LINE_SWITCH(H, cells >= kNtCells, segs_dev, wg_seg_dev)
#undef HX_LINE_CASE
    return hipGetLastError();
}
#undef HX_LINE_SWITCH

}  // namespace hx
