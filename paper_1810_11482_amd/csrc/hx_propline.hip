// Propagator pass over neighbouring partitions of a line (f32), for gfx950:
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
//   * Boundaries.  Blocks near an end take their cells one by one: from the
//     neighbour's cells, or, past a zero-Dirichlet end, from the odd
//     reflection of the line about the ghost cell (u_{-1} = 0, u_{-2-k} =
//     -u_k), which the steps preserve exactly.
//   * Blocks start where `out` is 128-byte aligned, so a block's stores cover
//     whole lines whatever the alignment of the line.
// Bound: HBM (or the last-level cache) for long lines, launch and one block's
// latency for short ones.  Measured, a pass of 20 / 50 / 200 steps: 2^19 cells
// 7.8 / 8.0 / 9.8 us, 2^22 11.7 / 11.9 / 15.5 us, 2^24 28 / 30 / 38 us, 2^26
// 98 / 109 / 135 us (5.5 / 4.9 / 4.0 TB/s); the direct form needs 110 us for
// 200 steps of 12345679 cells, this one 31 us.  At most 85 VGPRs (6 waves per
// SIMD; the stepping path spills 47, which the others do not touch): with 128
// (4 waves) 2^24 cells took 33.5 us in place of 30.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
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
constexpr int kTapHalf = 192;     // split taps of one level sent with a launch
constexpr int kReach = 256;       // deepest pass
// The shallowest pass the library takes in this form.  From here on its error
// against 64 bits is the smaller one on positive noise and on smooth fields at
// every rate measured (r = 1/20 .. 1/4, 12 to 200 steps: 0.46-0.64e-7 against
// 0.56-10e-7), per cell also on noise of both signs.
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

// One partition as a block sees it.
struct Part {
    const float* in;
    float* out;
    int64_t n;
    const float* lo;  // hw cells before the first, or null: a zero-Dirichlet end
    const float* hi;  // hw cells after the last, or null
    int hw;
};

// Cell c of the line: the partition's own, its neighbours' (clamped to what
// they hold: cells further out meet no tap and no check), or the reflection.
__device__ __forceinline__ float line_cell(const Part& s, int64_t c) {
    if (c >= 0 && c < s.n) return s.in[c];
    if (c < 0) {
        if (s.lo) return s.lo[s.hw + c < 0 ? 0 : s.hw + c];
        return c == -1 ? 0.f : -s.in[-c - 2];
    }
    const int64_t k = c - s.n;
    if (s.hi) return s.hi[k >= s.hw ? s.hw - 1 : k];
    return k == 0 ? 0.f : -s.in[s.n - k];
}

__device__ __forceinline__ f32x4 line_cells4(const Part& s, int64_t c, bool inside) {
    if (inside) return *(__attribute__((address_space(1))) const f32x4u*)(s.in + c);
    f32x4 v;
#pragma unroll 1
    for (int e = 0; e < 4; ++e) v[e] = line_cell(s, c + e);
    return v;
}

__device__ __forceinline__ float far4(const f32x4& x) {
    float m = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) m = __builtin_elementwise_maximum(m, fabsf(x[e]));
    return m;
}

// The stepping path of one block: its cells c0 .. c0 + 1023 advanced D steps
// over the window of 256 cells on each side, 24 consecutive cells per lane, in
// the rescaled direct form.
__device__ __forceinline__ void step_line(const Part& s, const Seg1D& rate, int64_t c0, int D) {
    constexpr int K = 24;
    const int l = threadIdx.x & 63;
    const int64_t b = c0 - kReach + (int64_t)K * l;
    float a[K];
#pragma unroll
    for (int t = 0; t < K; ++t) a[t] = line_cell(s, b + t);
    const float beta = (float)rate.beta, ap = (float)rate.alpha_p;
    int since = 0;
    for (int k = 0; k < D; ++k) {
        step_tile_scaled<float, K>(a, beta, false, false, 0, 0);
        if (++since == rate.period) {
            since = 0;
            scale_tile<float, K>(a, ap);
        }
    }
    if (since) scale_tile<float, K>(a, (float)rate.alpha_rem);
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const int64_t c = b + t;
        if (c >= c0 && c < c0 + 1024 && c >= 0 && c < s.n) s.out[c] = a[t];
    }
}

// What a launch needs besides the partitions.
struct LineTaps {
    uint16_t tap[2][kTapHalf];  // level (hi, lo) of tap j = -H - 31 + k, scaled by 2^texp
    uint32_t levels;            // products per window chunk, as prop1d_levels16
    int32_t texp, H, D;
    float chk;                  // 2^21 E 2^texp: the check's threshold per unit of |x| in reach
    uint32_t first[kMaxParts + 1];  // workgroups before partition p
    uint32_t per;                   // the most workgroups a partition has
};

// NT: nontemporal loads of the block's own cells and stores (arrays that do
// not stay in the caches between passes).
template <int NC, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8)))
void k_prop1d_line(PartSet1D ps, LineTaps a, Seg1D rate) {
    constexpr int U = units_of(NC);
    constexpr int kUnits = 16 * U;
    __shared__ __attribute__((aligned(16))) char lds_all[4 * 2 * kPlane + 16 * kUnits];
    __shared__ float wmax[4];
    char* const tl = lds_all + 4 * 2 * kPlane;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const lds = lds_all + wv * 2 * kPlane;
    const int l = threadIdx.x & 63, i = l & 31, g = l >> 5;
    int p = (int)(blockIdx.x / a.per);
    while (blockIdx.x >= a.first[p + 1]) ++p;
    Part s;
    s.in = static_cast<const float*>(ps.in[p]);
    s.out = static_cast<float*>(ps.out[p]);
    s.n = ps.n[p];
    s.hw = a.D;
    s.lo = p > 0 ? static_cast<const float*>(ps.in[p - 1]) + (ps.n[p - 1] - a.D)
                 : static_cast<const float*>(ps.halo_lo);
    s.hi = static_cast<const float*>(p + 1 < ps.count ? ps.in[p + 1] : ps.halo_hi);
    const int shift = (int)((reinterpret_cast<uintptr_t>(s.out) >> 2) & 31);
    const int64_t c0 = 1024 * (4 * (int64_t)(blockIdx.x - a.first[p]) + wv) - shift;
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
            step_line(s, rate, c0, a.D);
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
        o[j] = *reinterpret_cast<const f32x4*>(lds + tpos(8 * j + (l >> 3), l & 7));
    const int64_t oc = c0 + 4 * l;
    if (c0 >= 0 && c0 + 1024 <= s.n) {
        typedef __attribute__((address_space(1))) f32x4 GO;
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
                if (c >= 0 && c < s.n) s.out[c] = o[j][e];
            }
    }
}

// From this many cells on, a pass's arrays (8 bytes per cell) outgrow the
// 256 MB last-level cache and are better streamed past it.
constexpr int64_t kNtCells = int64_t(1) << 25;

// The taps p_j, 0 <= j <= K, of the D-step propagator (p_{-j} = p_j), by the
// downward recurrence (D - j + 1) p_{j-1} = (D + j + 1) p_{j+1} + (a/r) j p_j
// of the coefficients of (r/x + a + r x)^D, a = 1 - 2r, whose terms are all
// positive (no cancellation), normalised to sum 1; K = D, or where the taps
// have fallen below 1e-40 of the largest.
int line_taps(double r, int D, std::vector<double>& p) {
    const double sigma = std::sqrt(2.0 * r * D);
    const int K = std::min(D, (int)(14.0 * sigma) + 20);
    p.assign(K + 2, 0.0);
    p[K] = 1e-280;
    const double q = (1.0 - 2.0 * r) / r;
    for (int j = K; j >= 1; --j)
        p[j - 1] = ((D + j + 1) * p[j + 1] + q * j * p[j]) / (D - j + 1);
    double sum = p[0];
    for (int j = 1; j <= K; ++j) sum += 2.0 * p[j];
    for (double& x : p) x /= sum;
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

bool propline_setup(double r, int D, PropLine* out) {
    // (up to r = 1/4 the taps fall monotonically from p_0)
    if (!(r >= 1e-3 && r <= 0.25) || D < 1 || D > kReach) return false;
    std::vector<double> p;
    const int K = line_taps(r, D, p);
    auto tap = [&](int j) { return std::abs(j) <= K ? p[std::abs(j)] : 0.0; };
    // Everything omitted is kept near the fp16 split's own floors (2^-39 of the
    // window's largest), so that only outputs some 2^-15 of their surroundings
    // or smaller fail the check: the zero crossings of a smooth field mostly
    // pass.  The half window: the least multiple of 8 cells whose outer taps
    // sum to less than 2^-39 (all sum to 1), at most 64.
    std::vector<double> tail(K + 2, 0.0);  // tail[j] = sum of p_k, k >= j
    for (int j = K; j >= 0; --j) tail[j] = tail[j + 1] + p[j];
    auto past = [&](int j) { return j <= K ? tail[std::max(j, 0)] : 0.0; };
    int H = 8;
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
    for (int m = 0; m < 32; ++m) {
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
    std::fill(&out->tap[0][0], &out->tap[0][0] + 2 * kTapHalf, (uint16_t)0);
    // (a tap's rounding is handed on to the next one out, whose lower half is
    // finer, so that the rounded taps still sum to 1: a smooth field meets the
    // sum of the roundings)
    const double scale = std::ldexp(1.0, texp);
    double carry = 0.0;
    for (int j = 0; j <= std::min(K, H + 31); ++j) {
        const double x = p[j] * scale + carry;
        uint16_t hi, lo;
        const float xh = to_half((float)x, &hi), xl = to_half((float)(x - xh), &lo);
        carry = (x - xh - xl) * (j ? 1.0 : 0.5);
        for (int k : {H + 31 + j, H + 31 - j}) {
            if (k >= 8 * units_of(NC) + 8) continue;
            out->tap[0][k] = hi;
            out->tap[1][k] = lo;
        }
    }
    return true;
}

// Fitted to passes of 20 to 200 steps over lines from 2^12 to 2^28 cells
// (deviation at most 9 %).
double propline_us(double r, int64_t cells, int D) {
    const double v = 2.0 * r * D;
    if (!(r >= 1e-3 && r <= 0.25) || D < kPropMinDepth || D > kReach || v > 104.0 ||
        cells < kPropLineMin)
        return std::numeric_limits<double>::infinity();
    const int H = std::min(64, ((int)(7.05 * std::sqrt(v)) + 8) / 8 * 8), NC = 2 + H / 8;
    const double setup = 0.5 + std::min(4.5, 0.028 * D);
    return setup + 6.4 + 0.16 * NC + (D > 64 ? 1.2 : 0.0) +
           1e-6 * (double)cells * (1.19 + 0.03 * NC + (D > 64 ? 0.3 : 0.0));
}

hipError_t launch_propline(const PartSet1D& set, const PropLine& pl, hipStream_t stream) {
    static_assert(sizeof(PropLine::tap) == sizeof(LineTaps::tap), "one table");
    if (set.count < 1 || set.count > kMaxParts) return hipErrorInvalidValue;
    LineTaps a{};
    std::copy(&pl.tap[0][0], &pl.tap[0][0] + 2 * kTapHalf, &a.tap[0][0]);
    a.levels = pl.levels;
    a.texp = pl.texp;
    a.H = pl.H;
    a.D = pl.D;
    a.chk = pl.chk;
    int64_t cells = 0;
    for (int p = 0; p < set.count; ++p) {
        if (set.n[p] < kPropLineMin) return hipErrorInvalidValue;
        const int shift = (int)((reinterpret_cast<uintptr_t>(set.out[p]) >> 2) & 31);
        const int64_t wg = (set.n[p] + shift + 4095) / 4096;
        if (a.first[p] + wg >= (int64_t(1) << 31)) return hipErrorInvalidValue;
        a.first[p + 1] = a.first[p] + (uint32_t)wg;
        a.per = std::max(a.per, (uint32_t)wg);
        cells += set.n[p];
    }
    Seg1D rate{};
    rate.r = set.r;
    set_rate_1d(rate, pl.D);
    const dim3 grid(a.first[set.count]), block(256);
    const bool nt = cells >= kNtCells;
    switch ((32 + 2 * pl.H) / 16) {
#define HX_LINE_CASE(N)                                                                        \
    case N:                                                                                    \
        if (nt)                                                                                \
            hipLaunchKernelGGL((k_prop1d_line<N, true>), grid, block, 0, stream, set, a, rate); \
        else                                                                                   \
            hipLaunchKernelGGL((k_prop1d_line<N, false>), grid, block, 0, stream, set, a, rate); \
        break;
        HX_LINE_CASE(3)
        HX_LINE_CASE(4)
        HX_LINE_CASE(5)
        HX_LINE_CASE(6)
        HX_LINE_CASE(7)
        HX_LINE_CASE(8)
        HX_LINE_CASE(9)
        HX_LINE_CASE(10)
#undef HX_LINE_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace hx
