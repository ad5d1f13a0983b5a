// Tile form of the fused variable-coefficient passes, for grids that do not
// fill the chip (gfx950).
//
// The streaming passes (hx_varcoef.hip) take at most four steps each (their
// strips overlap by one lane) and a serial chain of rows per wave: on a small
// grid a pass costs 7 to 11 us whatever its size, and a gradient of T steps has
// about 3 T / 4 of them.  Here a workgroup of W waves holds a tile of 256
// columns x W R rows of the state and of its face conductivities in registers
// and advances it `steps` steps, one barrier per step: a wave's rows exchange
// with their neighbours' through the wave's own registers, west/east by DPP
// wave shifts, and the first and last row of each wave through LDS (two
// buffers in turn).  The outer `steps` rows and `halo` columns go stale and are
// not stored.
//
// The face conductivities are formed once per pass.  Cells outside the domain
// hold state 0 (reset after every step) and the conductivity of the nearest
// cell inside, so every domain edge face comes out as (kappa + kappa) / 2 =
// kappa, the single step's edge rule.  The arithmetic and its order are the
// single step's: the same bits as `steps` single steps.
//
// MID stores the state after every step (the states the backward sweep reads).
// ADJ advances lam and takes each step's gradient terms from u_t, whose rows
// are read per step (L2: a segment's states of a small grid stay there); the
// accumulator stays in registers for the whole pass.  u_t's rows of the next
// step arrive while this one's update runs.
//
// Bound: vector issue (float: 9 operations per cell and step, 26 with the
// gradient) at two to four waves per SIMD, and about 5 us per pass to launch,
// load and store.  Three rows per wave in the adjoint of doubles: four spill
// 150 of the 256 registers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <limits>
#include <vector>

#include "hx_internal.h"

namespace hx {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef f64x2 f64x2u __attribute__((aligned(8)));
template <typename T> struct Vec;
template <> struct Vec<float> { typedef f32x4 t; typedef f32x4u u; enum { N = 4 }; };
template <> struct Vec<double> { typedef f64x2 t; typedef f64x2u u; enum { N = 2 }; };

constexpr int DPP_WAVE_SHL1 = 0x130;
constexpr int DPP_WAVE_SHR1 = 0x138;

template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

constexpr int64_t kTilesMax = int64_t(1) << 22;  // workgroups of a launch

extern __shared__ __attribute__((aligned(16))) unsigned char hx_lds_vctile[];

struct VCTile {
    const void* f;      // forward: u; adjoint: lam
    const void* kappa;
    void* out;          // the state after the last step
    void* mid;          // MID: the states after steps 1 .. steps - 1, `stride` bytes apart
    int64_t stride;
    const void* us[kVcTileMax];  // ADJ: u_t of each step
    void* gacc;                  // ADJ: the accumulator (not read when zin; not stored when
    double* total;               // total is given: added there instead, or to zero: fresh)
    int zin, fresh;
    int64_t nx, ny;
    double dt;
    int steps, halo;
    int64_t nstrips;
};

// A lane's four columns and its wave's rows.
struct Place {
    int64_t nx, ny, x, y;
    bool whole;     // the tile lies inside the domain
    bool store[4];  // columns the lane stores
    int64_t xu;     // load_u's column, and by how many cells it lies before x
    int shift;      // (a straddling lane's; else 0)
};

// Four cells of row y (clamped into the grid) at the lane's columns (clamped).
template <typename T>
__device__ __forceinline__ void load4(const T* f, const Place& p, int64_t y, T (&v)[4]) {
    typedef typename Vec<T>::u UT;
    constexpr int VN = Vec<T>::N;
    const int64_t yc = y < 0 ? 0 : (y >= p.ny ? p.ny - 1 : y);
    const T* row = f + yc * p.nx;
    if (p.whole) {
#pragma unroll
        for (int q = 0; q < 4 / VN; ++q) {
            const UT a = *(__attribute__((address_space(1))) const UT*)(row + p.x + q * VN);
#pragma unroll
            for (int e = 0; e < VN; ++e) v[q * VN + e] = a[e];
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t c = p.x + j;
            v[j] = *(__attribute__((address_space(1))) const T*)(
                row + (c < 0 ? 0 : (c >= p.nx ? p.nx - 1 : c)));
        }
    }
}

// The same of u_t, once per row and step: one load per lane.  Cells outside the
// domain are any value of the row; a lane that straddles the row's end (nx not
// a multiple of 4) loads the row's last four cells and shifts them down.
template <typename T, bool EDGE>
__device__ __forceinline__ void load_u(const T* f, const Place& p, int64_t y, T (&v)[4]) {
    typedef typename Vec<T>::u UT;
    constexpr int VN = Vec<T>::N;
    if (EDGE && p.nx < 4) {
        load4<T>(f, p, y, v);
        return;
    }
    const int64_t yc = !EDGE ? y : (y < 0 ? 0 : (y >= p.ny ? p.ny - 1 : y));
    const T* row = f + yc * p.nx + (EDGE ? p.xu : p.x);
#pragma unroll
    for (int q = 0; q < 4 / VN; ++q) {
        const UT a = *(__attribute__((address_space(1))) const UT*)(row + q * VN);
#pragma unroll
        for (int e = 0; e < VN; ++e) v[q * VN + e] = a[e];
    }
    if constexpr (EDGE) {
        if (p.shift > 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const bool s = k < p.shift;
#pragma unroll
                for (int j = 0; j < 3; ++j) v[j] = s ? v[j + 1] : v[j];
            }
        }
    }
}

template <typename T>
__device__ __forceinline__ void store4(T* f, const Place& p, int64_t y, const T (&v)[4]) {
    typedef typename Vec<T>::u UT;
    constexpr int VN = Vec<T>::N;
    T* row = f + y * p.nx + p.x;
    if (p.store[0] && p.store[3]) {
#pragma unroll
        for (int q = 0; q < 4 / VN; ++q) {
            UT a;
#pragma unroll
            for (int e = 0; e < VN; ++e) a[e] = v[q * VN + e];
            *(__attribute__((address_space(1))) UT*)(row + q * VN) = a;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (p.store[j]) *(__attribute__((address_space(1))) T*)(row + j) = v[j];
    }
}

template <typename T>
__device__ __forceinline__ T* edge_row(int buf, int row) {
    // 2 W edge rows of 256 cells per buffer: wave w's first in row 2 w, its last in 2 w + 1
    const int rows = 2 * (int)(blockDim.x >> 6);
    return reinterpret_cast<T*>(hx_lds_vctile) + ((buf * rows + row) * 64 + (threadIdx.x & 63)) * 4;
}

template <typename T>
__device__ __forceinline__ void put4(T* p, const T (&v)[4]) {
    typedef typename Vec<T>::t VT;
    constexpr int VN = Vec<T>::N;
#pragma unroll
    for (int q = 0; q < 4 / VN; ++q) {
        VT x;
#pragma unroll
        for (int e = 0; e < VN; ++e) x[e] = v[q * VN + e];
        reinterpret_cast<VT*>(p)[q] = x;
    }
}

template <typename T>
__device__ __forceinline__ void get4(const T* p, T (&v)[4]) {
    typedef typename Vec<T>::t VT;
    constexpr int VN = Vec<T>::N;
#pragma unroll
    for (int q = 0; q < 4 / VN; ++q) {
        const VT x = reinterpret_cast<const VT*>(p)[q];
#pragma unroll
        for (int e = 0; e < VN; ++e) v[q * VN + e] = x[e];
    }
}

// One row of one step: fc + dt * sum of face * (neighbour - fc) in the single
// step's order (west, east, north, south).  fe: the cells' east faces, fw: cell
// 0's west face.
template <typename T>
__device__ __forceinline__ void row_step(T dt, const T (&no)[4], const T (&c)[4], const T (&so)[4],
                                         const T (&fe)[4], T fw, const T (&fn)[4],
                                         const T (&fs)[4], T (&out)[4]) {
    const T left = dpp_move<DPP_WAVE_SHR1>(c[3]);
    const T right = dpp_move<DPP_WAVE_SHL1>(c[0]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        T a = (j > 0 ? fe[j - 1] : fw) * ((j > 0 ? c[j - 1] : left) - c[j]);
        a = fmaT(fe[j], (j < 3 ? c[j + 1] : right) - c[j], a);
        a = fmaT(fn[j], no[j] - c[j], a);
        a = fmaT(fs[j], so[j] - c[j], a);
        out[j] = fmaT(dt, a, c[j]);
    }
}

// One row of one step's gradient terms, from u_t and lam_{t+1}, into g.
template <typename T, bool EDGE>
__device__ __forceinline__ void row_grad(T dt, const Place& p, int64_t y, const T (&un)[4],
                                         const T (&u)[4], const T (&us)[4], const T (&ln)[4],
                                         const T (&l)[4], const T (&ls)[4], T (&g)[4]) {
    const T ul = dpp_move<DPP_WAVE_SHR1>(u[3]), ur = dpp_move<DPP_WAVE_SHL1>(u[0]);
    const T ll = dpp_move<DPP_WAVE_SHR1>(l[3]), lr = dpp_move<DPP_WAVE_SHL1>(l[0]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const T uc = u[j], lc = l[j];
        T hw = ((j > 0 ? u[j - 1] : ul) - uc) * ((j > 0 ? l[j - 1] : ll) - lc) * T(0.5);
        T he = ((j < 3 ? u[j + 1] : ur) - uc) * ((j < 3 ? l[j + 1] : lr) - lc) * T(0.5);
        T hn = (un[j] - uc) * (ln[j] - lc) * T(0.5);
        T hs = (us[j] - uc) * (ls[j] - lc) * T(0.5);
        if constexpr (EDGE) {
            const T prod = uc * lc;
            hw = p.x + j == 0 ? prod : hw;
            he = p.x + j == p.nx - 1 ? prod : he;
            hn = y == 0 ? prod : hn;
            hs = y == p.ny - 1 ? prod : hs;
        }
        g[j] = fmaT(-dt, (hw + he) + (hn + hs), g[j]);
    }
}

// Cells outside the domain back to the ghost value 0 (EDGE).
template <typename T, bool EDGE>
__device__ __forceinline__ void ghost(const Place& p, int64_t y, T (&v)[4]) {
    if constexpr (EDGE) {
        const bool out = y < 0 || y >= p.ny;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool o = out | (p.x + j < 0) | (p.x + j >= p.nx);
            v[j] = o ? T(0) : v[j];
        }
    }
}

template <typename T, int R, bool ADJ, bool MID, bool EDGE>
__device__ __forceinline__ void tile_run(const VCTile& a, const Place& p, int64_t y0, int64_t y1,
                                         int w, int W) {
    const T dt = static_cast<T>(a.dt);
    // state, east faces, cell 0's west face, south faces (row 0: north, too)
    T f[R][4], fe[R][4], fw[R], fs[R + 1][4];
    {
        const T* F = static_cast<const T*>(a.f);
        const T* K = static_cast<const T*>(a.kappa);
        T kn[4], k[4];
        load4<T>(K, p, p.y - 1, kn);
#pragma unroll
        for (int r = 0; r <= R; ++r) {
            load4<T>(K, p, p.y + r, k);
#pragma unroll
            for (int j = 0; j < 4; ++j) fs[r][j] = (kn[j] + k[j]) * T(0.5);
            if (r < R) {
                load4<T>(F, p, p.y + r, f[r < R ? r : 0]);
                const T kl = dpp_move<DPP_WAVE_SHR1>(k[3]), kr = dpp_move<DPP_WAVE_SHL1>(k[0]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    fe[r < R ? r : 0][j] = (k[j] + (j < 3 ? k[j + 1] : kr)) * T(0.5);
                fw[r < R ? r : 0] = (kl + k[0]) * T(0.5);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) kn[j] = k[j];
        }
    }
    // fs[r] is the face north of row r, fs[r + 1] the one south of it
#pragma unroll
    for (int r = 0; r < R; ++r) ghost<T, EDGE>(p, p.y + r, f[r]);
    T g[ADJ ? R : 1][4];
    if constexpr (ADJ) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t y = p.y + r;
            if (a.zin || y < y0 || y >= y1) {
#pragma unroll
                for (int j = 0; j < 4; ++j) g[r][j] = T(0);
            } else {
                load4<T>(static_cast<const T*>(a.gacc), p, y, g[r]);
            }
        }
    }
    // ADJ: u_t's rows p.y - 1 .. p.y + R
    T ub[ADJ ? R + 2 : 1][4];
    auto load_ub = [&](int t) {
        const T* U = static_cast<const T*>(a.us[t]);
#pragma unroll
        for (int r = 0; r < (ADJ ? R + 2 : 0); ++r) load_u<T, EDGE>(U, p, p.y - 1 + r, ub[r]);
    };
    if constexpr (ADJ) load_ub(0);
    put4(edge_row<T>(0, 2 * w), f[0]);
    put4(edge_row<T>(0, 2 * w + 1), f[R - 1]);
    __syncthreads();
    // after step t the tile's outer t + 1 rows are stale: a wave whose rows all
    // are has nothing left to do
    const int alive = (w + 1) * R < (W - w) * R ? (w + 1) * R : (W - w) * R;
    for (int t = 0; t < a.steps; ++t) {
        if (t + 1 < alive) {
            T up[4], dn[4];
            get4(edge_row<T>(t & 1, w > 0 ? 2 * w - 1 : 0), up);
            get4(edge_row<T>(t & 1, w + 1 < W ? 2 * w + 2 : 2 * w + 1), dn);
            if constexpr (ADJ) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    row_grad<T, EDGE>(dt, p, p.y + r, ub[r], ub[r + 1], ub[r + 2],
                                      r > 0 ? f[r > 0 ? r - 1 : 0] : up, f[r],
                                      r + 1 < R ? f[r + 1 < R ? r + 1 : 0] : dn, g[r]);
                // the next step's u rows arrive during this step's update
                if (t + 1 < a.steps) load_ub(t + 1);
            }
            T first[4], last[4];
            row_step<T>(dt, up, f[0], f[1], fe[0], fw[0], fs[0], fs[1], first);
            row_step<T>(dt, f[R - 2], f[R - 1], dn, fe[R - 1], fw[R - 1], fs[R - 1], fs[R], last);
            ghost<T, EDGE>(p, p.y, first);
            ghost<T, EDGE>(p, p.y + R - 1, last);
            put4(edge_row<T>((t + 1) & 1, 2 * w), first);
            put4(edge_row<T>((t + 1) & 1, 2 * w + 1), last);
            T prev[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) prev[j] = f[0][j];
#pragma unroll
            for (int r = 1; r + 1 < R; ++r) {
                T old[4], v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) old[j] = f[r][j];
                row_step<T>(dt, prev, old, f[r + 1], fe[r], fw[r], fs[r], fs[r + 1], v);
                ghost<T, EDGE>(p, p.y + r, v);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f[r][j] = v[j];
                    prev[j] = old[j];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f[0][j] = first[j];
                f[R - 1][j] = last[j];
            }
            if (MID && t + 1 < a.steps) {
                T* m = reinterpret_cast<T*>(static_cast<char*>(a.mid) + t * a.stride);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (p.y + r >= y0 && p.y + r < y1) store4<T>(m, p, p.y + r, f[r]);
            }
        }
        // buffer (t + 1) & 1 was last read in step t - 1, before that step's
        // barrier; its new rows are read after this one
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t y = p.y + r;
        if (y < y0 || y >= y1) continue;
        store4<T>(static_cast<T*>(a.out), p, y, f[r]);
        if constexpr (ADJ) {
            if (a.total) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (p.store[j]) {
                        double* tp = a.total + y * p.nx + p.x + j;
                        *tp = (a.fresh ? 0.0 : *tp) + (double)g[r][j];
                    }
            } else {
                store4<T>(static_cast<T*>(a.gacc), p, y, g[r]);
            }
        }
    }
}

template <typename T, int R, int WMAX, bool ADJ, bool MID>
__global__ __launch_bounds__(64 * WMAX) void k_vc_tile(VCTile a) {
    const int W = blockDim.x >> 6;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t xb = (int64_t)(blockIdx.x % a.nstrips) * (256 - 2 * a.halo) - a.halo;
    const int64_t yb = (int64_t)(blockIdx.x / a.nstrips) * (W * R - 2 * a.steps) - a.steps;
    Place p;
    p.nx = a.nx;
    p.ny = a.ny;
    p.x = xb + 4 * lane;
    p.y = yb + (int64_t)w * R;
    // (the faces read one row and the gradient one row of u beyond the tile)
    p.whole = xb >= 0 && xb + 256 <= a.nx && yb >= 1 && yb + (int64_t)W * R < a.ny;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        p.store[j] = 4 * lane + j >= a.halo && 4 * lane + j < 256 - a.halo && p.x + j >= 0 &&
                     p.x + j < a.nx;
    p.xu = p.x < 0 ? 0 : (p.x + 4 > a.nx ? a.nx - 4 : p.x);
    p.shift = p.x < a.nx && p.x + 4 > a.nx ? (int)(p.x + 4 - a.nx) : 0;
    const int64_t y0 = yb + a.steps;
    const int64_t ye = yb + (int64_t)W * R - a.steps;
    const int64_t y1 = ye < a.ny ? ye : a.ny;
    if (p.whole)
        tile_run<T, R, ADJ, MID, false>(a, p, y0, y1, w, W);
    else
        tile_run<T, R, ADJ, MID, true>(a, p, y0, y1, w, W);
}

template <typename T, int R, int WMAX, bool ADJ>
hipError_t launch_t(VCTile a, int W, hipStream_t st) {
    if (W < 2 || W > WMAX || a.steps < 1 || a.steps > kVcTileMax || 2 * a.steps >= W * R)
        return hipErrorInvalidValue;
    a.halo = (a.steps + 3) / 4 * 4;
    const int64_t wout = 256 - 2 * a.halo, hout = (int64_t)W * R - 2 * a.steps;
    a.nstrips = (a.nx + wout - 1) / wout;
    const int64_t tiles = a.nstrips * ((a.ny + hout - 1) / hout);
    if (tiles >= kTilesMax) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(64 * W);
    const size_t sh = (size_t)4 * W * 256 * sizeof(T);  // 2 buffers of 2 rows per wave
    if (!ADJ && a.mid)
        hipLaunchKernelGGL((k_vc_tile<T, R, WMAX, false, true>), grid, block, sh, st, a);
    else
        hipLaunchKernelGGL((k_vc_tile<T, R, WMAX, ADJ, false>), grid, block, sh, st, a);
    return hipGetLastError();
}

// Modelled times of a pass of d steps, us, by dtype and kind (forward, MID,
// adjoint).  Tile: a + max(d l, d g i + g m), g the workgroups per CU (counted
// up half way to whole ones while they are few).  Streaming: max((a + l d) k, b
// + (c (m + i d) + h max(0, c - 20)) k), c the cells in millions, k = 1 + x
// where nx is no multiple of 4.  Fitted to 17 grids from 64^2 to 8192^2 (mean
// deviation 6-13 %).  Measured per step at the best depth, streaming / tile,
// float: 300^2 forward 2.0 / 1.2 us, recompute 2.4 / 1.5, adjoint 4.0 / 2.7;
// 777 x 1001 3.7 / 1.6, 4.6 / 2.1, 8.2 / 4.6; 2048^2 5.7 / 3.3, 6.5 / 4.6, 11.1
// / 13.7; 8192^2 forward 40 / 34, recompute 93 / 67; double: 777 x 1001 4.1 /
// 1.7, 5.2 / 2.6, 16.4 / 7.2.
struct TileCost {
    int waves;
    double a, l, i, m;
};
constexpr TileCost kTile[2][3][3] = {
    {{{12, 9.70, 0.719, 0.424, 4.51}, {8, 8.06, 0.311, 0.204, 2.94}, {4, 5.87, 0.010, 0.009, 1.57}},
     {{12, 8.36, 1.30, 1.07, 6.67}, {8, 7.05, 0.831, 0.488, 4.64}, {4, 5.90, 0.375, 0.150, 1.96}},
     {{8, 10.8, 2.02, 1.56, 10.9}, {4, 9.09, 1.08, 0.507, 5.41}, {0, 0, 0, 0, 0}}},
    {{{8, 4.23, 1.11, 0.539, 7.76}, {4, 3.83, 0.746, 0.046, 2.99}, {0, 0, 0, 0, 0}},
     {{8, 4.47, 1.57, 1.06, 9.36}, {4, 3.00, 1.44, 0.268, 4.09}, {0, 0, 0, 0, 0}},
     {{8, 9.10, 2.66, 1.96, 12.4}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}}}};
struct StreamCost {
    double a, l, m, i, x, b, h;
};
constexpr StreamCost kStream[2][3] = {{{3.93, 1.09, 1.92, 0.230, 0.864, 3.40, 0.0},
                                       {3.47, 1.53, 0.011, 1.27, 0.942, 4.01, 1.75},
                                       {4.62, 2.52, 2.87, 1.89, 1.59, 4.19, 1.39}},
                                      {{3.80, 1.38, 5.01, 0.537, 0.733, 5.17, 0.0},
                                       {3.43, 1.98, 1.95, 2.14, 0.661, 2.36, 1.40},
                                       {4.24, 4.27, 5.60, 2.53, 1.15, 2.63, 2.51}}};

// The form of a pass of d steps (its waves; 0: streaming) and its time.
double pass_us(int dtype, int kind, int64_t nx, int64_t ny, int d, int* waves) {
    const int rows = dtype && kind == 2 ? 3 : 4;
    const int deepest = dtype && kind == 2 ? 2 : kVcFusedMax;
    const double c = 1e-6 * (double)nx * (double)ny;
    const bool rag = nx % 4 != 0;
    double best = std::numeric_limits<double>::infinity();
    *waves = 0;
    if (d <= deepest) {
        const StreamCost& k = kStream[dtype ? 1 : 0][kind];
        const double f = 1.0 + (rag ? k.x : 0.0);
        best = std::max((k.a + k.l * d) * f,
                        k.b + (c * (k.m + k.i * d) + k.h * std::max(0.0, c - 20.0)) * f);
    }
    const int halo = (d + 3) / 4 * 4;
    const int64_t strips = (nx + 255 - 2 * halo) / (256 - 2 * halo);
    // (large aligned grids are bound by memory, where the fit says too little)
    const double margin = !rag && c > 12.0 ? 1.2 : 1.05;
    for (const TileCost& k : kTile[dtype ? 1 : 0][kind]) {
        const int64_t hout = k.waves * rows - 2 * d;
        if (d < 2 || d > kVcTileMax || 4 * d > 1.3 * k.waves * rows || hout < 1) continue;
        const int64_t tiles = strips * ((ny + hout - 1) / hout);
        if (tiles >= kTilesMax) continue;
        double g = (double)tiles / 256.0;
        if (g > 1.0 && g < 4.0) g = 0.5 * (g + std::ceil(g - 0.05));
        const double t = margin * (k.a + std::max(d * k.l, d * g * k.i + g * k.m));
        if (t < best) {
            best = t;
            *waves = k.waves;
        }
    }
    return best;
}

}  // namespace

std::vector<VCPass> choose_vc_passes(int dtype, int kind, int64_t nx, int64_t ny, int steps,
                                     bool tiles) {
    // np passes as even as they can be, np by the least modelled time
    std::vector<VCPass> passes;
    if (steps < 1) return passes;
    const int deepest = dtype && kind == 2 ? 2 : kVcFusedMax;
    const int most = (steps + deepest - 1) / deepest;
    double us[kVcTileMax + 1] = {};
    int waves[kVcTileMax + 1] = {};
    int best = most;
    if (tiles) {
        for (int d = 1; d <= kVcTileMax; ++d) us[d] = pass_us(dtype, kind, nx, ny, d, &waves[d]);
        double best_us = std::numeric_limits<double>::infinity();
        for (int np = (steps + kVcTileMax - 1) / kVcTileMax; np <= most; ++np) {
            const int d = steps / np, more = steps % np;
            const double t = (np - more) * us[d] + (more ? more * us[d + 1] : 0.0);
            if (t < best_us) {
                best = np;
                best_us = t;
            }
        }
    }
    for (int j = 0; j < best; ++j) {
        const int d = steps / best + (j < steps % best ? 1 : 0);
        passes.push_back(VCPass{d, waves[d]});
    }
    return passes;
}

hipError_t launch_vc_tile(int dtype, bool adjoint, int steps, int waves, const VCArgs& v,
                          void* mid, int64_t mid_stride, const void* const* ustates, bool zin,
                          double* total, bool fresh, hipStream_t st) {
    VCTile a{};
    a.f = adjoint ? v.lam : v.u;
    a.kappa = v.kappa;
    a.out = v.out;
    a.mid = mid;
    a.stride = mid_stride;
    a.gacc = v.gacc;
    a.total = total;
    a.zin = zin ? 1 : 0;
    a.fresh = fresh ? 1 : 0;
    a.nx = v.nx;
    a.ny = v.ny;
    a.dt = v.dt;
    a.steps = steps;
    if (steps < 1 || steps > kVcTileMax || (adjoint && !ustates)) return hipErrorInvalidValue;
    for (int q = 0; adjoint && q < steps; ++q) a.us[q] = ustates[q];
    if (dtype == 0)
        return adjoint ? launch_t<float, 4, 8, true>(a, waves, st)
                       : launch_t<float, 4, 16, false>(a, waves, st);
    return adjoint ? launch_t<double, 3, 8, true>(a, waves, st)
                   : launch_t<double, 4, 8, false>(a, waves, st);
}

}  // namespace hx
