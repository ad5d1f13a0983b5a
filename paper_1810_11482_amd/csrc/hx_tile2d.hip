// Tile form of the 2D band pass, for gfx950: the grids that are too small to
// fill the device with streaming waves (hx_stencil2d.hpp).
//
// A streaming wave walks its rows one after another and a row climbs D levels
// one after another, so a pass over a small grid is one long serial chain on
// a few waves (a 1024 x 1024 pass of eight steps took 199 us on 20 waves).
// Here a workgroup of W waves holds a tile of 256 columns x W R rows in
// registers: lane l of wave w the cells of columns 4 l .. 4 l + 3 in rows
// w R .. w R + R - 1.  The tile advances all its steps in place; the outer
// `steps` rows and `halo` columns are context, loaded and advanced with the
// rest and not stored, so neighbouring tiles do not communicate.  West and
// east neighbours come from DPP wave shifts, north and south ones from the
// lane's own rows, except the rows next to the wave's block, which the waves
// exchange through LDS once per step: a wave computes and publishes its two
// outer rows first, then its inner rows, so the others rarely wait (one
// barrier per step, the exchange buffers alternating).
//
// The context costs (1 + 2 steps / (W R)) (256 / (256 - 2 halo)) of the work,
// which a grid that leaves most of the chip idle does not notice and a large
// one does: choose_form2d below draws the line.  The arithmetic and its order
// are the streaming form's, so a pass of a given depth has the same bits in
// both.
//
// Bound: 16 vector instructions per four cells and step, at 4 to 8 waves per
// SIMD (38 registers at four rows per wave, 70 at eight; double 60 and 125),
// plus about 5 us per pass to launch, load and store.  Measured per step,
// pass included: 256^2 float 0.83 us (12.4 us per pass of 15 steps; the
// streaming form's best 2.2 us), 1024^2 1.04 us (streaming 2.5), 4096^2 5.0 us
// (6.5), 8192^2 18.0 us (20.0), 16384^2 61.7 us (50.3); 4096^2 double 7.9 us
// (10.7), 16384^2 110 us (118).
#include <algorithm>
#include <cmath>

#include "hx_stencil2d.hpp"

namespace hx {
namespace {

extern __shared__ __attribute__((aligned(16))) unsigned char hx_lds_tile2d[];

template <typename T>
struct TileIO {
    const T* in;
    const T* top;
    const T* bot;
    int64_t nx, ny, hw;
    int64_t x;         // this lane's first column
    int64_t y;         // the wave's first row
    bool top_ghost, bot_ghost;
};

// Row y of the band, or its halo; a zero ghost row gives null.
template <typename T>
__device__ __forceinline__ const T* tile_row(const TileIO<T>& io, int64_t y) {
    if (y < 0) return io.top_ghost && y >= -io.hw ? io.top + (io.hw + y) * io.nx : nullptr;
    if (y < io.ny) return io.in + y * io.nx;
    return io.bot_ghost && y - io.ny < io.hw ? io.bot + (y - io.ny) * io.nx : nullptr;
}

// The lane's four cells of rows y .. y + R - 1; cells outside the band are 0.
// WHOLE: the tile lies inside [0, nx) and its rows exist.
template <typename T, int R, bool WHOLE>
__device__ __forceinline__ void tile_load(const TileIO<T>& io, T (&a)[R][4]) {
    typedef typename V16<T>::u UT;
    constexpr int VN = V16<T>::N;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T* row = tile_row(io, io.y + r);
        if (WHOLE) {
#pragma unroll
            for (int q = 0; q < 4 / VN; ++q) {
                const UT v = *(__attribute__((address_space(1))) const UT*)(row + io.x + q * VN);
#pragma unroll
                for (int e = 0; e < VN; ++e) a[r][q * VN + e] = v[e];
            }
        } else {
            // every load from a clamped address, so that none waits on a branch
            const T* base = row ? row : io.in;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t c = io.x + j;
                const int64_t cc = c < 0 ? 0 : (c >= io.nx ? io.nx - 1 : c);
                const T v = *(__attribute__((address_space(1))) const T*)(base + cc);
                a[r][j] = (row && c == cc) ? v : T(0);
            }
        }
    }
}

// One row: update(c, (n + s) + (w + e)) of the old values.
template <typename T, bool SC>
__device__ __forceinline__ void tile_row_step(const Rate2<T>& rt, const T (&no)[4],
                                              const T (&cn)[4], const T (&so)[4], T (&out)[4]) {
    const T left = dpp_move<DPP_WAVE_SHR1>(cn[3]);
    const T right = dpp_move<DPP_WAVE_SHL1>(cn[0]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const T we = (j > 0 ? cn[j - 1] : left) + (j < 3 ? cn[j + 1] : right);
        const T ns = no[j] + so[j];
        const T t = ns + we;
        out[j] = update<T, SC>(rt, cn[j], t);
    }
}

template <typename T>
__device__ __forceinline__ T* edge_row(int buf, int row) {
    // 2 W edge rows of 256 cells per buffer: wave w's first in row 2 w, its last in 2 w + 1
    const int rows = 2 * (int)(blockDim.x >> 6);
    return reinterpret_cast<T*>(hx_lds_tile2d) + ((buf * rows + row) * 64 + (threadIdx.x & 63)) * 4;
}

template <typename T>
__device__ __forceinline__ void put4(T* p, const T (&v)[4]) {
    typedef typename V16<T>::t VT;
    constexpr int VN = V16<T>::N;
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
    typedef typename V16<T>::t VT;
    constexpr int VN = V16<T>::N;
#pragma unroll
    for (int q = 0; q < 4 / VN; ++q) {
        const VT x = reinterpret_cast<const VT*>(p)[q];
#pragma unroll
        for (int e = 0; e < VN; ++e) v[q * VN + e] = x[e];
    }
}

// Which cells a lane resets to 0 after every step (EDGE tiles): columns
// outside [0, nx), rows past a zero-Dirichlet end.
template <int R, bool EDGE>
struct TileMask {
    bool col[4];
    bool row[R];
};
template <int R>
struct TileMask<R, false> {};

template <typename T, int R, bool EDGE>
__device__ __forceinline__ void tile_mask(const TileMask<R, EDGE>& m, int r, T (&v)[4]) {
    if constexpr (EDGE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (m.row[r] || m.col[j]) ? T(0) : v[j];
    }
}

template <typename T>
__device__ __forceinline__ void scale4(T (&v)[4], T f) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= f;
}

template <typename T, int R, bool EDGE, bool SC>
__device__ __forceinline__ void tile_steps2d(const TileIO<T>& io, const Rate2<T>& rt, int steps,
                                             int w, int W, T (&a)[R][4]) {
    TileMask<R, EDGE> m;
    if constexpr (EDGE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) m.col[j] = io.x + j < 0 || io.x + j >= io.nx;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t y = io.y + r;
            m.row[r] = (y < 0 && !io.top_ghost) || (y >= io.ny && !io.bot_ghost);
        }
    }
    put4(edge_row<T>(0, 2 * w), a[0]);
    put4(edge_row<T>(0, 2 * w + 1), a[R - 1]);
    __syncthreads();
    // after step t the tile's outer t + 1 rows are stale: a wave whose rows
    // all are has nothing left to do
    const int alive = (w + 1) * R < (W - w) * R ? (w + 1) * R : (W - w) * R;
    T f = T(1);            // the factor of a rescaling step
    bool scaled = false;   // the last step rescaled
    for (int t = 0; t < steps; ++t) {
        if (t + 1 < alive) {
            // Buffer t & 1 holds the rows just outside the wave's block, as
            // the last step left them before its rescale.  The tile's first
            // and last wave have none (their outer rows are stale context).
            T up[4], dn[4];
            get4(edge_row<T>(t & 1, w > 0 ? 2 * w - 1 : 0), up);
            get4(edge_row<T>(t & 1, w + 1 < W ? 2 * w + 2 : 2 * w + 1), dn);
            if (SC && scaled) {
                scale4(up, f);
                scale4(dn, f);
            }
            T first[4], last[4];
            tile_row_step<T, SC>(rt, up, a[0], a[1], first);
            tile_row_step<T, SC>(rt, a[R - 2], a[R - 1], dn, last);
            tile_mask<T>(m, 0, first);
            tile_mask<T>(m, R - 1, last);
            put4(edge_row<T>((t + 1) & 1, 2 * w), first);
            put4(edge_row<T>((t + 1) & 1, 2 * w + 1), last);
            T prev[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) prev[j] = a[0][j];
#pragma unroll
            for (int r = 1; r + 1 < R; ++r) {
                T old[4], v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) old[j] = a[r][j];
                tile_row_step<T, SC>(rt, prev, old, a[r + 1], v);
                tile_mask<T>(m, r, v);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[r][j] = v[j];
                    prev[j] = old[j];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[0][j] = first[j];
                a[R - 1][j] = last[j];
            }
            scaled = SC && ((rt.mask >> t) & 1u);
            if (scaled) {
                f = t + 1 == steps && rt.tail ? rt.arem : rt.ap;
#pragma unroll
                for (int r = 0; r < R; ++r) scale4(a[r], f);
            }
        }
        // buffer (t + 1) & 1 was last read in step t - 1, before that step's
        // barrier; its new rows are read after this one
        __syncthreads();
    }
}

template <typename T, int R, bool RAG, bool SC>
__global__ __launch_bounds__(R == 4 ? 1024 : 512) void k_tile2d(BandSet set, int steps, int halo, int64_t nstrips) {
    typedef typename V16<T>::t VT;
    constexpr int VN = V16<T>::N;
    const int W = blockDim.x >> 6;
    const int64_t tile = xcd_block2d(blockIdx.x, gridDim.x);
    int kb = 0;
    while (kb + 1 < set.n && tile >= set.first[kb + 1]) ++kb;
    const Band2D& b = set.b[kb];
    const int64_t tl = tile - set.first[kb];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t xb = (tl % nstrips) * (256 - 2 * halo) - halo;  // the tile's first column
    const int64_t yb = (tl / nstrips) * (W * R - 2 * steps) - steps;  // and first row
    TileIO<T> io;
    io.in = static_cast<const T*>(b.in);
    io.top = static_cast<const T*>(b.halo_top);
    io.bot = static_cast<const T*>(b.halo_bot);
    io.nx = b.nx;
    io.ny = b.ny;
    io.hw = b.hw;
    io.x = xb + 4 * lane;
    io.y = yb + (int64_t)w * R;
    io.top_ghost = b.bc_top == BC_GHOST;
    io.bot_ghost = b.bc_bot == BC_GHOST;
    const Rate2<T> rt = make_rate<T, SC>(b, steps);
    const bool xin = xb >= 0 && xb + 256 <= b.nx;
    const bool whole = xin && yb >= 0 && yb + (int64_t)W * R <= b.ny;
    T a[R][4];
    if (whole) {
        tile_load<T, R, true>(io, a);
        tile_steps2d<T, R, false, SC>(io, rt, steps, w, W, a);
    } else {
        tile_load<T, R, false>(io, a);
        tile_steps2d<T, R, true, SC>(io, rt, steps, w, W, a);
    }
    const int64_t y0 = yb + steps;
    const int64_t y1 = yb + (int64_t)W * R - steps < b.ny ? yb + (int64_t)W * R - steps : b.ny;
    const int lc = 4 * lane;
    typedef __attribute__((address_space(1))) T GT;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t y = io.y + r;
        if (y < y0 || y >= y1) continue;
        GT* row = (GT*)(static_cast<T*>(b.out) + y * b.nx + io.x);
        if (RAG) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (lc + j >= halo && lc + j < 256 - halo && io.x + j >= 0 && io.x + j < b.nx)
                    row[j] = a[r][j];
        } else {
            typedef typename V16<T>::u UT;
#pragma unroll
            for (int q = 0; q < 4 / VN; ++q) {
                const int c = lc + q * VN;
                if (c >= halo && c < 256 - halo && io.x + q * VN >= 0 && io.x + q * VN < b.nx) {
                    VT x;
#pragma unroll
                    for (int e = 0; e < VN; ++e) x[e] = a[r][q * VN + e];
                    *(__attribute__((address_space(1))) UT*)(row + q * VN) = x;
                }
            }
        }
    }
}

template <typename T, int R>
hipError_t launch_tile_r(const BandSet& set, int64_t tiles, bool sc, bool rag, const Geom2D& g,
                         int64_t nstrips, hipStream_t st) {
    const dim3 block(64 * g.wpg), grid((unsigned)tiles);
    const size_t sh = (size_t)4 * g.wpg * 256 * sizeof(T);  // 2 buffers of 2 rows per wave
    if (sc && !rag)
        hipLaunchKernelGGL((k_tile2d<T, R, false, true>), grid, block, sh, st, set, g.steps,
                           g.halo, nstrips);
    else if (sc)
        hipLaunchKernelGGL((k_tile2d<T, R, true, true>), grid, block, sh, st, set, g.steps, g.halo,
                           nstrips);
    else if (!rag)
        hipLaunchKernelGGL((k_tile2d<T, R, false, false>), grid, block, sh, st, set, g.steps,
                           g.halo, nstrips);
    else
        hipLaunchKernelGGL((k_tile2d<T, R, true, false>), grid, block, sh, st, set, g.steps,
                           g.halo, nstrips);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tile_t(const Band2D* bands, int n, const Geom2D& g, hipStream_t st) {
    constexpr int VN = V16<T>::N;
    const int64_t wout = 256 - 2 * g.halo, hout = (int64_t)g.wpg * g.rows - 2 * g.steps;
    const int64_t nx = bands[0].nx, nstrips = (nx + wout - 1) / wout;
    BandSet set{};
    set.n = n;
    bool sc = true;
    int64_t total = 0;
    for (int k = 0; k < n; ++k) {
        Band2D bb = bands[k];
        set_rate_2d(bb, g.steps);
        sc = sc && bb.period > 0;
        set.b[k] = bb;
        set.first[k] = total;
        total += nstrips * ((bb.ny + hout - 1) / hout);
    }
    set.first[n] = total;
    if (total >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const bool rag = nx % VN != 0;
    return g.rows == 8 ? launch_tile_r<T, 8>(set, total, sc, rag, g, nstrips, st)
                       : launch_tile_r<T, 4>(set, total, sc, rag, g, nstrips, st);
}

}  // namespace

hipError_t launch_tile2d_bands(int dtype, const Band2D* b, int n, const Geom2D& g,
                               hipStream_t stream) {
    if (n < 1 || n > kMaxBands || g.wpg < 2 || (g.rows != 4 && g.rows != 8) ||
        g.wpg > (g.rows == 4 ? 16 : 8) ||
        g.steps < 1 || g.steps > 31 || 2 * g.steps >= g.wpg * g.rows || g.halo < g.steps ||
        g.halo >= 128)
        return hipErrorInvalidValue;
    for (int k = 1; k < n; ++k)
        if (b[k].nx != b[0].nx) return hipErrorInvalidValue;
    return dtype == 0 ? launch_tile_t<float>(b, n, g, stream)
                      : launch_tile_t<double>(b, n, g, stream);
}

namespace {

// Modelled time of one tile pass, us: a + max(D l, D g i + g m) with g the
// workgroups per CU (counted up to whole ones while they are few), l a lone
// workgroup's step, i a step's share of a full CU and m a tile's loads and
// stores.  Fitted to passes of 4 to 24 steps over 22 grids from 128^2 to
// 16384^2 (mean deviation 4-7 %); over those grids the form and depth it picks
// are within 1 % of the best in all but six, within 24 % in the worst.
struct TileCost {
    int rows, wpg;
    double a, l, i, m;
};
constexpr TileCost kTileCost[2][3] = {
    {{4, 8, 7.83, 0.285, 0.094, 1.88}, {4, 16, 8.52, 0.598, 0.523, 4.89},
     {8, 8, 13.0, 0.539, 0.307, 3.33}},
    {{4, 8, 8.86, 0.383, 0.131, 3.69}, {4, 16, 10.7, 0.855, 0.555, 10.4},
     {8, 8, 13.9, 0.822, 0.364, 7.80}}};

int halo2d(int dtype, int depth) {
    const int vn = dtype ? 2 : 4;
    return (depth + vn - 1) / vn * vn;
}

double tile_us(const TileCost& c, int64_t tiles, int depth) {
    double g = (double)tiles / 256.0;
    if (g > 1.0 && g < 4.0) g = 0.5 * (g + std::ceil(g - 0.05));
    return c.a + std::max(depth * c.l, depth * g * c.i + g * c.m);
}

// From this many float cells on, the streaming form's smaller redundancy wins at
// every depth: 10000 x 12000 cells 25.8 us per step against 31.1, 16384^2 50.3
// against 61.7.  (The two sides of the line are modelled apart: here by the times
// of one aligned grid, without terms for bands or ragged rows.)
constexpr double kStreamCells = 1.0e8;

constexpr int kTileMax = 24;  // deepest tile pass considered

// Below that, and in double, the streaming form takes passes of up to 8 steps
// (float: 10, too) where it is modelled faster, with few rows per wave (16, 24
// or 32, at 10 steps up to 64: more waves and shorter chains against up to a
// doubling of the work).  t = a + max(S (l0 +
// D l), q (S m + (rows + D) D i), bytes) (1 + rag) + c min(the last two), with
// S = rows + 2 D row steps, w the waves per SIMD and q w rounded up half way
// while it is small, bytes = 2 per cell at bw (1 + h / w).  Fitted to passes of
// 2 to 8 steps over 14 grids from 512^2 to 16384^2, aligned and ragged, whole
// and in bands (mean deviation 7-8 %).  Measured, stream / tile: 4096^2 in 16
// bands, 4 steps, 35 / 42 us float, 55 / 63 double; 9000 x 2300 in 23 bands, 6
// steps, 54 / 69 and 99 / 127; 10001 x 10000, 8 steps, double 398 / 491;
// 2048^2, 4 steps, 20.8 / 17.7; 8192^2, 4 steps, 127 / 119; 5070 x 16192 in 5
// bands, 10 steps, 195 / 226.
struct StreamCost {
    double a, l0, l, m, i, bw, rag, h, c;
};
constexpr StreamCost kStreamCost[2] = {
    {6.70, 0.387, 0.0374, 0.0, 0.0419, 5.12e6, 0.0185, 0.648, 0.21},
    {4.61, 0.421, 0.0411, 0.333, 0.0354, 4.49e6, 0.0426, 0.124, 0.054}};

double stream_us(int dtype, int64_t nx, int64_t waves, double cells, int depth, int rows) {
    const StreamCost& k = kStreamCost[dtype ? 1 : 0];
    const double w = (double)waves / 1024.0, s = rows + 2 * depth;
    const double q = w < 4.0 ? 0.5 * (w + std::ceil(w - 0.02)) : w + 0.3;
    const double comp = q * (s * k.m + (rows + depth) * depth * k.i);
    const double bytes = cells * (dtype ? 16 : 8) / k.bw * (1.0 + k.h / std::max(w, 0.1));
    const double rag = nx % (dtype ? 2 : 4) ? k.rag : 0.0;
    return k.a + std::max(std::max(s * (k.l0 + k.l * depth), comp), bytes) * (1.0 + rag) +
           k.c * std::min(comp, bytes);
}

}  // namespace

Form2D choose_form2d(int dtype, int64_t nx, const int64_t* ny, int n, int depth, double* us) {
    Form2D f{};
    f.g.cpl = 4;
    f.g.steps = depth;
    f.g.halo = halo2d(dtype, depth);
    double cells = 0.0;
    for (int k = 0; k < n; ++k) cells += (double)nx * (double)ny[k];
    if (dtype == 0 && cells >= kStreamCells && stencil2d_supported(dtype, 4, depth)) {
        // 16384^2: 10 steps 509 us at 56 rows per wave and one wave per
        // workgroup (508 at 64 and four), 8 steps 474 us at 32 and four, 12
        // and 16 steps 628 and 799 us at 96 and one; shallow passes are bound
        // by their bytes, and most waves fetch them fastest
        f.tile = false;
        f.g.rows = depth <= 6 ? 24 : (depth <= 8 ? 32 : (depth == 10 ? 56 : 96));
        f.g.wpg = depth <= 8 ? 4 : 1;
        const double step = depth <= 8 ? 2.30e-7 : (depth == 10 ? 2.08e-7 : 2.40e-7);
        *us = cells * std::max(depth * step, 1.6e-6);
        return f;
    }
    f.tile = true;
    const int64_t strips = (nx + 255 - 2 * f.g.halo) / (256 - 2 * f.g.halo);
    *us = 0.0;
    for (const TileCost& c : kTileCost[dtype ? 1 : 0]) {
        const int64_t hout = c.rows * c.wpg - 2 * depth;
        if (hout < 1) continue;
        int64_t tiles = 0;
        for (int k = 0; k < n; ++k) tiles += strips * ((ny[k] + hout - 1) / hout);
        // (in runs of passes the tile form takes 1.2 times the fitted time)
        const double t = 1.2 * tile_us(c, tiles, depth);
        if (*us == 0.0 || t < *us) {
            *us = t;
            f.g.rows = c.rows;
            f.g.wpg = c.wpg;
        }
    }
    static const int kRows[2][3] = {{16, 24, 32}, {24, 32, 64}};
    for (int rows : kRows[depth == 10]) {
        if (depth < 1 || (depth > 8 && depth != 10) || !stencil2d_supported(dtype, 4, depth))
            break;
        int64_t waves = 0;
        for (int k = 0; k < n; ++k) waves += strips * ((ny[k] + rows - 1) / rows);
        const double t = stream_us(dtype, nx, waves, cells, depth, rows);
        if (t < *us) {
            *us = t;
            f.tile = false;
            f.g.rows = rows;
            f.g.wpg = 4;
        }
    }
    return f;
}

std::vector<int> choose_depths2d(int dtype, int64_t nx, int64_t ny, int steps) {
    // np passes as even as they can be, np by the least modelled time
    double us[kTileMax + 1] = {};
    for (int d = 1; d <= std::min(kTileMax, steps); ++d) choose_form2d(dtype, nx, &ny, 1, d, &us[d]);
    int best = 0;
    double best_us = 0.0;
    for (int np = (steps + kTileMax - 1) / kTileMax; np <= (steps + 2) / 3; ++np) {
        const int d = steps / np, more = steps % np;
        const double t = (np - more) * us[d] + (more ? more * us[d + 1] : 0.0);
        if (best == 0 || t < best_us) {
            best = np;
            best_us = t;
        }
    }
    std::vector<int> plan;
    for (int p = 0; p < best; ++p) plan.push_back(steps / best + (p < steps % best ? 1 : 0));
    return plan;
}

}  // namespace hx
