// 2D explicit five-point heat stencil with temporal blocking, for gfx950: the
// streaming band kernel, instantiated by the hx_stencil2d_*.hip units.
//
// Operation: u'_ij = u_ij + r (u_{i-1,j} + u_{i+1,j} + u_{i,j-1} + u_{i,j+1}
// - 4 u_ij) on a row-major band of ny x nx cells (the Sec. V-A.1 stencil
// extended to a grid), D steps fused per pass, zero-Dirichlet on the left and
// right edges, top and bottom either zero-Dirichlet or supplied by halo rows.
//
// Mapping (2.5D streaming with a register pipeline).  A wave owns a strip of
// 64*C columns (C adjacent columns per lane) and a chunk of R output rows.  It
// streams the strip's input rows from R0 - D to R1 + D - 1 once, top to
// bottom.  Time level k (1..D) keeps the previous two rows it received from
// level k-1 in registers (a three-slot ring per level, rotated by unrolling
// the row loop three times); each new level-(k-1) row lets level k produce the
// row above it.  A row therefore enters from HBM once, climbs all D levels inside
// registers, and leaves to HBM once: a pass costs one read and one write per
// cell plus the 2*D halo rows per chunk and 2*H halo columns per strip, whatever
// D is.  West/east neighbours across lanes come from DPP wave shifts; north and
// south neighbours are the pipeline's own rows, so there is no LDS and no
// barrier.  Outer context columns (H >= D per side) go stale one column per
// level and are never stored.
//
// Per cell-step: t = (n + s) + (w + e), then for 0 <= r <= 7/32 the rescaled
// update w' = fma(r/(1-4r), t, w) (set_rate_2d), otherwise d = fma(-4, c, t);
// c' = fma(r, d, c).  A pass's result depends on its depth only, not on the
// tile geometry.
#pragma once

#include <hip/hip_runtime.h>

#include "hx_internal.h"

namespace hx {
namespace {

enum { BC_PERIODIC = 0, BC_DIRICHLET0 = 1, BC_GHOST = 2 };

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename T> struct V16;
// u: the vector at the alignment of one element (rows may start anywhere)
typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef f64x2 f64x2u __attribute__((aligned(8)));
template <> struct V16<float> { typedef f32x4 t; typedef f32x4u u; enum { N = 4 }; };
template <> struct V16<double> { typedef f64x2 t; typedef f64x2u u; enum { N = 2 }; };

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

// The per-cell update of one level: direct (k = r) or rescaled (SC: b =
// r/(1-4r), and the level's row is multiplied by ap at every rescale level,
// by arem at the last one when the depth is not a multiple of the period;
// `mask` has bit l set for the levels l+1 that rescale).
template <typename T>
struct Rate2 {
    T k, b, ap, arem;
    uint32_t mask;
    bool tail;
};

template <typename T, bool SC>
__device__ __forceinline__ Rate2<T> make_rate(const Band2D& band, int D) {
    Rate2<T> rt;
    rt.k = static_cast<T>(band.r);
    rt.b = static_cast<T>(band.beta);
    rt.ap = static_cast<T>(band.alpha_p);
    rt.arem = static_cast<T>(band.alpha_rem);
    rt.mask = 0;
    rt.tail = false;
    if constexpr (SC) {
        const int p = band.period;
        for (int l = 0; l < D; ++l)
            if ((l + 1) % p == 0) rt.mask |= 1u << l;
        rt.tail = (D % p) != 0;
        if (rt.tail) rt.mask |= 1u << (D - 1);
    }
    return rt;
}

template <typename T, bool SC>
__device__ __forceinline__ T update(const Rate2<T>& rt, T c, T t) {
    if constexpr (SC) {
        return fmaT(rt.b, t, c);
    } else {
        const T d = fmaT(T(-4), c, t);
        return fmaT(rt.k, d, c);
    }
}

template <typename T, int C, int D, bool SC>
__device__ __forceinline__ void rescale_level(const Rate2<T>& rt, int l, T* v) {
    if constexpr (SC) {
        if ((rt.mask >> l) & 1u) {
            const T f = (l + 1 == D && rt.tail) ? rt.arem : rt.ap;
#pragma unroll
            for (int j = 0; j < C; ++j) v[j] *= f;
        }
    }
}

// Level-0 rows live in a ring of Q rows (Q a multiple of 3): rows yy-2 .. yy
// are the pipeline's input window and rows yy+1 .. yy+Q-3 are loads in flight,
// so Q-3 rows are prefetched ahead of their use.  Row y sits in slot
// (y - ystart) mod Q.
constexpr int ring_rows() { return 6; }

// Memory side of a wave.  Every row step issues the same loads (the prefetch;
// rows past the chunk are clamped to its last row) and, once the pipeline is
// full, the same stores, so no memory operation sits under a branch or an exec
// mask, the compiler's wait counts cover only the row being consumed, and Q-3
// rows stay in flight behind the arithmetic.  A row's address is a
// wave-uniform base (the row at the strip's first column) plus a 32-bit lane
// offset.  Stores go through a buffer resource over the strip's part of the
// row; lanes that must not store (halo columns, columns past nx) use an
// out-of-range offset, which the hardware drops.
//
// Vectors are loaded and stored with the alignment of one element, so rows may
// start anywhere: the hardware takes them, at the cost of one more line per
// kilobyte.
//
// EDGE waves (a strip reaching past [0, nx), or rows that are zero-Dirichlet
// ghosts) run the same code plus selects: zero rows and columns outside
// [0, nx) are loaded from a valid clamped address and replaced by 0, and every
// level re-zeroes them.  RAG (nx not a multiple of the vector width): a lane's
// vector may straddle the end of a row, so EDGE waves load and store cell by
// cell; the other waves are unchanged.
template <typename T, int C>
struct FastIO {
    const T* in;                        // rows 0 of the band, of its top and bottom halo rows,
    const T* top;                       // at the strip's first column
    const T* bot;
    int64_t nx, ny, hw;
    int64_t ylo, yhi;                   // clamp range of level-0 rows
    bool top_ghost, bot_ghost;          // top/bottom rows come from halo buffers
    int out_bytes;                      // bytes of a row from column xb to the strip's end or nx
    uint32_t xload[C];                  // byte offset of each vector's (RAG EDGE: cell's) load
    uint32_t off[C];                    // byte offset of its store, or out of range
    uint32_t col[C];                    // all ones if the cell lies inside [0, nx), else 0 (not
                                        // RAG: of each vector's first cell)
};

// x where m is all ones, 0 where it is 0: nothing (unlike a select on a
// condition) the compiler turns into a branch around each cell's step or, for
// a zero row, around its load and the wait for it, which made a RAG edge row
// 1.5 times as slow and a whole 4096^2 pass in double by a fifth.
__device__ __forceinline__ float keep(float x, uint32_t m) {
    return __uint_as_float(__float_as_uint(x) & m);
}
__device__ __forceinline__ double keep(double x, uint32_t m) {
    return __hiloint2double(__double2hiint(x) & (int)m, __double2loint(x) & (int)m);
}

// Where the branches are cheaper all the same: the straight-line edge code of
// eight float levels needs 137 registers, three waves per SIMD in place of four
// for the interior waves, too (16384^2 at 32 rows per wave: 512 us against 474;
// eight columns per lane 256 registers, 10 % slower).  Ten and more levels run
// at the same waves per SIMD either way, and 2 to 6 % faster without branches.
template <typename T, int C, int D, bool RAG>
constexpr bool kEdgeBranch = sizeof(T) == 4 && D == 8 && !RAG;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int BUF_DWORD3 = 0x00020000;  // raw 32-bit buffer (gfx9 family)
constexpr uint32_t OOB_OFFSET = 0x7ffffff0u;

// Row y is a zero ghost: outside the band on a zero-Dirichlet side, or past
// the supplied halo rows.
template <typename T, int C>
__device__ __forceinline__ bool zero_row_fast(const FastIO<T, C>& io, int64_t y) {
    return (y < 0 && (!io.top_ghost || y < -io.hw)) ||
           (y >= io.ny && (!io.bot_ghost || y >= io.ny + io.hw));
}

template <typename T, int C, int D, bool EDGE, bool RAG>
__device__ __forceinline__ void load_fast(const FastIO<T, C>& io, int64_t y, T (&dst)[C]) {
    typedef typename V16<T>::u UT;
    typedef __attribute__((address_space(1))) const char GC;
    constexpr int VN = V16<T>::N;
    y = y < io.ylo ? io.ylo : (y > io.yhi ? io.yhi : y);
    const bool zr = EDGE && zero_row_fast(io, y);
    const uint32_t zm = zr ? 0u : ~0u;
    const int64_t ys = zr ? 0 : y;
    const bool lo = ys < 0, hi = ys >= io.ny;
    const int64_t row = lo ? io.hw + ys : (hi ? ys - io.ny : ys);
    // (values, not the struct's members, so that the struct stays in registers)
    const T *in = io.in, *top = io.top, *bot = io.bot;
    GC* base = (GC*)((lo ? top : (hi ? bot : in)) + row * io.nx);
    if constexpr (EDGE && RAG) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const T x = *(__attribute__((address_space(1))) const T*)(base + io.xload[j]);
            dst[j] = keep(x, io.col[j] & zm);
        }
    } else {
#pragma unroll
        for (int q = 0; q < C / VN; ++q) {
            const UT x = *(__attribute__((address_space(1))) const UT*)(base + io.xload[q]);
#pragma unroll
            for (int e = 0; e < VN; ++e) {
                const int j = q * VN + e;
                if constexpr (EDGE && kEdgeBranch<T, C, D, RAG>)
                    dst[j] = zr ? T(0) : keep(x[e], io.col[q * VN]);
                else
                    dst[j] = EDGE ? keep(x[e], io.col[q * VN] & zm) : x[e];
            }
        }
    }
}

__device__ __forceinline__ void store_cell(__amdgpu_buffer_rsrc_t rs, float v, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, (int)off, 0, 0);
}
__device__ __forceinline__ void store_cell(__amdgpu_buffer_rsrc_t rs, double v, uint32_t off) {
    u32x2 bits;
    __builtin_memcpy(&bits, &v, sizeof(bits));
    __builtin_amdgcn_raw_buffer_store_b64(bits, rs, (int)off, 0, 0);
}

template <typename T, int C, bool EDGE, bool RAG>
__device__ __forceinline__ void store_fast(const FastIO<T, C>& io, T*& orow, const T (&v)[C]) {
    typedef typename V16<T>::t VT;
    constexpr int VN = V16<T>::N;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(orow, (short)0, io.out_bytes, BUF_DWORD3);
    orow += io.nx;
    if constexpr (EDGE && RAG) {
#pragma unroll
        for (int j = 0; j < C; ++j) store_cell(rs, v[j], io.off[j]);
    } else {
#pragma unroll
        for (int q = 0; q < C / VN; ++q) {
            VT x;
#pragma unroll
            for (int e = 0; e < VN; ++e) x[e] = v[q * VN + e];
            u32x4 bits;
            __builtin_memcpy(&bits, &x, sizeof(bits));
            __builtin_amdgcn_raw_buffer_store_b128(bits, rs, (int)io.off[q], 0, 0);
        }
    }
}

// One row step of the pipeline for the row yy whose ring position is M
// (compile-time, the row loop is unrolled Q times): the load of row yy+Q-3 is
// issued into the slot of row yy-3, no longer needed; then level l+1 (l =
// 0..LV-1) produces row yy-l-1 from its three level-l rows.  Level 0 reads the
// Q-row ring, levels 1..D-1 keep their last three rows in a three-slot ring
// at position M mod 3.  Every slot index is a compile-time constant, so
// rotating rows costs no register moves.  LV < D while the pipeline fills
// (stream_rows_fast).
template <typename T, int C, int D, int Q, int M, int LV, bool STORE, bool EDGE, bool RAG, bool SC>
__device__ __forceinline__ void row_step_fast(const FastIO<T, C>& io, T*& orow, int64_t yy,
                                              T (&Z)[Q][C], T (&R)[D][3][C],
                                              const Rate2<T>& rt) {
    constexpr int VN = V16<T>::N;
    constexpr int M3 = M % 3, OLD = (M3 + 1) % 3, NEW = (M3 + 2) % 3;
    load_fast<T, C, D, EDGE, RAG>(io, yy + Q - 3, Z[(M + Q - 3) % Q]);
    T last[C];
#pragma unroll
    for (int l = 0; l < LV; ++l) {
        const T* cn = l == 0 ? Z[(M + Q - 1) % Q] : R[l][NEW];
        const T* no = l == 0 ? Z[(M + Q - 2) % Q] : R[l][OLD];
        const T* so = l == 0 ? Z[M] : R[l][M3];
        const T left = dpp_move<DPP_WAVE_SHR1>(cn[C - 1]);
        const T right = dpp_move<DPP_WAVE_SHL1>(cn[0]);
        T* dst = l + 1 < D ? R[l + 1 < D ? l + 1 : 0][M3] : last;
        const bool zr = EDGE && zero_row_fast(io, yy - l - 1);
        const uint32_t zm = zr ? 0u : ~0u;
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const T c = cn[j];
            const T we = (j > 0 ? cn[j - 1] : left) + (j + 1 < C ? cn[j + 1] : right);
            const T ns = no[j] + so[j];
            const T t = ns + we;
            const T v = update<T, SC>(rt, c, t);
            if constexpr (EDGE && kEdgeBranch<T, C, D, RAG>)
                dst[j] = zr ? T(0) : keep(v, io.col[j / VN * VN]);
            else
                dst[j] = EDGE ? keep(v, io.col[RAG ? j : j / VN * VN] & zm) : v;
        }
        rescale_level<T, C, D, SC>(rt, l, dst);
    }
    if constexpr (STORE) store_fast<T, C, EDGE, RAG>(io, orow, last);
}

// N consecutive row steps starting at ring position M.  Steps that store
// stop at the chunk's end.
template <typename T, int C, int D, int Q, int M, int N, int LV, bool STORE, bool EDGE, bool RAG,
          bool SC>
__device__ __forceinline__ void steps_fast(const FastIO<T, C>& io, T*& orow, int64_t& yy,
                                           int64_t yend, T (&Z)[Q][C], T (&R)[D][3][C],
                                           const Rate2<T>& rt) {
    if constexpr (N > 0) {
        if (STORE && yy >= yend) return;
        row_step_fast<T, C, D, Q, M, LV, STORE, EDGE, RAG, SC>(io, orow, yy, Z, R, rt);
        ++yy;
        steps_fast<T, C, D, Q, (M + 1) % Q, N - 1, LV, STORE, EDGE, RAG, SC>(io, orow, yy, yend,
                                                                            Z, R, rt);
    }
}

// Groups G .. WF-1 of Q rows that fill the pipeline.  Level l+1 of the chunk
// is needed from row y0-D+l+1 on, which input row ystart+m reaches once
// m >= 2l+2: the rows up to m = Q G + Q - 1 need at most (Q G + Q - 1) / 2
// levels, so a group runs only those (half of the fill's work for nothing
// otherwise: with 64-row chunks at D = 10 that was a ninth of all of it).
template <typename T, int C, int D, int Q, int G, int WF, bool EDGE, bool RAG, bool SC>
__device__ __forceinline__ void fill_fast(const FastIO<T, C>& io, T*& orow, int64_t& yy,
                                          int64_t yend, T (&Z)[Q][C], T (&R)[D][3][C],
                                          const Rate2<T>& rt) {
    if constexpr (G < WF) {
        constexpr int need = (Q * G + Q - 1) / 2;
        constexpr int LV = need < D ? need : D;
        steps_fast<T, C, D, Q, 0, Q, LV, false, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
        fill_fast<T, C, D, Q, G + 1, WF, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
    }
}

// Rows ystart .. ystart+2D-1 fill the pipeline (nothing to store yet); from
// then on every row step stores row yy - D, an output row of the chunk.
//
// ROLL: the fill as two loops, three groups of eight levels where those are
// enough (D >= 12), then groups of all D.  With every group's own level count
// the first rows take so little arithmetic that a wave runs ahead of its three
// rows in flight; where waves follow one another on a SIMD that cost more than
// the levels saved: 16384^2, 12 steps, 32 rows per wave, 18 % fewer vector
// instructions but twice the wave cycles waiting, 908 us against 795 rolled (10
// steps 599 / 525, 16 steps 1204 / 1056; 64 rows 741 / 677, 525 / 511, 963 /
// 877).  Grids whose waves all run at once gain from the short fill (4096^2, 10
// steps, 32 rows 62 us against 66), and so do all with ragged rows (16384 x
// 16382, 12 steps, 32 rows 698 against 752).
template <typename T, int C, int D, int Q, bool ROLL, bool EDGE, bool RAG, bool SC>
__device__ __forceinline__ void stream_rows_fast(const FastIO<T, C>& io, T*& orow, int64_t ystart,
                                                 int64_t yend, T (&Z)[Q][C], T (&R)[D][3][C],
                                                 const Rate2<T>& rt) {
    constexpr int W = 2 * D, WF = W / Q, WR = W % Q;
    constexpr int LR = (W - 1) / 2;  // levels the remaining WR rows need (below D)
#pragma unroll
    for (int m = 0; m < Q - 3; ++m) load_fast<T, C, D, EDGE, RAG>(io, ystart + m, Z[m]);
    int64_t yy = ystart;
    if constexpr (ROLL) {
        constexpr int G8 = D >= 12 ? 3 : 0;  // (rows 0 .. 17 need at most 8 levels)
        for (int i = 0; i < G8; ++i)
            steps_fast<T, C, D, Q, 0, Q, 8, false, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
        for (int i = G8; i < WF; ++i)
            steps_fast<T, C, D, Q, 0, Q, D, false, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
    } else {
        fill_fast<T, C, D, Q, 0, WF, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
    }
    steps_fast<T, C, D, Q, 0, WR, LR, false, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
    while (yy < yend)
        steps_fast<T, C, D, Q, WR, Q, D, true, EDGE, RAG, SC>(io, orow, yy, yend, Z, R, rt);
}

// One launch advances up to kMaxBands bands of one grid (same nx, r and
// depth) by one pass: band k owns waves [first[k], first[k+1]), each wave a
// (strip, chunk) of that band.  The set travels as the kernel argument.
struct BandSet {
    Band2D b[kMaxBands];
    int64_t first[kMaxBands + 1];
    int n;
};

// The dispatcher hands consecutive workgroups to the eight XCDs in turn, and
// each XCD has its own L2.  Neighbouring waves (adjacent strips of one chunk)
// share the lines at their strip edges; this bijection of [0, n) gives every
// XCD a contiguous range of workgroups, so that neighbouring strips mostly run
// under one L2 (measured 1.5-2 % faster on the 16384^2 pass).
__device__ __forceinline__ uint32_t xcd_block2d(uint32_t b, uint32_t n) {
    constexpr uint32_t X = 8;
    const uint32_t q = n / X, r = n % X, x = b % X;
    return x * q + (x < r ? x : r) + b / X;
}

template <typename T, int C, int D, bool ROLL, bool RAG, bool SC>
__global__ __launch_bounds__(256) void k_stencil2d(BandSet set, int rows, int halo,
                                                   int64_t nstrips) {
    constexpr int VN = V16<T>::N;
    constexpr int S = 64 * C;
    constexpr int Q = ring_rows();
    static_assert(C % VN == 0, "columns per lane must be a multiple of the vector width");
    static_assert(Q % 3 == 0 && Q >= 6, "the level-0 ring must be a multiple of 3 rows");
    const int wpg = blockDim.x >> 6;
    const int64_t wave = (int64_t)xcd_block2d(blockIdx.x, gridDim.x) * wpg +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= set.first[set.n]) return;
    int kb = 0;
    while (kb + 1 < set.n && wave >= set.first[kb + 1]) ++kb;
    const Band2D& b = set.b[kb];
    const int64_t wl = wave - set.first[kb];
    const int lane = threadIdx.x & 63;
    const int64_t strip = wl % nstrips;
    const int64_t chunk = wl / nstrips;
    const int64_t xb = strip * (S - 2 * halo) - halo;  // first column held by lane 0
    const int64_t y0 = chunk * rows;                   // output rows [y0, y1)
    const int64_t y1 = (y0 + rows < b.ny) ? y0 + rows : b.ny;
    const bool xin = xb >= 0 && xb + S <= b.nx;        // whole strip inside [0, nx)
    const Rate2<T> k = make_rate<T, SC>(b, D);

    // Rows above the first streamed row only feed rows that are never stored;
    // they start as zeros so that no stale register value is ever read.
    T R[D][3][C];
    T Z[Q][C];
#pragma unroll
    for (int l = 0; l < D; ++l)
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int j = 0; j < C; ++j) R[l][m][j] = T(0);
#pragma unroll
    for (int m = Q - 2; m < Q; ++m)
#pragma unroll
        for (int j = 0; j < C; ++j) Z[m][j] = T(0);

    const int64_t ystart = y0 - D;
    const int64_t yend = y1 + D;
    // Waves whose strip and rows stay clear of the zero-Dirichlet edges take
    // the interior variant.
    const bool edge = !xin || (ystart - D < 0 && b.bc_top != BC_GHOST) ||
                      (yend > b.ny && b.bc_bot != BC_GHOST);
    FastIO<T, C> io;
    const int64_t xb0 = xb < 0 ? 0 : xb;
    io.in = static_cast<const T*>(b.in) + xb0;
    io.top = static_cast<const T*>(b.halo_top) + xb0;
    io.bot = static_cast<const T*>(b.halo_bot) + xb0;
    T* orow = static_cast<T*>(b.out) + y0 * b.nx + xb0;  // row of the next store
    io.nx = b.nx;
    io.ny = b.ny;
    io.hw = b.hw;
    io.ylo = ystart;
    io.yhi = yend - 1;
    io.top_ghost = b.bc_top == BC_GHOST;
    io.bot_ghost = b.bc_bot == BC_GHOST;
    io.out_bytes = (int)((xb + S < b.nx ? xb + S : b.nx) - xb0) * (int)sizeof(T);
#pragma unroll
    for (int j = 0; j < C; ++j) {
        const int64_t x = xb + (int64_t)lane * C + j;
        io.col[j] = x >= 0 && x < b.nx ? ~0u : 0u;
    }
    const bool cells = RAG && edge;  // offsets per cell, else per vector (index q)
#pragma unroll
    for (int j = 0; j < C; ++j) {
        // without RAG, nx is a multiple of the vector width, so a lane vector
        // is either wholly inside [0, nx) or wholly outside; one outside (a
        // cell outside) loads a clamped address and is replaced by zeros
        const int w = cells ? 1 : VN;
        const int lc = lane * C + j * w;
        const int64_t x = xb + lc;
        const int64_t xc = x < 0 ? 0 : (x + w > b.nx ? b.nx - w : x);
        io.xload[j] = (uint32_t)((xc - xb0) * (int64_t)sizeof(T));
        io.off[j] = (lc >= halo && lc < S - halo && x >= 0 && x < b.nx)
                        ? (uint32_t)((x - xb0) * (int64_t)sizeof(T))
                        : OOB_OFFSET;
    }
    if (edge)
        stream_rows_fast<T, C, D, Q, ROLL, true, RAG, SC>(io, orow, ystart, yend, Z, R, k);
    else
        stream_rows_fast<T, C, D, Q, ROLL, false, RAG, SC>(io, orow, ystart, yend, Z, R, k);
}

template <typename T, int C, int D, bool ROLL = (D >= 12)>
hipError_t launch_cd(const Band2D* bands, int n, const Geom2D& g, hipStream_t st) {
    constexpr int VN = V16<T>::N;
    const int64_t wout = 64LL * C - 2LL * g.halo;
    const int64_t nx = bands[0].nx;
    const int64_t nstrips = (nx + wout - 1) / wout;
    BandSet set{};
    set.n = n;
    bool sc = true;
    int64_t total = 0;
    for (int k = 0; k < n; ++k) {
        Band2D bb = bands[k];
        set_rate_2d(bb, D);
        sc = sc && bb.period > 0;
        set.b[k] = bb;
        set.first[k] = total;
        total += nstrips * ((bb.ny + g.rows - 1) / g.rows);
    }
    set.first[n] = total;
    const dim3 block(64 * g.wpg);
    const dim3 grid((unsigned)((total + g.wpg - 1) / g.wpg));
    const bool rag = nx % VN != 0;
    if (sc && !rag)
        hipLaunchKernelGGL((k_stencil2d<T, C, D, ROLL, false, true>), grid, block, 0, st, set, g.rows,
                           g.halo, nstrips);
    else if (sc)
        hipLaunchKernelGGL((k_stencil2d<T, C, D, false, true, true>), grid, block, 0, st, set, g.rows,
                           g.halo, nstrips);
    else if (!rag)
        hipLaunchKernelGGL((k_stencil2d<T, C, D, ROLL, false, false>), grid, block, 0, st, set, g.rows,
                           g.halo, nstrips);
    else
        hipLaunchKernelGGL((k_stencil2d<T, C, D, false, true, false>), grid, block, 0, st, set, g.rows,
                           g.halo, nstrips);
    return hipGetLastError();
}

}  // namespace
}  // namespace hx
