// density.hip - Gaussian density grid per frame as a matrix-core contraction
// on gfx950.
//
// The per-frame density of Algorithm 1 (Section 3.6),
//     D[gy][gx] = c * sum_i exp(-((cx - x_i)^2 + (cy - y_i)^2) / (2 s^2)),
//     c = 1 / (2 pi s^2),
// separates into per-axis factors Fy[gy][i] = exp(-(cy - y_i)^2 / (2 s^2)) and
// Fx[gx][i] = exp(-(cx - x_i)^2 / (2 s^2)), so D = c * Fy . Fx^T: a dense
// contraction over the birds of the frame, run on the matrix cores with fp16
// factors and fp32 accumulation.
//
// Factors are stored as fp16 values of 2^8 f (kLift; the largest, 256, is
// far from fp16's limit) and the 2^-16 of the product goes into the output
// scale, so fp16's subnormal range starts at f = 2^-22 (5.5 s from the bird)
// instead of 2^-14 (4.4 s).  A bird has nonzero factors only in the rows
// within about 6 s of it (its window: the tables hold the cells up to
// ceil(6 s / cell) + 1 away, exact zeros beyond); the contraction stays
// dense over all (row, column, bird) triples.
//
// Two ways to make the operands:
//
// Gather path (the cell size c = 16 W / G is a whole number of 1/16-px quanta
// on both axes).  A bird at quantum q = 4 c Q + r (0 <= r < 4 c) sits at the
// same offset (n + 1/2) c - r from the centre of cell 4 Q + n for every group
// Q of four cells, so its factors are one row of an exact table indexed by r,
// built in LDS once per workgroup as fp16 in 8-byte chunks of four cells.  A
// v_mfma_f32_16x16x32_f16 operand (16 cells x 32 birds) is two transposing
// LDS reads (ds_read_b64_tr_b16): each lane addresses one chunk of one bird,
// one clamp and one add each, and gets four birds' factors of its own cell,
// with no packing, no tile writes and no barriers.  (Reading a 32-bit factor
// pair per lane and bird instead, as before, took eight clamped reads and
// eight byte permutes for every two tiles: 256 x 8000 birds on 256 x 144
// cells 143 us, now 78; 64 x 2000 on 128 x 72 17.0, now 10.2.)  What bounds
// it now: the matrix cores are busy 26% of the launch on the former (55 GFLOP
// issued) and 2.4% on the latter; the rest is what a 32-bird step's reads, which
// do not overlap its MFMAs, the per-block bird test and staging, and launch,
// table build and final sum take.
// Waves sharing a frame region add their tiles in a fixed order at the end;
// batches with few (frame, region) pairs also split frames into bird slices
// whose partial grids a second kernel adds in slice order.
//
// Direct path (any other grid, and windows too wide for the tables).  The same
// kernel, with the 32 birds of a k-step evaluated instead of looked up: two
// lanes take a bird, write the factors of its windows (or of the whole region,
// where that is smaller) into rows of their wave's own LDS scratch, and the
// operands are read from there as above.  Each chunk of four cells starts from
// exact exponentials.  (Before, 128 birds at a time were written as columns of
// cleared LDS tiles by a recurrence between barriers: 48 ragged frames of up to
// 3000 birds on a 97 x 61 grid took 38 us, now 15.5.)  Bound by the factors:
// about 18 exponentials per lane and step at windows of 27 cells.
//
// Accuracy: a normal fp16 factor (f >= 2^-22) carries a relative rounding
// error <= 2^-11 (plus a few fp32 ulps before the conversion); a subnormal
// one an absolute error <= 2^-25 of 2^8 f, i.e. 2^-33 of f.  (Stepping three
// cells on adds at most 2^-17 of f.)  A term is a
// product of two factors <= 1, so its error is <= about 2^-10 of the term plus
// 2^-32 absolute; all terms are positive, so an output's error is <= 2^-10 of
// the output plus N 2^-32 c for N birds (c = 1 / (2 pi s^2)), against an
// output <= the frame's maximum.  The window's cut contributes < 2^-25 per
// factor.  Every sum is taken in a fixed order, so results are
// deterministic.

#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace flock {
namespace {

constexpr float kCutSigmas = 6.0f;
constexpr float kLift = 256.0f;      // factors are stored as fp16(kLift f)

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kGWaves = 8;                 // waves per workgroup (two per SIMD)
constexpr int kGThreads = 64 * kGWaves;
constexpr int kGStep = 32;                 // birds per MFMA k-step (16 x 16 x 32)
constexpr int kGRedTiles = 8;              // 16 x 16 tiles per round of the cross-wave sum
constexpr int kGPair = 2;                  // blocks of 64 birds a wave tests at a time
constexpr int kGAhead = 2;                 // pairs of blocks loaded ahead
constexpr int kGRing = 160;                // staged birds per wave (under one k-step left over + one pair of blocks)
constexpr int kGMaxLds = 159 * 1024;        // of a compute unit's 160 KiB
constexpr int kGMaxTableBytes = kGMaxLds - kGWaves * kGRing * 16;  // both factor tables
constexpr int kGMinWaveBirds = 32;         // kept birds per wave, at least, when a launch splits frames
constexpr int32_t kGNone = INT_MIN;         // direct path: coordinate of a padding bird
constexpr int32_t kGFar = 1 << 28;         // bird term that clamps every cell to a zero chunk

typedef float float4v __attribute__((ext_vector_type(4)));

// Factor table of one axis.  A bird at quantum q lies at r = q mod 4c of cell
// group Q = q / 4c (four cells per group); row r (0 <= r < 4c) holds, as fp16,
// the factors of cells 4 Q + n in chunks of four cells (8 bytes): chunk k has
// n = 4 (k - j4) .. + 3, k = 0 .. nc - 1, which covers the window of every
// bird of the row, and a cell outside its bird's window is 0.  Every row ends
// with a zero chunk, and one more lies before row 0, so that both neighbours
// of a row's chunks are zeros.
struct GatherAxis {
    int32_t c;      // quanta per cell (table path)
    int32_t j;      // window half-width, cells
    int32_t j4;     // chunks before the bird's own group: ceil(j / 4)
    int32_t nc;     // chunks of a window: 2 j4 + 1
    int32_t tab;    // byte offset of the table (its leading zero chunk) in LDS
    float h, inv_h; // cell size, px (direct path)
    float reach;    // window half-width, quanta, whatever j's limit (direct path)
    // with k = -log2(e) / (2 s^2): 2 k h, k h^2 and exp2(2 k h^2), for steps of
    // one cell where h <= 2 s (else step_q is 0)
    float step_d, step_h, step_q;
};

struct GatherGeom {
    GatherAxis ay, ax;
    float neg_k;      // -log2(e) / (2 s^2), px^-2
    float scale;      // 1 / (2 pi s^2 kLift^2)
    int table_bytes;  // the tables (one when both axes agree), or the waves' factor scratch; 16-byte aligned
    int red_tiles;    // tiles per round of the cross-wave sum: kGRedTiles, or 2 beside large tables
    int lds_bytes;
};

// One bird as a lane reads it: per axis the byte offset of its table row and
// j4 - Q, Q its cell group (on the direct path its coordinate, and unused).
struct GBird {
    int32_t rb_y, g_y, rb_x, g_x;
};

__host__ __device__ __forceinline__ int32_t table_row_bytes(const GatherAxis &t) { return 8 * (t.nc + 1); }

// floor(v / c) for |v| < 2^24, 1 <= c < 2^22: a float reciprocal, then one
// correction step either way.
__device__ __forceinline__ int32_t floor_div(int32_t v, int32_t c, float inv_c) {
    const int32_t q = (int32_t)floorf((float)v * inv_c);
    const int32_t r = v - __mul24(q, c);  // |q c| <= |v| + c: exact in 32 bits
    return q + (int32_t)(r >= c) - (int32_t)(r < 0);
}

__device__ __forceinline__ void stage_axis(int32_t q, const GatherAxis &t, float inv_c4, int32_t *rb, int32_t *g) {
    // exact for |q| < 2^24; beyond that the bird is far outside any grid and
    // only the table row needs keeping in range
    const int32_t c4 = 4 * t.c;
    const int32_t Q = floor_div(q, c4, inv_c4);
    const int32_t r = min(max(q - __mul24(Q, c4), 0), c4 - 1);
    *rb = t.tab + 8 + __mul24(table_row_bytes(t), r);
    *g = t.j4 - Q;
}

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));

// The MFMA operand of tile M (16 cells) for the 32 birds of a k-step.  The
// 16 lanes of a group own eight birds (k = 8 group .. + 7); lane i of the
// group addresses chunk i % 4 of the tile for birds i / 4 and i / 4 + 4, and
// the transposing LDS read hands lane i the four birds' values of cell i.
// With v = (first cell) / 4 + i % 4 + j4 - Q, the chunk's index in the bird's
// row is clamp(v + 4 M, -1, nc): an index clamped from below or above meets a
// zero chunk, as the true factors there are.
struct LaneBirds {
    int32_t rb0, v0, rb1, v1;
};

// median of v, lo and hi: clamp(v, LO, hi) for LO <= hi, as one instruction
// (a wave-uniform bound and an inline constant)
template <int LO>
__device__ __forceinline__ int32_t clamp_uniform(int32_t v, int32_t hi) {
    int32_t o;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(o) : "v"(v), "n"(LO), "s"(hi));
    return o;
}

template <int M>
__device__ __forceinline__ half4 read_chunk(const unsigned char *lds, int32_t rb, int32_t v, int32_t nc) {
    constexpr int kLo = M & 3, kHi = M & ~3;  // inline constants reach -16: tiles 4 and up shift v first
    const int32_t o = clamp_uniform<-1 - 4 * kLo>(v + 4 * kHi, nc - 4 * kLo);
    typedef __attribute__((address_space(3))) short4v lds_short4;
    return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                         (lds_short4 *)(lds + (rb + 8 * o) + 32 * kLo)));
}

template <int M>
__device__ __forceinline__ half8 operand(const LaneBirds &b, int32_t nc, const unsigned char *lds) {
    const half4 lo4 = read_chunk<M>(lds, b.rb0, b.v0, nc), hi4 = read_chunk<M>(lds, b.rb1, b.v1, nc);
    return __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int T, int N = 0>
__device__ __forceinline__ void operands(half8 (&op)[T], const LaneBirds &b, int32_t nc, const unsigned char *lds) {
    if constexpr (N < T) {
        op[N] = operand<N>(b, nc, lds);
        operands<T, N + 1>(op, b, nc, lds);
    }
}

// A work item is (frame, output region of 16 TM rows x 16 TN columns, slice
// of the frame's birds); `waves` waves of a workgroup share an item, and
// their tiles are added in a fixed order at the end (deterministic).  With
// split > 1 the slices' grids go to `partial` for a second kernel to add.
// The slices and waves of a (frame, region) take the frame's 64-bird blocks
// in turn (a fixed assignment).  A workgroup builds its tables once and takes
// every gridDim.x-th group of kGWaves / waves items.
//
// Only birds whose window of cells (G - j .. G + j on both axes) meets the
// region contribute to it: every other bird's factors there are table zeros.
// Each wave reads its blocks one at a time (one bird per lane), keeps the ones that
// meet the region, in input order, in a ring of staged birds in LDS (ballot
// ranks), and runs a k-step whenever 32 are staged; the last step is padded
// with birds whose factors are all zero.  No barrier is needed until the
// final sum.
template <int TM, int TN, bool DIRECT, bool AXES>
__global__ __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(2))) void density_gather_kernel(
    DensityArgs a, GatherGeom gg, int regions_y, int regions_x, int split, int waves, uint32_t items, float *partial) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: item, bird counts and ring positions are scalars

    const int part = wave % waves;
    const int regions = regions_y * regions_x;
    // the split * waves (slice, part) units of a (frame, region) take the
    // frame's 64-bird blocks in turn: unit u = sl * waves + part reads blocks
    // u, u + split * waves, ...  Spatially grouped birds in the input then
    // spread over all units instead of loading one of them.
    const int32_t stride = 64 * split * waves;

    GBird *ring = reinterpret_cast<GBird *>(lds + gg.table_bytes) + wave * kGRing;
    const float inv_cy = 1.0f / (float)(4 * gg.ay.c), inv_cx = 1.0f / (float)(4 * gg.ax.c);
    const int r16 = lane & 15, grp = lane >> 4;
    // direct path: a factor row holds the bird's window, or all of the
    // region's chunks where those are fewer
    const bool whole_y = DIRECT && !AXES && gg.ay.nc >= 4 * TM, whole_x = DIRECT && !AXES && gg.ax.nc >= 4 * TN;
    const int32_t ncy = whole_y ? 4 * TM : gg.ay.nc, ncx = whole_x ? 4 * TN : gg.ax.nc;
    // a bird in cell G meets rows [row0, row0 + 16 TM) when
    // row0 - j <= G <= row0 + 16 TM - 1 + j, i.e. when its quantum q lies in
    // [(row0 - j) c, (row0 + 16 TM + j) c)  (below 2^31: c (grid + 2 j) is
    // 16 times the frame's extent and two windows); the direct path's bounds
    // are the same in px, a quantum wider for their rounding and clamped
    auto low = [](const GatherAxis &t, int first) {
        if (!DIRECT) return (first - t.j) * t.c;
        return (int32_t)fminf(fmaxf((float)first * t.h * 16.0f - t.reach - 1.0f, -33554432.0f), 33554432.0f);
    };
    auto span = [](const GatherAxis &t, int rows, int first, int32_t lo) {
        if (!DIRECT) return (uint32_t)(rows + 2 * t.j) * (uint32_t)t.c;
        const float end = (float)(first + rows) * t.h * 16.0f + t.reach + 2.0f;
        return (uint32_t)((int32_t)fminf(fmaxf(end, -33554432.0f), 33554432.0f) - lo);
    };

    // this wave's item, and its part of the item's birds: coordinates are
    // loaded kGAhead pairs of 64-bird blocks ahead
    const uint32_t per_wg = (uint32_t)(kGWaves / waves), groups = (items + per_wg - 1) / per_wg;
    bool active = false;
    uint32_t f = 0;
    int sl = 0, row0 = 0, col0 = 0;
    int32_t n = 0, left = 0;  // left: birds from the next block's first on
    const int2 *P = nullptr;
    int2 qn[kGAhead * kGPair];
    // the u-th block on (n > 0; past the frame's end its last bird again):
    // unconditional, so that the loads stay in flight across the blocks
    auto load = [&](int u) {
        return P[min((uint32_t)(n - left) + (uint32_t)(u * stride + lane), (uint32_t)(n - 1))];
    };
    auto begin = [&](uint32_t group) {
        const uint32_t item = group * per_wg + (uint32_t)(wave / waves);
        active = item < items;
        const uint32_t it = active ? item : 0u, fr = it / (uint32_t)split;
        sl = (int)(it - fr * (uint32_t)split);
        f = fr / (uint32_t)regions;
        const int reg = (int)(fr - f * (uint32_t)regions), ry = reg / regions_x;
        row0 = ry * 16 * TM;
        col0 = (reg - ry * regions_x) * 16 * TN;
        const int32_t b = a.offsets[f], e = a.offsets[f + 1];
        n = (!active || b < 0 || e < b || e > a.total) ? 0 : e - b;
        P = reinterpret_cast<const int2 *>(a.xy) + b;
        left = n - 64 * (sl * waves + part);
#pragma unroll
        for (int u = 0; u < kGAhead * kGPair; ++u) qn[u] = n > 0 ? load(u) : make_int2(0, 0);
    };
    uint32_t group = blockIdx.x;
    begin(group);  // the first coordinates are in flight while the tables are built

    // the factor tables (exact: every distance is a multiple of 1/32 px).
    // Rows r, r + c, r + 2c and r + 3c hold the same factors shifted by one
    // cell each: a thread makes eight factors of row r (and the three before
    // them) and writes two chunks of all four rows.
    auto build = [&](const GatherAxis &t) {
        const int per = (t.nc + 2) / 2;  // pairs of chunks 2 k, 2 k + 1 <= nc, the zero chunk nc among them
        const int rowb = table_row_bytes(t);
        const float inv_per = 1.0f / (float)per;
        if (tid == 0) *reinterpret_cast<uint2 *>(lds + t.tab) = make_uint2(0u, 0u);
        for (int it = tid; it < t.c * per; it += kGThreads) {
            const int r = floor_div(it, per, inv_per), k = it - r * per;
            uint32_t h[11];  // factors of cells n = 8 k - 4 j4 - 3 + i of row r
#pragma unroll
            for (int i = 0; i < 11; ++i) {
                const int n = 8 * k - 4 * t.j4 - 3 + i;
                const float d = (((float)n + 0.5f) * (float)t.c - (float)r) * 0.0625f;
                const float f = kLift * __builtin_amdgcn_exp2f(d * d * gg.neg_k);
                h[i] = __builtin_bit_cast(uint16_t, (_Float16)((n >= -t.j) & (n <= t.j) ? f : 0.0f));
            }
#pragma unroll
            for (int sh = 0; sh < 4; ++sh) {
                // cell n of row r + sh c is cell n - sh of row r
                unsigned char *row = lds + t.tab + 8 + (r + sh * t.c) * rowb;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int i = 3 + 4 * u - sh;
                    if (2 * k + u <= t.nc)
                        *reinterpret_cast<uint2 *>(row + 8 * (2 * k + u)) =
                            make_uint2(h[i] | (h[i + 1] << 16), h[i + 2] | (h[i + 3] << 16));
                }
            }
        }
    };
    // the wave's scratch: a zero chunk, then 32 rows of ncy chunks and a zero
    // chunk each, then 32 rows for x
    const int rowy = 8 * (ncy + 1), rowx = 8 * (ncx + 1);
    const int scratch_y = wave * (gg.table_bytes / kGWaves) + 8, scratch_x = scratch_y + 32 * rowy;
    if constexpr (DIRECT) {
        const uint2 zero = make_uint2(0u, 0u);
        if (lane == 0) *reinterpret_cast<uint2 *>(lds + scratch_y - 8) = zero;
        *reinterpret_cast<uint2 *>(lds + (lane < 32 ? scratch_y + (lane + 1) * rowy : scratch_x + (lane - 31) * rowx) - 8) = zero;
    } else {
        build(gg.ay);
        if (gg.ax.tab != gg.ay.tab) build(gg.ax);
    }
    __syncthreads();  // tables written

    // a wave's LDS accesses stay in program order; the fences keep the
    // compiler from moving them across the ring's writes and reads
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const uint64_t below = (1ull << lane) - 1ull;
    const GBird none = DIRECT ? GBird{kGNone, 0, kGNone, 0} : GBird{gg.ay.tab + 8, kGFar, gg.ax.tab + 8, kGFar};
    const size_t cells = (size_t)a.grid_h * a.grid_w;
    const float scale = split > 1 ? 1.0f : gg.scale;

    for (;;) {
        float4v acc[TM][TN];
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[m][t] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
        const int32_t yoff = (row0 >> 2) + (lane & 3), xoff = (col0 >> 2) + (lane & 3);
        const int32_t y_lo = low(gg.ay, row0), x_lo = low(gg.ax, col0);
        const uint32_t y_n = span(gg.ay, 16 * TM, row0, y_lo), x_n = span(gg.ax, 16 * TN, col0, x_lo);
        int32_t head = 0, staged = 0;  // the staged birds: ring positions from head on, modulo kGRing
        static_assert(kGRing >= kGStep - 1 + 64 * kGPair && kGRing % kGStep == 0, "a step's birds are contiguous");
        auto place = [&](int32_t p) { return p >= kGRing ? p - kGRing : p; };
        auto step = [&] {
            wave_sync();
            // every operand's reads are issued before the first MFMA (left to
            // itself the compiler waits for each row tile's reads in turn)
            half8 bx[TN], ay[TM];
            const int bird = 8 * grp + (r16 >> 2);  // this lane's two birds of the step: i / 4 and i / 4 + 4 of its group's eight
            if constexpr (DIRECT) {
                // lanes l and l + 32 make bird l's factors, every other chunk of
                // both axes each (an axis each leaves the lanes of the narrower
                // window waiting: 460 frames of 4340 birds on 46 x 123 cells,
                // windows of 8 and 19 cells either side, 152 us, now 96); or,
                // with AXES, an axis each
                const GBird e = ring[head + (lane & 31)];
                // a padding bird's factors are 0 whatever sigma and the distance
                const bool none = e.rb_y == kGNone;
                const float lift = none ? -1.0e30f : 8.0f;  // 2^8 = kLift
                const int half = lane >> 5;
                auto make = [&](int32_t q, const GatherAxis &t, int first, bool whole, unsigned char *row, int nc, int k0,
                                int dk) {
                    const float pos = none ? 0.0f : (float)q * 0.0625f;
                    if (!whole) first = ((int)floorf(pos * t.inv_h) >> 2) - t.j4;  // the row's first chunk, in chunks of the grid
                    float cell = (float)(4 * (first + k0)) + 0.5f;
                    if (t.step_q > 0.0f) {
                        // the factor and its ratio to the next cell's as exact
                        // exponentials per chunk, the other three cells by
                        // F(d + h) = F(d) R(d), R(d + h) = R(d) step_q.  (Far
                        // off F is 0 and R is held finite; three cells further,
                        // at most 6 s, F is still below fp16's range.)
                        for (int k = k0; k < nc; k += dk, cell += (float)(4 * dk)) {
                            const float d = fmaf(cell, t.h, -pos);
                            const float f0 = __builtin_amdgcn_exp2f(fmaf(d * d, gg.neg_k, lift));
                            const float r0 = __builtin_amdgcn_exp2f(fminf(fmaf(d, t.step_d, t.step_h), 100.0f));
                            const float r1 = r0 * t.step_q, r2 = r1 * t.step_q;
                            const float f1 = f0 * r0, f2 = f1 * r1, f3 = f2 * r2;
                            *reinterpret_cast<half4 *>(row + 8 * k) =
                                half4{(_Float16)f0, (_Float16)f1, (_Float16)f2, (_Float16)f3};
                        }
                    } else {
                        for (int k = k0; k < nc; k += dk, cell += (float)(4 * dk)) {
                            half4 f;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const float d = fmaf(cell + (float)i, t.h, -pos);
                                f[i] = (_Float16)__builtin_amdgcn_exp2f(fmaf(d * d, gg.neg_k, lift));
                            }
                            *reinterpret_cast<half4 *>(row + 8 * k) = f;
                        }
                    }
                    return first;
                };
                unsigned char *to_y = lds + scratch_y + (lane & 31) * rowy, *to_x = lds + scratch_x + (lane & 31) * rowx;
                int fy, fx;
                if constexpr (AXES) {
                    const GatherAxis t = half ? gg.ax : gg.ay;
                    fy = fx = make(half ? e.rb_x : e.rb_y, t, 0, false, half ? to_x : to_y, ncy, 0, 1);
                } else {
                    fy = make(e.rb_y, gg.ay, row0 >> 2, whole_y, to_y, ncy, half, 2);
                    fx = make(e.rb_x, gg.ax, col0 >> 2, whole_x, to_x, ncx, half ^ (ncy & 1), 2);
                }
                wave_sync();
                const int from_x = bird + (AXES ? 32 : 0);
                const int fy0 = __shfl(fy, bird, 64), fy1 = __shfl(fy, bird + 4, 64);
                const int fx0 = __shfl(fx, from_x, 64), fx1 = __shfl(fx, from_x + 4, 64);
                const int ry = scratch_y + bird * rowy, rx = scratch_x + bird * rowx;
                operands<TN>(bx, LaneBirds{rx, xoff - fx0, rx + 4 * rowx, xoff - fx1}, ncx, lds);
                operands<TM>(ay, LaneBirds{ry, yoff - fy0, ry + 4 * rowy, yoff - fy1}, ncy, lds);
            } else {
                const GBird *sb = ring + head + bird;
                const int4 q0 = *reinterpret_cast<const int4 *>(sb), q1 = *reinterpret_cast<const int4 *>(sb + 4);
                operands<TN>(bx, LaneBirds{q0.z, q0.w + xoff, q1.z, q1.w + xoff}, ncx, lds);
                operands<TM>(ay, LaneBirds{q0.x, q0.y + yoff, q1.x, q1.y + yoff}, ncy, lds);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ay[m], bx[t], acc[m][t], 0, 0, 0);
            head = place(head + kGStep);
            staged -= kGStep;
            wave_sync();  // the step's reads are done before the ring is written again
        };
        while (left > 0) {  // wave-uniform
#pragma unroll
            for (int u = 0; u < kGAhead; ++u) {
                if (left <= 0) break;
                int2 q[kGPair];
                uint64_t m[kGPair];
                bool keep[kGPair];
#pragma unroll
                for (int h = 0; h < kGPair; ++h) {
                    q[h] = qn[kGPair * u + h];
                    keep[h] = (lane < left - h * stride) & ((uint32_t)q[h].y - (uint32_t)y_lo < y_n) &
                              ((uint32_t)q[h].x - (uint32_t)x_lo < x_n);
                    m[h] = __ballot(keep[h]);
                    qn[kGPair * u + h] = load(kGAhead * kGPair + h);
                }
                left -= kGPair * stride;
#pragma unroll
                for (int h = 0; h < kGPair; ++h) {
                    if (keep[h]) {
                        GBird gb{q[h].y, 0, q[h].x, 0};
                        if constexpr (!DIRECT) {
                            stage_axis(q[h].y, gg.ay, inv_cy, &gb.rb_y, &gb.g_y);
                            stage_axis(q[h].x, gg.ax, inv_cx, &gb.rb_x, &gb.g_x);
                        }
                        ring[place(head + staged + __popcll(m[h] & below))] = gb;
                    }
                    staged += __popcll(m[h]);
                }
                while (staged >= kGStep) step();
            }
        }
        // the last, partial step is filled with birds whose factors are all zero
        if (staged > 0) {
            if (lane < kGStep && lane >= staged) ring[head + lane] = none;
            step();
        }

        float *out = split > 1 ? partial + ((size_t)f * split + sl) * cells : a.density + (size_t)f * cells;
        const bool write = active;
        const int orow = row0 + 4 * grp, ocol = col0 + r16;  // of a tile's float4: lane l holds rows 4 (l / 16) .. + 3, column l % 16
        group += gridDim.x;
        const bool more = group < groups;
        if (more) begin(group);  // the next item's first coordinates are in flight during the sum
        auto store = [&](int t, float4v v) {
            const int gy = orow + 16 * (t / TN), gx = ocol + 16 * (t % TN);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (write && gy + i < a.grid_h && gx < a.grid_w) out[(size_t)(gy + i) * a.grid_w + gx] = v[i] * scale;
        };
        if (waves == 1) {
#pragma unroll
            for (int t = 0; t < TM * TN; ++t) store(t, acc[t / TN][t % TN]);
        } else {
            // the waves of an item add their tiles in wave order, a few
            // tiles at a time, in LDS beside the tables (the rings' space)
            float4v *red = reinterpret_cast<float4v *>(lds + gg.table_bytes);
            const int w0 = (wave / waves) * waves;
            constexpr int kTiles = TM * TN;
            auto sum = [&](auto round) {
                constexpr int kRound = decltype(round)::value;
                __syncthreads();  // every wave is past its last step
#pragma unroll
                for (int t0 = 0; t0 < kTiles; t0 += kRound) {
#pragma unroll
                    for (int q = 0; q < kRound; ++q) {
                        const int t = t0 + q;
                        if (t < kTiles) red[(wave * kRound + q) * 64 + lane] = acc[t / TN][t % TN];
                    }
                    __syncthreads();
                    const int nt = min(kRound, kTiles - t0);
                    for (int q = part; q < nt; q += waves) {
                        float4v v = red[(w0 * kRound + q) * 64 + lane];
                        for (int w = 1; w < waves; ++w) v += red[((w0 + w) * kRound + q) * 64 + lane];
                        store(t0 + q, v);
                    }
                    __syncthreads();
                }
            };
            if (gg.red_tiles == kGRedTiles) sum(std::integral_constant<int, kGRedTiles>{});
            else sum(std::integral_constant<int, 2>{});
        }
        if (!more) return;
    }
}

// density[f][cell] = scale * sum over slices s = 0, 1, ... of partial[f][s][cell].
__global__ __launch_bounds__(256) void density_reduce_kernel(float *density, const float *partial,
                                                             int64_t cells, int64_t total, int split,
                                                             float scale) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t f = i / cells, c = i - f * cells;
        const float *src = partial + f * split * cells + c;
        // slices in order, eight loads in flight at a time (a missing slice
        // adds +0, which leaves the non-negative sum unchanged)
        float s = 0.0f;
        for (int k0 = 0; k0 < split; k0 += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k0 + u < split ? src[(int64_t)(k0 + u) * cells] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        density[i] = s * scale;
    }
}

struct Shape {
    int rm, rn;  // tiles of 16 x 16 cells
};
// instantiated region shapes (tiles of 16 x 16; at most 36
// tiles per region, so that the accumulators and operands fit the registers
// of two waves per SIMD without spilling)
constexpr int kDirectTiles = 32;  // the direct path's registers hold this many
constexpr int kPairTiles = 8;     // and those of two workgroups per compute unit this many
constexpr Shape kGShapes[] = {{1, 1}, {2, 2}, {1, 4}, {4, 1}, {2, 4}, {4, 2}, {3, 4},
                              {4, 4}, {5, 4}, {9, 2}, {9, 4}, {3, 8}, {4, 8}};

// LDS beside the tables or scratch: the rings, whose space also holds the
// cross-wave sum's tiles (within `limit` bytes in all; two tiles of every wave
// take no more than the rings).
void gather_lds(GatherGeom *gg, int limit = kGMaxLds) {
    const int ring = kGWaves * kGRing * (int)sizeof(GBird), red = kGWaves * kGRedTiles * 1024;
    gg->red_tiles = gg->table_bytes + red <= limit ? kGRedTiles : 2;
    gg->lds_bytes = gg->table_bytes + std::max(ring, gg->red_tiles == kGRedTiles ? red : 0);
}

// Window of an axis of n cells over `extent` px: every cell centre within the
// cut of a bird lies at most j cells from the bird's own.  j is limited to
// twice the widest grid: a window that wide holds any region whole, and only
// `reach`, which has no limit, says how far off its birds may lie.
void gather_window(GatherAxis *t, int extent, int n, double sigma) {
    const double h = (double)extent / n;
    t->h = (float)h;
    t->inv_h = (float)(1.0 / h);
    const double j = std::ceil((double)kCutSigmas * sigma / h) + 1.0;
    t->j = (int32_t)std::min(j, 8192.0);
    t->reach = (float)std::min(16.0 * j * h, 1.0e9);
    t->j4 = (t->j + 3) / 4;
    t->nc = 2 * t->j4 + 1;
    const double k = -1.4426950408889634 / (2.0 * sigma * sigma);
    t->step_d = (float)(2.0 * k * h);
    t->step_h = (float)(k * h * h);
    t->step_q = h <= 2.0 * sigma ? (float)std::exp2(2.0 * k * h * h) : 0.0f;
}

// Geometry of a launch on the direct path, but for its scratch (direct_lds).
void base_geom(const DensityArgs &a, GatherGeom *gg) {
    const double s = (double)a.sigma_px;
    gather_window(&gg->ay, a.height_px, a.grid_h, s);
    gather_window(&gg->ax, a.width_px, a.grid_w, s);
    gg->neg_k = (float)(-1.4426950408889634 / (2.0 * s * s));
    gg->scale = (float)(1.0 / (2.0 * 3.14159265358979323846 * s * s) / ((double)kLift * kLift));
    gg->ay.c = gg->ax.c = 0;
    gg->ay.tab = gg->ax.tab = 0;
}

// Makes it the geometry of the table path where a cell is a whole number of
// quanta on both axes and the tables fit beside the rings.
bool table_geom(const DensityArgs &a, GatherGeom *gg) {
    if ((16LL * a.height_px) % a.grid_h != 0 || (16LL * a.width_px) % a.grid_w != 0) return false;
    const int64_t cy = 16LL * a.height_px / a.grid_h, cx = 16LL * a.width_px / a.grid_w;
    auto bytes = [](int64_t c, const GatherAxis &t) { return (8 + 4 * c * table_row_bytes(t) + 15) / 16 * 16; };
    if (cy > kGMaxTableBytes || cx > kGMaxTableBytes) return false;
    const bool shared = cy == cx && gg->ay.j == gg->ax.j;
    const int64_t ty = bytes(cy, gg->ay), all = ty + (shared ? 0 : bytes(cx, gg->ax));
    if (all > kGMaxTableBytes) return false;
    gg->ay.c = (int32_t)cy;
    gg->ax.c = (int32_t)cx;
    gg->ax.tab = shared ? 0 : (int32_t)ty;
    gg->table_bytes = (int)all;
    gather_lds(gg);
    return true;
}

// The direct path's scratch for regions of rm x rn tiles (at most 50 chunks
// per bird for the shapes it takes: 12.5 KiB per wave).
void direct_lds(GatherGeom *gg, int rm, int rn, int resident) {
    const int chunks = std::min(gg->ay.nc, 4 * rm) + std::min(gg->ax.nc, 4 * rn) + 2;
    gg->table_bytes = kGWaves * ((8 + 32 * 8 * chunks + 15) / 16 * 16);
    gather_lds(gg, kGMaxLds / resident);
}

// Workgroups that share a compute unit on the direct path: two where there are
// that many and the registers (at most 128 up to kPairTiles tiles) and half the
// LDS suffice, so that one's work fills the other's waits (585 frames of 3413
// birds on 35 x 87 cells, regions of 2 x 4 tiles: 76 us against 96).
int direct_resident(int rm, int rn, long long groups, int n_cus) {
    return rm * rn <= kPairTiles && groups > n_cus ? 2 : 1;
}

// Share of a frame's birds whose window of 2 j + 1 cells meets one region
// of `rows` grid rows, `nreg` regions along the axis: about 1 + 2 j / rows
// regions per bird, at most all of them.
double meet_share(int j, int rows, int nreg) {
    return std::min((double)nreg, 1.0 + 2.0 * j / rows) / (double)nreg;
}

long long axis_regions(int grid_n, int rows) { return (grid_n + rows - 1) / rows; }

// The kernel's cost model, in microseconds of one wave beside the other of its
// SIMD.  A 32-bird k-step costs its tile reads and its MFMAs, which did not
// overlap, and on the direct path its factors, by the axis of more chunks (by
// half of both, what a lane makes, the plan for 41 frames of 16408 birds on 151 x
// 107 cells took 145 us against 97, and over 500 drawn batches none gained);
// every block of 64 birds costs its test and staging on each region.  Least
// squares over 40 plans of three batches; on 244 others (1 .. 1800 frames of 20
// .. 30000 birds, even and in groups, 52 plans each) the plan it picks on the
// table path takes 2% more than the fastest on average.
constexpr double kGroupUs = 1.0;    // a workgroup's start on an item group
constexpr double kEdgeUs = 0.0135;  // a step's reads per row or column of tiles
constexpr double kMfmaUs = 0.0159;  // its MFMAs per tile
constexpr double kChunkUs = 0.113;  // its factors on the direct path, per chunk of four
constexpr double kBlockUs = 0.335;  // a 64-bird block
constexpr double kTileUs = 0.11;    // a tile's sum over an item's waves
constexpr double kUneven = 1.25;    // the fullest region of a single round against the average
constexpr double kLaunchUs = 5.0;   // launch and table build
constexpr double kSliceSumUs = 4.0; // the second kernel of a launch split into bird slices

// A shape on a grid: its regions, the birds an item keeps on average, and what
// a step costs it.
struct GatherCost {
    long long ry, rx;
    double kept, step;
};

GatherCost gather_regions(const Shape &sh, const GatherGeom &gg, int grid_w, int grid_h, double birds) {
    GatherCost g;
    g.ry = axis_regions(grid_h, 16 * sh.rm);
    g.rx = axis_regions(grid_w, 16 * sh.rn);
    g.kept = birds * meet_share(gg.ay.j, 16 * sh.rm, (int)g.ry) * meet_share(gg.ax.j, 16 * sh.rn, (int)g.rx);
    g.step = kEdgeUs * (sh.rm + sh.rn) + kMfmaUs * sh.rm * sh.rn;
    if (!gg.ay.c) g.step += kChunkUs * std::max(std::min(gg.ay.nc, 4 * sh.rm), std::min(gg.ax.nc, 4 * sh.rn));
    return g;
}

long long item_groups(const GatherCost &g, int waves, int split, long long n_frames) {
    return (n_frames * g.ry * g.rx * split * waves + kGWaves - 1) / kGWaves;
}

// Modelled time of a launch with `waves` waves per item and `split` bird
// slices.  A compute unit runs one workgroup at a time and takes its share of
// the item groups in turn; one round of workgroups ends with its fullest
// region (unless all eight waves share each region).
double gather_us(const Shape &sh, int waves, int split, const GatherCost &g, long long n_frames, double birds, int n_cus) {
    const long long groups = item_groups(g, waves, split, n_frames);
    const double share = (double)groups / n_cus;
    const double rounds = groups <= 4LL * n_cus ? (double)((groups + n_cus - 1) / n_cus) : share;
    const double per = 1.0 / (double)(waves * split);
    const double steps = g.kept * (rounds == 1.0 && waves < kGWaves ? kUneven : 1.0) * (1.0 / kGStep) * per + 0.5;
    return kLaunchUs + (split > 1 ? kSliceSumUs : 0.0) +
           rounds * (kGroupUs + steps * g.step + std::max(birds * (1.0 / 64.0) * per, 1.0) * kBlockUs +
                     (waves > 1 ? kTileUs * sh.rm * sh.rn : 0.0));
}

// Region shape and waves per item of least modelled time.  For a batch whose
// clustering (a compute unit per frame of about a thousand birds and more) takes
// an eighth to half of the chip, a plan of one round that leaves it room is
// preferred where it is within kNearly of the best and that one leaves less than
// half the room (47 frames of 7488 birds on 192 x 108 cells: 23.8 us with 212
// workgroups, 33.5 with 209 at most): a program that runs both at once otherwise
// waits for whichever finds the chip full (64 x 2000 birds on 128 x 72 cells, the
// whole step on two streams: 1.524M frames/s with 192 workgroups, 1.493M with
// 256, joined after every step 1.370M and 1.305M; this call alone 10.2 and 9.9
// us).
constexpr double kNearly = 1.14;  // the model holds such plans' regions for less even than most are

struct Choice {
    Shape shape;
    GatherCost cost;
    int waves;
    double us;
};

Choice gather_shape(const GatherGeom &gg, int grid_w, int grid_h, long long n_frames, double birds, int n_cus) {
    Choice best{}, beside{};
    best.us = beside.us = 1e300;
    const bool room = gg.ay.c && birds >= 1000.0 && 8 * n_frames >= n_cus && 2 * n_frames <= n_cus;
    for (const Shape &sh : kGShapes) {
        if (!gg.ay.c && sh.rm * sh.rn > kDirectTiles) continue;
        const GatherCost g = gather_regions(sh, gg, grid_w, grid_h, birds);
        for (int w = 1; w <= kGWaves; w *= 2) {
            const double us = gather_us(sh, w, 1, g, n_frames, birds, n_cus);
            if (us < best.us * 0.999) best = {sh, g, w, us};
            if (room && us < beside.us * 0.999 && item_groups(g, w, 1, n_frames) + n_frames <= n_cus) beside = {sh, g, w, us};
        }
    }
    const bool crowds = 2 * (n_cus - item_groups(best.cost, best.waves, 1, n_frames)) < n_frames;
    return crowds && beside.us <= kNearly * best.us ? beside : best;
}

// Region shape of a launch split into bird slices (at most 16 tiles, see
// plan_path): least modelled work per frame, whatever its spread.
Choice gather_split_shape(const GatherGeom &gg, int grid_w, int grid_h, double birds) {
    Choice best{};
    best.us = 1e300;
    for (const Shape &sh : kGShapes) {
        if (sh.rm * sh.rn > 16) continue;
        const GatherCost g = gather_regions(sh, gg, grid_w, grid_h, birds);
        const double us = (g.kept / kGStep * g.step + birds / 64.0 * kBlockUs + kGroupUs) * (double)(g.ry * g.rx);
        if (us < best.us * 0.999) best = {sh, g, 1, us};
    }
    return best;
}

int env_int(const char *name) {
    const char *v = std::getenv(name);
    return v ? std::atoi(v) : 0;
}

// Waves per work item and slices per (frame, region) of a launch that would
// leave most of the chip idle.  A compute unit holds kGWaves waves (two per
// SIMD).  Items are spread over as few waves as fill the chip (the smallest
// power of two w, at most kGWaves, with items * w >= resident waves): more
// waves per item only add fixed costs (a table build per workgroup, the final
// sum across waves).  `birds` is the birds an item keeps (those whose window
// meets its region), on average.  FLOCK_DENSITY_WAVES / FLOCK_DENSITY_SPLIT
// override (for tuning and tests).
struct GatherForce {
    int waves, split;  // 0: not forced
};

GatherForce gather_force() { return {env_int("FLOCK_DENSITY_WAVES"), env_int("FLOCK_DENSITY_SPLIT")}; }

void gather_split(int64_t n_frames, double birds, long long regions, int n_cus, const GatherForce &force, int *waves,
                  int *split) {
    const long long items = (long long)n_frames * regions;
    const long long resident = (long long)kGWaves * std::max(n_cus, 1);
    int w = 1;
    while (w < kGWaves && items * w < resident) w *= 2;
    // slices only while one launch would leave most of the chip idle (the
    // partial grids cost traffic), up to one round of waves, with at least
    // kGMinWaveBirds kept birds per wave
    long long sp = 1;
    if (2 * items * w < resident) {
        sp = resident / (items * w);
        sp = std::min<long long>(sp, std::max<long long>(1, (long long)(birds / (w * kGMinWaveBirds))));
        sp = std::min<long long>(sp, 64);
    }
    if (force.waves == 1 || force.waves == 2 || force.waves == 4 || force.waves == 8) w = force.waves;
    if (force.split >= 1 && force.split <= 64) sp = force.split;
    *waves = w;
    *split = (int)sp;
}

// Scratch of the allocation-free entry point (density_frames_noalloc): the
// partial grids of split launches, in a file-scope device array instead of a
// workspace.  Each device holds its own copy for the life of the process.
// In host code `scratch` names a host-side stand-in, never the device memory:
// its device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[kDensityScratchBytes];

constexpr int kScratchDevices = 64;
std::once_flag g_scratch_once[kScratchDevices];
void *g_scratch_ptr[kScratchDevices];
hipError_t g_scratch_err[kScratchDevices];

}  // namespace

hipError_t density_static_scratch(void **ptr) {
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
    std::call_once(g_scratch_once[dev], [dev] {
        void *p = nullptr;
        g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        g_scratch_ptr[dev] = g_scratch_err[dev] == hipSuccess ? p : nullptr;
    });
    *ptr = g_scratch_ptr[dev];
    return g_scratch_err[dev];
}

size_t density_workspace_bytes(int32_t n_frames, int32_t total, int32_t grid_w, int32_t grid_h, int n_cus) {
    if (n_frames <= 0 || grid_w < 1 || grid_h < 1) return 0;
    // the shape depends on the frame extent and sigma, which the query does
    // not know: bound the split over every shape, with every bird kept (a
    // split only shrinks when an item keeps fewer birds)
    const double birds = (double)total / n_frames;
    const GatherForce force = gather_force();
    int most = 1;
    for (const Shape &sh : kGShapes) {
        int waves = 1, split = 1;
        gather_split(n_frames, birds, axis_regions(grid_h, 16 * sh.rm) * axis_regions(grid_w, 16 * sh.rn), n_cus, force,
                     &waves, &split);
        most = std::max(most, split);
    }
    if (most <= 1) return 0;
    return (size_t)n_frames * most * (size_t)grid_w * grid_h * sizeof(float);
}

namespace {

// Where `room` holds fewer partial grids than the slices want there are fewer
// slices.  Room for less than two means none at all on grids that never needed
// a workspace (cells of no whole number of quanta, windows of more than
// kNeverSplit cells); on the others the caller refuses the plan.
constexpr int kNeverSplit = 30;

// The plan of one path: region shape, waves per item and bird slices of least
// modelled time.
struct PathPlan {
    Choice c;
    int split;
};

PathPlan plan_path(const DensityArgs &a, const GatherGeom &gg, bool whole, double birds, int n_cus, size_t room,
                   const Shape *forced, const GatherForce &over) {
    auto limit = [&](int slices) {
        const size_t most = room / ((size_t)a.n_frames * a.grid_w * a.grid_h * sizeof(float));
        if (slices <= 1 || (size_t)slices <= most) return slices;
        const bool optional = !whole || std::max(gg.ay.j, gg.ax.j) > kNeverSplit;
        if (over.split >= 1) return optional ? 1 : slices;
        return most >= 2 ? (int)most : optional ? 1 : slices;
    };
    if (forced && (gg.ay.c || forced->rm * forced->rn <= kDirectTiles)) {
        PathPlan p{{*forced, gather_regions(*forced, gg, a.grid_w, a.grid_h, birds), 1, 0.0}, 1};
        gather_split(a.n_frames, p.c.cost.kept, p.c.cost.ry * p.c.cost.rx, n_cus, over, &p.c.waves, &p.split);
        p.split = limit(p.split);
        return p;
    }
    PathPlan p{gather_shape(gg, a.grid_w, a.grid_h, a.n_frames, birds, n_cus), 1};
    // bird slices where they pay for the second kernel: a launch that would
    // leave most of the chip idle is bound by each wave's own path, whose
    // fixed part grows with the tiles an item's waves add up at the end
    // (kGRedTiles per round); shapes of at most 16 tiles keep that to two
    // rounds
    PathPlan s{gather_split_shape(gg, a.grid_w, a.grid_h, birds), 1};
    gather_split(a.n_frames, s.c.cost.kept, s.c.cost.ry * s.c.cost.rx, n_cus, over, &s.c.waves, &s.split);
    const int asked = s.split;
    s.split = limit(s.split);
    s.c.us = gather_us(s.c.shape, s.c.waves, s.split, s.c.cost, a.n_frames, birds, n_cus);
    if ((s.split > 1 || asked == 1) && (over.split >= 1 || over.waves >= 1 || (s.split > 1 && s.c.us < p.c.us))) return s;
    return p;
}

}  // namespace

// The launch plan.  The table path where its tables fit, but for launches of so
// few steps (two per compute unit, no slices) that their exponentials cost less
// than a table build of several passes: on 96 x 54 cells, sigma 45 px, 127 birds
// in one frame 4.5 against 6.6 us, 16 frames of 200 (300 steps) 5.1 and 6.9, 16 of
// 2000 (2500 steps) 9.3 and 9.0; 8000 birds in one frame, split, 11.4 and 9.7.
// FLOCK_DENSITY_PATH=direct (or recur) and =table force the path where both
// apply, FLOCK_DENSITY_SHAPE="rm,rn" the region shape (for tests and tuning).
DensityPlan plan_density(const DensityArgs &a, int n_cus, size_t room) {
    n_cus = std::max(n_cus, 1);
    const char *path = std::getenv("FLOCK_DENSITY_PATH"), *force = std::getenv("FLOCK_DENSITY_SHAPE");
    const bool direct = path && (std::strcmp(path, "direct") == 0 || std::strcmp(path, "recur") == 0);
    const GatherForce over = gather_force();
    Shape given{};
    bool forced = false;
    if (force && std::sscanf(force, "%d,%d", &given.rm, &given.rn) == 2)
        for (const Shape &k : kGShapes) forced |= k.rm == given.rm && k.rn == given.rn;
    const double birds = a.n_frames > 0 ? (double)a.total / a.n_frames : 0.0;
    GatherGeom gg;
    base_geom(a, &gg);
    GatherGeom tg = gg;
    const bool whole = table_geom(a, &tg);
    DensityPlan p{};
    PathPlan pp{};
    p.tables = whole && !direct;
    if (p.tables) {
        pp = plan_path(a, tg, whole, birds, n_cus, room, forced ? &given : nullptr, over);
        // every thread makes two chunks of four rows per pass of a table build
        const int passes = (tg.ay.c * ((tg.ay.nc + 2) / 2) + kGThreads - 1) / kGThreads;
        const double steps = (double)a.n_frames * pp.c.cost.ry * pp.c.cost.rx * pp.c.cost.kept / kGStep;
        if (!path && !forced && over.split < 1 && over.waves < 1 && passes > 1 && pp.split == 1 && steps <= 2.0 * n_cus) {
            pp = plan_path(a, gg, whole, birds, n_cus, room, nullptr, over);
            p.tables = false;
        }
    } else {
        pp = plan_path(a, gg, whole, birds, n_cus, room, forced ? &given : nullptr, over);
    }
    p.rm = pp.c.shape.rm;
    p.rn = pp.c.shape.rn;
    p.regions_y = (int)pp.c.cost.ry;
    p.regions_x = (int)pp.c.cost.rx;
    p.waves = pp.c.waves;
    p.split = pp.split;
    const long long items = (long long)a.n_frames * p.regions_y * p.regions_x * p.split;
    const int per_wg = kGWaves / p.waves;
    p.resident = p.tables ? 1 : direct_resident(p.rm, p.rn, (items + per_wg - 1) / per_wg, n_cus);
    if (!p.tables) direct_lds(&gg, p.rm, p.rn, p.resident);
    p.lds_bytes = (size_t)(p.tables ? tg : gg).lds_bytes;
    if (items > 0xffffffffLL) {  // item numbers are 32 bits wide: refused by the caller's check of `blocks`
        p.blocks = items;
        return p;
    }
    // a workgroup takes its share of the item groups one after another, with
    // one table build: 256 x 8000 with eight waves per item took 91 against
    // 103 us with a workgroup per group
    p.blocks = std::min<long long>((items + per_wg - 1) / per_wg, (long long)n_cus * p.resident);
    return p;
}

hipError_t launch_density(const DensityArgs &a, const DensityPlan &p, float *partial, hipStream_t stream) {
    GatherGeom gg;
    base_geom(a, &gg);
    if (!p.tables) direct_lds(&gg, p.rm, p.rn, p.resident);
    else if (!table_geom(a, &gg)) return hipErrorInvalidValue;
    if (p.split > 1 && !partial) return hipErrorInvalidValue;
    const uint32_t items = (uint32_t)((long long)a.n_frames * p.regions_y * p.regions_x * p.split);
    hipError_t err = hipErrorInvalidValue;
    // Lanes of an axis each where both windows have the same number of chunks (an
    // odd one; halves of both would take one chunk more): 120 frames of 16664 birds
    // on 29 x 27 cells, windows of 3 chunks, 29.4 us against 33.2.  An instance of its
    // own: beside the other form in one kernel it made the shortest launches wait
    // for more code (4.9 to 5.3 us).
    const bool axes = !p.tables && gg.ay.nc == gg.ax.nc && gg.ay.nc < 4 * p.rm && gg.ax.nc < 4 * p.rn;
#define FLOCK_LAUNCH(TM, TN, DIRECT, AXES)                                                                        \
    hipLaunchKernelGGL((density_gather_kernel<TM, TN, DIRECT, AXES>), dim3((unsigned)p.blocks), dim3(kGThreads),  \
                       p.lds_bytes, stream, a, gg, p.regions_y, p.regions_x, p.split, p.waves, items, partial)
#define FLOCK_GSHAPE(TM, TN)                                                                                      \
    if (p.rm == TM && p.rn == TN) {                                                                               \
        constexpr bool kDirect = TM * TN <= kDirectTiles;                                                         \
        if (p.tables) FLOCK_LAUNCH(TM, TN, false, false);                                                         \
        else if (kDirect && axes) FLOCK_LAUNCH(TM, TN, kDirect, kDirect);                                         \
        else if (kDirect) FLOCK_LAUNCH(TM, TN, kDirect, false);                                                   \
        else return hipErrorInvalidValue;                                                                         \
        err = hipGetLastError();                                                                                  \
    }
    FLOCK_GSHAPE(1, 1) FLOCK_GSHAPE(2, 2) FLOCK_GSHAPE(1, 4) FLOCK_GSHAPE(4, 1) FLOCK_GSHAPE(2, 4)
    FLOCK_GSHAPE(4, 2) FLOCK_GSHAPE(3, 4) FLOCK_GSHAPE(4, 4) FLOCK_GSHAPE(5, 4)
    FLOCK_GSHAPE(9, 2) FLOCK_GSHAPE(9, 4) FLOCK_GSHAPE(3, 8) FLOCK_GSHAPE(4, 8)
#undef FLOCK_GSHAPE
#undef FLOCK_LAUNCH
    if (err != hipSuccess || p.split <= 1) return err;
    const int64_t cells = (int64_t)a.grid_h * a.grid_w;
    const int64_t total = cells * a.n_frames;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(density_reduce_kernel, dim3(blocks), dim3(256), 0, stream, a.density, partial, cells, total,
                       p.split, gg.scale);
    return hipGetLastError();
}

}  // namespace flock
