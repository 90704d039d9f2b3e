// heatmap.hip - heatmap analytics of density grids on gfx950.
//
// What is computed (the clustering module of Section 2.3 thresholds the
// density heatmaps and applies connected component analysis; Algorithm 1
// computes the heatmap, its entropy and a clustering degree per frame):
//   hot cell     density >= threshold;
//   component    connected hot cells under the 4-neighbourhood (shared edge)
//                or the 8-neighbourhood (shared edge or corner), labelled by
//                its smallest row-major cell index gy * grid_w + gx; cold
//                cells get -1;
//   per component  cells and mass = cell_area * sum of density, stored at
//                the label cell (0 elsewhere);
//   entropy      -sum p ln p over positive cells, p = density / S, S the sum
//                of the positive cells (0 when S = 0);
//   degree       (sum of density over hot cells) / S (0 when S = 0).
//
// Design.  Grids whose int32 forest fits in LDS beside the component slots
// (grid_w * grid_h <= 39,936 cells with 160 KiB) take
// heat_frame_kernel, one workgroup per frame (described there).  Larger grids
// take four tiled kernels:
//   1. heat_tile_kernel, one 256-thread workgroup per 32 x 32 tile: loads the
//      tile once, unites hot neighbours inside the tile in LDS (smallest
//      index hooking), writes each hot cell's tile root (frame index) into
//      `labels` as a forest, clears the component outputs and writes the
//      tile's partial sums (S, sum D ln D, hot sum, largest D) in a fixed
//      order;
//   2. heat_merge_kernel: threads on tile boundary cells unite hot pairs that
//      cross a tile edge in the global forest (agent-scope CAS hooking, the
//      smaller root wins); extra workgroups add each frame's tile partials in
//      tile order into entropy and degree and pick the frame's fixed-point
//      scale;
//   3. heat_label_kernel, per tile again: each hot cell walks to its root and
//      stores it; cells and fixed-point mass are summed per root in an LDS
//      table, then added once per (tile, root) to the root's outputs (integer
//      atomics, so the sums do not depend on their order);
//   4. heat_mass_kernel: the root cells turn their fixed-point mass into
//      cell_area * sum.
// Every output is a deterministic function of the input.

#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>

#include "cluster_common.h"
#include "internal.h"
#include "ln_table.h"

namespace flock {
namespace {

using namespace cl;

constexpr int kHT = 32;                 // tile side, cells
constexpr int kHThreads = 256;          // 4 cells per thread
constexpr int kHRows = kHThreads / kHT; // rows per pass
constexpr int kHTable = 1024;           // LDS table slots for (root -> sums) per tile

struct TilePart {
    double s, e, hot;  // sum D, sum D ln D over positive cells; sum D over hot cells
    uint32_t maxbits;  // largest positive D, as its float bits (0 if none)
    uint32_t pad;
};

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}

__device__ const LnTable kLnTable = make_ln_table();

// Copied to LDS by the first 2 kLnBuckets threads; the caller syncs before use.
__device__ __forceinline__ void ln_table_load(LnTable &t) {
    const int k = threadIdx.x;
    if (k < 2 * kLnBuckets) reinterpret_cast<double *>(&t)[k] = reinterpret_cast<const double *>(&kLnTable)[k];
}

// Natural log of a positive float in fp64, from a table of bucket centres:
// v = m 2^e exactly (m in [1, 2)), c is the centre of m's bucket of width
// 1/kLnBuckets, and ln v = e ln 2 + ln c + ln(1 + r) with r = m / c - 1,
// |r| <= 2^-8, formed as fma(m, 1/c, -1); ln(1 + r) is its Taylor series
// through r^7 (truncation below 2^-67).  The absolute error is a few 1e-16
// (ln 2 and the table entries are rounded to fp64; |e| <= 149), about the
// library routine's, at a fraction of its instructions.
__device__ __forceinline__ double ln_pos(float vf, const LnTable &t) {
    const uint64_t b = (uint64_t)__double_as_longlong((double)vf);
    const int e = (int)(b >> 52) - 1023;
    const int k = (int)((b >> 45) & (kLnBuckets - 1));
    const double m = __longlong_as_double((long long)((b & 0x000fffffffffffffull) | 0x3ff0000000000000ull));
    const double r = fma(m, t.inv_c[k], -1.0);
    // explicit fused steps: every kernel that sums logarithms gets the same bits
    double p = fma(r, 1.0 / 7.0, -1.0 / 6.0);
    p = fma(r, p, 0.2);
    p = fma(r, p, -0.25);
    p = fma(r, p, 1.0 / 3.0);
    p = fma(r, p, -0.5);
    p = fma(r, p, 1.0);
    return fma((double)e, 0.69314718055994530942, fma(r, p, t.ln_c[k]));
}

struct TileGeom {
    int f, x0, y0, w, h;
};

__device__ __forceinline__ TileGeom tile_of(const HeatArgs &a, long long b) {
    const long long per = (long long)a.tiles_x * a.tiles_y;
    TileGeom t;
    t.f = (int)(b / per);
    const int r = (int)(b - (long long)t.f * per);
    t.y0 = (r / a.tiles_x) * kHT;
    t.x0 = (r % a.tiles_x) * kHT;
    t.w = min(kHT, a.grid_w - t.x0);
    t.h = min(kHT, a.grid_h - t.y0);
    return t;
}

__global__ __launch_bounds__(kHThreads) void heat_tile_kernel(HeatArgs a, TilePart *part) {
    __shared__ int32_t par[kHT * kHT];
    __shared__ uint32_t s_row[kHT + 1];  // hot bits of the tile's rows, and a row of zeros
    __shared__ double s_red[3][kHThreads / 64];
    __shared__ uint32_t s_max[kHThreads / 64];
    __shared__ LnTable lnt;
    ln_table_load(lnt);
    __syncthreads();
    const TileGeom t = tile_of(a, blockIdx.x);
    const int tid = threadIdx.x, lx = tid % kHT, ly0 = tid / kHT;
    const size_t cells = (size_t)a.grid_w * a.grid_h;
    const float *D = a.density + (size_t)t.f * cells;

    double s = 0.0, e = 0.0, hs = 0.0;
    uint32_t mb = 0;
    float v[kHT / kHRows];
    bool hot[kHT / kHRows];
#pragma unroll
    for (int k = 0; k < kHT / kHRows; ++k) {
        const int ly = ly0 + kHRows * k, l = ly * kHT + lx;
        const bool in = lx < t.w && ly < t.h;
        const size_t c = (size_t)(t.y0 + ly) * a.grid_w + t.x0 + lx;
        v[k] = in ? D[c] : 0.0f;
        hot[k] = in && v[k] >= a.threshold;
        // a wave holds two rows: every hot cell points at its run's first cell
        const uint64_t hm = __ballot(hot[k]);
        const uint32_t rb = (uint32_t)(lx == (int)(tid & 63) ? hm : hm >> 32);
        const uint32_t cold = ~rb & ((1u << lx) - 1u);
        par[l] = hot[k] && cold ? ly * kHT + 32 - __clz((int)cold) : hot[k] ? ly * kHT : l;
        if (lx == 0) s_row[ly] = rb;
        if (v[k] > 0.0f) {
            s += (double)v[k];
            e += (double)v[k] * ln_pos(v[k], lnt);
            mb = max(mb, __float_as_uint(v[k]));
        }
        if (hot[k]) hs += (double)v[k];
        if (in) {
            a.comp_cells[(size_t)t.f * cells + c] = 0;
            a.comp_mass[(size_t)t.f * cells + c] = 0.0;
        }
    }
    if (tid == 0) s_row[kHT] = 0u;
    __syncthreads();
    // joins between consecutive rows, from their bits: a vertical pair only at
    // the first of consecutive ones (the others join the same two runs), for
    // the 8-neighbourhood a diagonal pair only where neither of the cells
    // between them is hot.  (Uniting every hot cell with its two or four
    // neighbours made the cells of one large component contend: 18.5 us of a
    // 512 x 288 grid's call, now 9.5.)
#pragma unroll
    for (int k = 0; k < kHT / kHRows; ++k) {
        if (!hot[k]) continue;
        const int ly = ly0 + kHRows * k, l = ly * kHT + lx;
        const uint32_t up = s_row[ly], dn = s_row[ly + 1], both = up & dn;
        if (((both & ~(both << 1)) >> lx) & 1u) uf_unite<kGroup>(par, l, l + kHT);
        if (a.connectivity == 8 && !((dn >> lx) & 1u)) {
            if ((((dn & ~up) >> 1) >> lx) & 1u) uf_unite<kGroup>(par, l, l + kHT + 1);
            if (((dn & ~up) << 1 >> lx) & 1u) uf_unite<kGroup>(par, l, l + kHT - 1);
        }
    }
    __syncthreads();
    // each hot cell's tile root (a smaller tile index is a smaller frame
    // index) starts the global forest; cold cells are -1
    int32_t *L = a.labels + (size_t)t.f * cells;
#pragma unroll
    for (int k = 0; k < kHT / kHRows; ++k) {
        const int ly = ly0 + kHRows * k;
        if (!(lx < t.w && ly < t.h)) continue;
        const size_t c = (size_t)(t.y0 + ly) * a.grid_w + t.x0 + lx;
        int32_t lab = -1;
        if (hot[k]) {
            const int r = uf_root<kGroup>(par, ly * kHT + lx);
            lab = (t.y0 + r / kHT) * a.grid_w + t.x0 + r % kHT;
        }
        L[c] = lab;
    }
    // the tile's partial sums, in a fixed order
    s = wave_sum_d(s);
    e = wave_sum_d(e);
    hs = wave_sum_d(hs);
    mb = wave_max_u(mb);
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
        s_red[0][wave] = s;
        s_red[1][wave] = e;
        s_red[2][wave] = hs;
        s_max[wave] = mb;
    }
    __syncthreads();
    if (tid == 0) {
        TilePart p{0.0, 0.0, 0.0, 0u, 0u};
        for (int w = 0; w < kHThreads / 64; ++w) {
            p.s += s_red[0][w];
            p.e += s_red[1][w];
            p.hot += s_red[2][w];
            p.maxbits = max(p.maxbits, s_max[w]);
        }
        part[blockIdx.x] = p;
    }
}

// Crossing forward edges of cell (gx, gy): right, down, down-left,
// down-right (the last two for the 8-neighbourhood), where the neighbour
// lies in another tile.  An edge is left out where the cells beside it join
// its ends anyway: a straight one whose parallel one step back is there too
// (the two cells on either side of it are neighbours), a diagonal one with a
// hot cell between its ends.
__device__ __forceinline__ void merge_cell(const HeatArgs &a, int f, int gx, int gy) {
    const size_t cells = (size_t)a.grid_w * a.grid_h;
    const float *D = a.density + (size_t)f * cells;
    const int32_t c = gy * a.grid_w + gx;
    if (!(D[c] >= a.threshold)) return;
    int32_t *L = a.labels + (size_t)f * cells;
    const bool xe = (gx % kHT) == kHT - 1, x0 = (gx % kHT) == 0, ye = (gy % kHT) == kHT - 1;
    // (the edges across a vertical seam look back within the tile only, so
    // that the four edges around a tile corner never all lean on each other)
    const bool left = gx > 0, right = gx + 1 < a.grid_w, same = gy % kHT != 0, below = gy + 1 < a.grid_h;
    auto hot = [&](bool in, int d) { return in && D[c + (in ? d : 0)] >= a.threshold; };
    const int w = a.grid_w;
    const bool r = hot(right, 1), l = hot(left, -1), d = hot(below, w);
    if (xe && r && !(hot(same, -w) && hot(same, 1 - w))) uf_unite<kAgent>(L, c, c + 1);
    if (ye && d && !(l && hot(left, w - 1))) uf_unite<kAgent>(L, c, c + w);
    if (a.connectivity == 8 && below && !d) {
        if ((x0 || ye) && !l && hot(left, w - 1)) uf_unite<kAgent>(L, c, c + w - 1);
        if ((xe || ye) && !r && hot(right, w + 1)) uf_unite<kAgent>(L, c, c + w + 1);
    }
}

__global__ __launch_bounds__(256) void heat_merge_kernel(HeatArgs a, const TilePart *part, int32_t *shift,
                                                         long long merge_blocks) {
    const int tid = threadIdx.x;
    if ((long long)blockIdx.x < merge_blocks) {
        // boundary cells of every frame: for each inner vertical tile edge
        // its two columns, for each inner horizontal edge its upper row
        const long long nv = 2LL * (a.tiles_x - 1) * a.grid_h, nh = (long long)(a.tiles_y - 1) * a.grid_w;
        const long long per = nv + nh;
        const long long i = (long long)blockIdx.x * 256 + tid;
        if (i >= per * a.n_frames) return;
        const int f = (int)(i / per);
        const long long j = i - (long long)f * per;
        int gx, gy;
        if (j < nv) {
            const long long k = j / (2LL * a.grid_h);
            const int side = (int)((j / a.grid_h) % 2);
            gx = (int)(kHT * (k + 1) - 1 + side);
            gy = (int)(j % a.grid_h);
        } else {
            const long long jj = j - nv;
            gy = (int)(kHT * (jj / a.grid_w + 1) - 1);
            gx = (int)(jj % a.grid_w);
        }
        merge_cell(a, f, gx, gy);
        return;
    }
    // one workgroup per frame: tile partials in tile order (strided per lane,
    // then a fixed shuffle tree), entropy, degree, the fixed-point scale
    const int f = (int)((long long)blockIdx.x - merge_blocks);
    if (tid >= 64) return;
    const long long per = (long long)a.tiles_x * a.tiles_y;
    const TilePart *P = part + (size_t)f * per;
    double s = 0.0, e = 0.0, hs = 0.0;
    uint32_t mb = 0;
    for (long long k = tid; k < per; k += 64) {
        s += P[k].s;
        e += P[k].e;
        hs += P[k].hot;
        mb = max(mb, P[k].maxbits);
    }
    s = wave_sum_d(s);
    e = wave_sum_d(e);
    hs = wave_sum_d(hs);
    mb = wave_max_u(mb);
    if (tid == 0) {
        a.entropy[f] = s > 0.0 ? log(s) - e / s : 0.0;
        a.degree[f] = s > 0.0 ? hs / s : 0.0;
        a.n_components[f] = 0;
        // every positive D is below 2^(E + 1), E its float exponent; with
        // 2^lg >= cells, D * 2^sh with sh = 62 - (E + 1) - lg keeps any sum of
        // cells below 2^62
        const int E = mb ? (int)((mb >> 23) & 0xffu) - 127 : 0;
        int lg = 0;
        while ((1LL << lg) < (long long)a.grid_w * a.grid_h) ++lg;
        shift[f] = 62 - (max(E, -126) + 1) - lg;
    }
}

__device__ __forceinline__ uint32_t slot_hash(int32_t root) { return ((uint32_t)root * 2654435761u) >> 22; }

__global__ __launch_bounds__(kHThreads) void heat_label_kernel(HeatArgs a, const int32_t *shift) {
    __shared__ int32_t keys[kHTable];
    __shared__ int32_t cnt[kHTable];
    __shared__ unsigned long long mass[kHTable];
    const TileGeom t = tile_of(a, blockIdx.x);
    const int tid = threadIdx.x, lx = tid % kHT, ly0 = tid / kHT;
    for (int k = tid; k < kHTable; k += kHThreads) {
        keys[k] = -1;
        cnt[k] = 0;
        mass[k] = 0ull;
    }
    __syncthreads();
    const size_t cells = (size_t)a.grid_w * a.grid_h;
    const float *D = a.density + (size_t)t.f * cells;
    int32_t *L = a.labels + (size_t)t.f * cells;
    const int sh = shift[t.f];
#pragma unroll
    for (int k = 0; k < kHT / kHRows; ++k) {
        const int ly = ly0 + kHRows * k;
        if (!(lx < t.w && ly < t.h)) continue;
        const int32_t c = (t.y0 + ly) * a.grid_w + t.x0 + lx;
        const float v = D[c];
        if (!(v >= a.threshold)) continue;
        // read-only walk: concurrent writers only store roots
        const int32_t root = uf_root<kAgent>(L, c);
        st_rlx<kAgent>(L + c, root);
        if (root == c) atomicAdd(a.n_components + t.f, 1);
        const unsigned long long q = (unsigned long long)llrint(ldexp((double)v, sh));
        // this root's slot in the tile table (linear probing; a tile has at
        // most kHT * kHT = kHTable distinct roots, so a slot is always found)
        uint32_t h = slot_hash(root);
        for (;;) {
            const int32_t old = atomicCAS(keys + h, -1, root);
            if (old == -1 || old == root) break;
            h = (h + 1) & (kHTable - 1);
        }
        atomicAdd(cnt + h, 1);
        atomicAdd(mass + h, q);
    }
    __syncthreads();
    int32_t *CC = a.comp_cells + (size_t)t.f * cells;
    unsigned long long *CM = reinterpret_cast<unsigned long long *>(a.comp_mass + (size_t)t.f * cells);
    for (int k = tid; k < kHTable; k += kHThreads) {
        const int32_t root = keys[k];
        if (root < 0) continue;
        atomicAdd(CC + root, cnt[k]);
        atomicAdd(CM + root, mass[k]);
    }
}

__global__ __launch_bounds__(256) void heat_mass_kernel(HeatArgs a, const int32_t *shift) {
    const size_t cells = (size_t)a.grid_w * a.grid_h;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= cells * (size_t)a.n_frames) return;
    const int f = (int)(i / cells);
    const int32_t c = (int32_t)(i - (size_t)f * cells);
    if (a.labels[i] != c) return;  // not a component's label cell
    const unsigned long long q = reinterpret_cast<const unsigned long long *>(a.comp_mass)[i];
    a.comp_mass[i] = ldexp((double)q, -shift[f]) * a.cell_area;
}

// ---------------------------------------------------------------------------
// Frame-resident path: one workgroup per frame, the whole grid's forest in LDS
// ---------------------------------------------------------------------------


// v of the lane `SHIFT` lanes below in the row of 16 (DPP control CTRL), 0
// where there is none.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_or_zero(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false);
    return ((unsigned long long)hi << 32) | lo;
}

// Inclusive prefix sum over the wave (64-bit values), by DPP: shifts of 1, 2,
// 4 and 8 lanes within the rows of 16, then the last lane of a row broadcast
// to the next row (rows 1 and 3), and of the lower half to the upper.
__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v) {
    v += dpp_or_zero<0x111, 0xf>(v);
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}

// Sum over the wave in the prefix sum's fixed order, in every lane.
__device__ __forceinline__ double wave_sum_dpp(double v) {
    auto shifted = [](double x, auto ctrl, auto rows) {
        return __longlong_as_double(
            (long long)dpp_or_zero<decltype(ctrl)::value, decltype(rows)::value>((unsigned long long)__double_as_longlong(x)));
    };
    using std::integral_constant;
    v += shifted(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});
    v += shifted(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    v += shifted(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    v += shifted(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    v += shifted(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});
    v += shifted(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Waits for this wave's memory operations: its stores and atomics have then
// reached the L2, where the workgroup's later atomics and uncached loads meet
// them.
__device__ __forceinline__ void wait_memory() { __builtin_amdgcn_s_waitcnt(0); }

// A value equal in every lane, as a scalar.
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
}

// LDS of one frame: the forest (an int32 per cell), two bits per cell in words
// of 64 consecutive cells (hot; first of its row; zero words past the end, as
// many as a read one row down needs), and the component slots, as many as are
// left, at most kMaxSlots.  Where fewer than kMinSlots would be (`spill`) the
// words wait in the frame's part of comp_mass instead, up to phase D.
constexpr int kMaxSlots = 2048, kMinSlots = 256, kMinSpillSlots = 96;
constexpr size_t kFrameStaticLds = 2560;  // at least the kernel's static shared variables
struct FrameLds {
    int words, padded;
    size_t hot, row0, slot;  // byte offsets
    __host__ __device__ size_t bytes(int slots) const { return slot + (size_t)slots * 16; }
};

__host__ __device__ inline FrameLds frame_lds(int gw, int gh, bool spill) {
    FrameLds l;
    l.words = (gw * gh + 63) / 64;
    l.padded = l.words + gw / 64 + 3;
    l.hot = ((size_t)gw * gh * sizeof(int32_t) + 15) / 16 * 16;
    l.row0 = l.hot + (size_t)l.padded * 8;
    l.slot = spill ? l.hot : (l.row0 + (size_t)l.padded * 8 + 15) / 16 * 16;
    return l;
}

// One frame per workgroup, the cells in words of 64 whatever the
// grid's width.  A wave takes every kFWaves-th word, kFlight of them at a time:
//   A. the partial sums, and each word's hot bits by ballot: every hot cell
//      points at the first cell of its horizontal run within the word (no
//      atomics);
//   B. joins, found from the bits by a thread per word: a run continued from
//      the word before, a vertical pair only at the first of consecutive ones
//      (the others join the same two runs), and for the 8-neighbourhood a
//      diagonal pair only where neither of the cells between them is hot;
//      queued and joined a thread each, while one thread turns the sums
//      (added in a fixed order) into entropy, degree and the fixed-point
//      scale;
//   C. every run's first cell points at its root, and roots take component
//      slots;
//   D. labels, and the outputs' zeros; per word, the runs' cell counts and
//      fixed-point masses by one prefix sum, each added to its component's
//      slot;
//   E. the slots' totals go to their label cells.
// Components beyond the slots add their runs to their label cells' outputs by
// global atomics, on outputs zeroed beforehand, and E converts those masses:
// 256 noisy frames of 256 x 144 cells with 2400 components each take 115 us,
// 254 when D ran again for every further 281 components, 187 when D left only
// the label cells out of its zeros.
//
// Bound by latency: the chain of phases on one compute unit per frame.
// 64 frames of 128 x 72 cells 23.1 us, 256 of 256 x 144 61, 600 of 128 x 72
// 55 (31.5, 102 and 69 when the logarithm table was computed by every
// workgroup, loads came one at a time, every cell tested its own joins, masses
// were added by global atomics and a second kernel converted them).
template <int kFThreads, bool SPILL>
__global__ __launch_bounds__(kFThreads) void heat_frame_kernel(HeatArgs a, int slots) {
    constexpr int kFWaves = kFThreads / 64;
    // the sums' order is that of kSumWaves waves whatever the workgroup's size
    // (a frame's bits do not depend on its batch): a wave of a smaller one adds
    // the words of kShares such waves apart
    constexpr int kSumWaves = 16, kShares = kSumWaves / kFWaves;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_red[3][kSumWaves];
    __shared__ uint32_t s_max[kFWaves];
    __shared__ int s_shift, s_ncomp, s_nq;
    __shared__ LnTable lnt;
    constexpr int kFlight = 3;
    const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gw = a.grid_w, gh = a.grid_h;
    const int cells = gw * gh;
    const FrameLds l = frame_lds(gw, gh, SPILL);
    int32_t *P = reinterpret_cast<int32_t *>(smem);
    unsigned long long *mass = reinterpret_cast<unsigned long long *>(smem + l.slot);
    int32_t *count = reinterpret_cast<int32_t *>(mass + slots), *label = count + slots;
    const float *D = a.density + (size_t)f * cells;
    int32_t *L = a.labels + (size_t)f * cells;
    int32_t *CC = a.comp_cells + (size_t)f * cells;
    double *CM = a.comp_mass + (size_t)f * cells;
    unsigned long long *CMu = reinterpret_cast<unsigned long long *>(CM);
    uint64_t *hotw, *row0w;
    if constexpr (SPILL) {
        hotw = reinterpret_cast<uint64_t *>(CM);  // 2 padded words: at most cells / 16
        row0w = hotw + l.padded;
    } else {
        hotw = reinterpret_cast<uint64_t *>(smem + l.hot);
        row0w = reinterpret_cast<uint64_t *>(smem + l.row0);
    }
    auto load = [&](int word) { return D[min(64 * word + lane, cells - 1)]; };  // past the end: not used

    // A
    ln_table_load(lnt);
    float v[kFlight];
#pragma unroll
    for (int u = 0; u < kFlight; ++u) v[u] = load(min(wave + kFWaves * u, l.words));
    if (tid == 0) s_ncomp = s_nq = 0;
    for (int i = l.words + tid; i < l.padded; i += kFThreads) hotw[i] = row0w[i] = 0ull;
    int x = (64 * wave + lane) % gw;              // column of this lane's cell
    const int xstep = (64 * kFWaves) % gw;
    __syncthreads();
    static_assert(kShares == 1 || (kShares == 2 && kFlight % 2 == 1), "the shares change places every kFlight words");
    double s[kShares], e[kShares], hs[kShares];  // [k]: this wave's words of the next place k, k + kShares, ..
#pragma unroll
    for (int k = 0; k < kShares; ++k) s[k] = e[k] = hs[k] = 0.0;
    auto change = [&] {
        if constexpr (kShares == 2) {
            const double t0 = s[0], t1 = e[0], t2 = hs[0];
            s[0] = s[1], e[0] = e[1], hs[0] = hs[1];
            s[1] = t0, e[1] = t1, hs[1] = t2;
        }
    };
    bool changed = false;
    uint32_t mb = 0;
    for (int w0 = wave; w0 < l.words; w0 += kFWaves * kFlight) {
        double ln[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) ln[u] = ln_pos(v[u] > 0.0f ? v[u] : 1.0f, lnt);
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int w = w0 + kFWaves * u, c = 64 * w + lane;
            const float d = v[u];
            v[u] = load(min(w + kFWaves * kFlight, l.words));
            const bool in = c < cells, hot = in & (d >= a.threshold), pos = in & (d > 0.0f);
            constexpr int kLast = kShares - 1;
            s[u & kLast] += pos ? (double)d : 0.0;
            e[u & kLast] = fma(pos ? (double)d : 0.0, ln[u], e[u & kLast]);
            mb = max(mb, pos ? __float_as_uint(d) : 0u);
            hs[u & kLast] += hot ? (double)d : 0.0;
            const uint64_t hm = __ballot(hot), r0 = __ballot(in & (x == 0));
            // first cells of the word's runs, and this lane's run's
            const uint64_t first = hm & ~((hm << 1) & ~r0);
            const uint64_t upto = first & (~0ull >> (63 - lane));
            if (in) P[c] = hot ? 64 * w + 63 - __clzll(upto) : -1;
            if (lane == 0 && w < l.words) {
                hotw[w] = hm;
                row0w[w] = r0;
            }
            x += xstep;
            x -= x >= gw ? gw : 0;
        }
        change();
        changed = !changed;
    }
    if (changed) change();
#pragma unroll
    for (int k = 0; k < kShares; ++k) {
        const double ws = wave_sum_dpp(s[k]), we = wave_sum_dpp(e[k]), wh = wave_sum_dpp(hs[k]);
        if (lane == 0) {
            s_red[0][wave + kFWaves * k] = ws;
            s_red[1][wave + kFWaves * k] = we;
            s_red[2][wave + kFWaves * k] = wh;
        }
    }
    mb = wave_max_u(mb);
    if (lane == 0) s_max[wave] = mb;
    if constexpr (SPILL) wait_memory();
    __syncthreads();
    // B (the queue is in the slots' space; pairs beyond it are joined in place)
    int2 *queue = reinterpret_cast<int2 *>(smem + l.slot);
    const int qcap = 2 * slots;
    // the 64 bits from bit b on
    auto bits = [&](int b) {
        const int i = b >> 6, o = b & 63;
        return (hotw[i] >> o) | (o ? hotw[i + 1] << (64 - o) : 0ull);
    };
    for (int i = tid; i < l.words; i += kFThreads) {
        const uint64_t m = hotw[i];
        if (m == 0ull) continue;
        const uint64_t r0 = row0w[i], last = (r0 >> 1) | (row0w[i + 1] << 63);  // cells before the next row's first
        const uint64_t before = i > 0 ? hotw[i - 1] >> 63 : 0ull;
        const uint64_t lh = ((m << 1) | before) & ~r0, rh = ((m >> 1) | (hotw[i + 1] << 63)) & ~last;  // left, right hot
        const uint64_t dn = bits(64 * i + gw), dl = bits(64 * i + gw - 1) & ~r0, dr = bits(64 * i + gw + 1) & ~last;
        const uint64_t join = m & lh & 1ull;
        const uint64_t down = m & dn & ~(lh & dl);
        const uint64_t alone = a.connectivity == 8 ? m & ~dn : 0ull;  // cold below
        const uint64_t right = alone & dr & ~rh, left = alone & dl & ~lh;
        const int pairs = __popcll(join) + __popcll(down) + __popcll(right) + __popcll(left);
        if (pairs == 0) continue;
        int at = atomicAdd(&s_nq, pairs);
        auto push = [&](uint64_t set, int d) {
            for (; set; set &= set - 1) {
                const int c = 64 * i + (int)__builtin_ctzll(set);
                if (at < qcap) queue[at] = make_int2(c, c + d);
                else uf_unite<kGroup>(P, c, c + d);
                ++at;
            }
        };
        push(join, -1);
        push(down, gw);
        push(right, gw + 1);
        push(left, gw - 1);
    }
    __syncthreads();
    const int nq = min(s_nq, qcap);
    for (int q = tid; q < nq; q += kFThreads) uf_unite<kGroup>(P, queue[q].x, queue[q].y);
    // the last thread, which seldom has a join, finishes the sums
    if (tid == kFThreads - 1) {
        double S = 0.0, E = 0.0, HS = 0.0;
        uint32_t M = 0;
        for (int w = 0; w < kSumWaves; ++w) {
            S += s_red[0][w];
            E += s_red[1][w];
            HS += s_red[2][w];
        }
        for (int w = 0; w < kFWaves; ++w) M = max(M, s_max[w]);
        a.entropy[f] = S > 0.0 ? log(S) - E / S : 0.0;
        a.degree[f] = S > 0.0 ? HS / S : 0.0;
        const int Ex = M ? (int)((M >> 23) & 0xffu) - 127 : 0;
        int lg = 0;
        while ((1LL << lg) < (long long)cells) ++lg;
        s_shift = 62 - (max(Ex, -126) + 1) - lg;
    }
    __syncthreads();
    // C (the walks only meet entries that move to roots); a root's entry then
    // becomes -2 - its slot
    auto run_firsts = [&](auto body) {
        for (int i = tid; i < l.words; i += kFThreads) {
            const uint64_t m = hotw[i];
            for (uint64_t b = m & ~((m << 1) & ~row0w[i]); b; b &= b - 1) body(64 * i + (int)__builtin_ctzll(b));
        }
    };
    run_firsts([&](int c) { st_rlx<kGroup>(P + c, uf_root<kGroup>(P, c)); });
    __syncthreads();
    run_firsts([&](int c) {
        if (P[c] == c) P[c] = -2 - atomicAdd(&s_ncomp, 1);
    });
    __syncthreads();
    // D
    const int sh = s_shift, ncomp = s_ncomp, here = min(slots, ncomp);
    const bool over = ncomp > slots;
    if (over) {  // the outputs' zeros first, in full lines: atomics follow
        for (int c = tid; c < cells; c += kFThreads) {
            CC[c] = 0;
            CMu[c] = 0ull;
        }
        wait_memory();
    }
    for (int t = tid; t < here; t += kFThreads) {
        mass[t] = 0ull;
        count[t] = 0;
    }
#pragma unroll
    for (int u = 0; u < kFlight; ++u) v[u] = load(min(wave + kFWaves * u, l.words));
    __syncthreads();
    x = (64 * wave + lane) % gw;
    for (int w0 = wave; w0 < l.words; w0 += kFWaves * kFlight) {
        int32_t root[kFlight], p[kFlight];
        uint64_t m[kFlight], r0[kFlight];
        if constexpr (SPILL) {  // the words' place may hold outputs by now: the bits again, from the forest
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const int c = 64 * (w0 + kFWaves * u) + lane;
                p[u] = P[min(c, cells - 1)];
                root[u] = (c < cells) & (p[u] != -1) ? c : -1;
                m[u] = __ballot(root[u] >= 0);
                r0[u] = __ballot((c < cells) & (x == 0));
                x += xstep;
                x -= x >= gw ? gw : 0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {  // words past the end are not beyond the zero words when clamped
                const int w = min(w0 + kFWaves * u, l.words);
                m[u] = hotw[w];
                r0[u] = row0w[w];
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                m[u] = uniform(m[u]);
                root[u] = __builtin_amdgcn_inverse_ballot_w64(m[u]) ? 64 * (w0 + kFWaves * u) + lane : -1;
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) p[u] = P[max(root[u], 0)];
        }
        // the words' walks in step (p < 0: at the root, or a cold cell);
        // after C two steps reach every root
        for (;;) {
            bool any = false;
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const bool on = (root[u] >= 0) & (p[u] >= 0);
                root[u] = on ? p[u] : root[u];
                any |= on;
            }
            if (!__any(any)) break;
#pragma unroll
            for (int u = 0; u < kFlight; ++u) p[u] = P[max(root[u], 0)];
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int w = w0 + kFWaves * u, c = 64 * w + lane;
            if (c < cells) {
                L[c] = root[u];
                if (!over && root[u] != c) {  // a label cell's outputs come from its component's sums
                    CC[c] = 0;
                    CM[c] = 0.0;
                }
            }
            const float d = v[u];
            v[u] = load(min(w + kFWaves * kFlight, l.words));
            if (m[u] == 0ull) continue;  // wave-uniform
            const unsigned long long q = root[u] >= 0 ? (unsigned long long)llrint(ldexp((double)d, sh)) : 0ull;
            const unsigned long long incl = wave_incl_scan_u64(q);
            // a run's first lane takes its sum: up to its last lane, less what lies before it
            const uint64_t firsts = m[u] & ~((m[u] << 1) & ~uniform(r0[u]));
            const uint64_t lasts = m[u] & (~(m[u] >> 1) | (firsts >> 1) | (1ull << 63));
            const uint64_t after = lasts >> lane;
            const int end = after ? lane + __builtin_ctzll(after) : lane;
            const unsigned long long at_end = __shfl(incl, end, 64);
            if (__builtin_amdgcn_inverse_ballot_w64(firsts)) {
                const int slot = -2 - p[u];
                if (slot < slots) {
                    atomicAdd(count + slot, end - lane + 1);
                    atomicAdd(mass + slot, at_end - (incl - q));
                    if (root[u] == c) label[slot] = c;
                } else {
                    atomicAdd(CC + root[u], end - lane + 1);
                    atomicAdd(CMu + root[u], at_end - (incl - q));
                }
            }
        }
    }
    wait_memory();
    __syncthreads();
    // E
    for (int t = tid; t < here; t += kFThreads) {
        const int32_t c = label[t];
        CC[c] = count[t];
        CM[c] = ldexp((double)mass[t], -sh) * a.cell_area;
    }
    if (over)
        for (int c = tid; c < cells; c += kFThreads)
            if (P[c] <= -2 - slots)
                CM[c] = ldexp((double)__hip_atomic_load(CMu + c, __ATOMIC_RELAXED, kAgent), -sh) * a.cell_area;
    if (tid == 0) a.n_components[f] = ncomp;
}

}  // namespace

size_t heatmap_workspace_bytes(int32_t n_frames, int32_t grid_w, int32_t grid_h) {
    if (n_frames <= 0 || grid_w < 1 || grid_h < 1) return 0;
    const long long tiles = (long long)((grid_w + kHT - 1) / kHT) * ((grid_h + kHT - 1) / kHT);
    const size_t parts = ((size_t)n_frames * tiles * sizeof(TilePart) + 255) & ~(size_t)255;
    return parts + (((size_t)n_frames * sizeof(int32_t) + 255) & ~(size_t)255);
}

// The frame-resident kernel's plan in `lds_limit` bytes of LDS, or no slots for
// grids that do not fit (the tiled kernels).  The path depends on the grid
// alone, since the two add a frame's sums in different orders: a few frames of
// a grid near the limit would be faster tiled (240 x 160 cells, 8 frames: 26
// against 57 us on smooth maps, 66 .. 88 against 84 .. 107 on noisy ones), many
// are not (128: 75 against 60, 238 .. 405 against 88 .. 146).
HeatPlan plan_heatmap(int32_t grid_w, int32_t grid_h, size_t lds_limit) {
    for (const bool spill : {false, true}) {
        const size_t used = frame_lds(grid_w, grid_h, spill).bytes(0) + kFrameStaticLds;
        if (used + (spill ? kMinSpillSlots : kMinSlots) * 16 > lds_limit) continue;
        return {(int)std::min<size_t>((lds_limit - used) / 16, kMaxSlots), spill};
    }
    return {0, false};
}

hipError_t launch_heatmap(HeatArgs a, void *workspace, const HeatPlan &plan, int n_cus, size_t lds_per_cu, hipStream_t stream) {
    if (plan.slots > 0) {
        const size_t lds = frame_lds(a.grid_w, a.grid_h, plan.spill).bytes(plan.slots);
        const dim3 grid((unsigned)a.n_frames);
        // more frames than compute units: 512-thread workgroups, where several
        // share a compute unit, wait less at each barrier and keep it busy
        // (1800 x 128 x 72: 115 us against 159 with 1024 threads, 512 x 64 x
        // 36: 18.5 against 27.7); with at most one frame per compute unit, or
        // half its LDS per frame, a frame takes 1024 (64 x 128 x 72: 23.8
        // against 26.3; 256 x 256 x 144: 64 against 71)
        if (plan.spill)
            hipLaunchKernelGGL((heat_frame_kernel<1024, true>), grid, dim3(1024), lds, stream, a, plan.slots);
        else if (a.n_frames > n_cus && 2 * (lds + kFrameStaticLds) <= lds_per_cu)
            hipLaunchKernelGGL((heat_frame_kernel<512, false>), grid, dim3(512), lds, stream, a, plan.slots);
        else
            hipLaunchKernelGGL((heat_frame_kernel<1024, false>), grid, dim3(1024), lds, stream, a, plan.slots);
        return hipGetLastError();
    }
    a.tiles_x = (a.grid_w + kHT - 1) / kHT;
    a.tiles_y = (a.grid_h + kHT - 1) / kHT;
    const long long tiles = (long long)a.tiles_x * a.tiles_y * a.n_frames;
    TilePart *part = static_cast<TilePart *>(workspace);
    const size_t parts = ((size_t)tiles * sizeof(TilePart) + 255) & ~(size_t)255;
    int32_t *shift = reinterpret_cast<int32_t *>(static_cast<unsigned char *>(workspace) + parts);
    const long long per = 2LL * (a.tiles_x - 1) * a.grid_h + (long long)(a.tiles_y - 1) * a.grid_w;
    const long long merge_blocks = (per * a.n_frames + 255) / 256;
    const long long cells = (long long)a.grid_w * a.grid_h * a.n_frames;
    hipLaunchKernelGGL(heat_tile_kernel, dim3((unsigned)tiles), dim3(kHThreads), 0, stream, a, part);
    hipLaunchKernelGGL(heat_merge_kernel, dim3((unsigned)(merge_blocks + a.n_frames)), dim3(256), 0, stream, a,
                       part, shift, merge_blocks);
    hipLaunchKernelGGL(heat_label_kernel, dim3((unsigned)tiles), dim3(kHThreads), 0, stream, a, shift);
    hipLaunchKernelGGL(heat_mass_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, stream, a, shift);
    return hipGetLastError();
}

}  // namespace flock
