// roi.hip - region-of-interest filter and per-frame region counts, and
// drinker-line proximity, on gfx950.
//
// What is computed (the wall pipeline counts the birds in a region near the
// wall, Section 2.2; Algorithm 1 filters the birds to the region of
// interest): a bird is kept when its point lies in the closed ROI polygon,
// edges and vertices included, under the even-odd rule; kept birds keep
// their input order.  Integer coordinates in 1/16 px, exact 64-bit products.
//
// Three kernels over fixed blocks of 2048 birds, whatever the frames
// (HBM-bound: 8 bytes read per bird, 12 written per kept bird):
//   1. roi_flag_kernel: the inside test per bird, a flag bit per bird and a
//      count per block; the kept birds staged in input order;
//   2. roi_write_kernel: each block's kept birds copied to the block's base +
//      rank, so kept birds keep their input order; the base is the sum of the
//      counts before the block, by the block itself (beyond kRSelfScan blocks
//      by roi_scan_kernel, one workgroup, first);
//   3. roi_counts_kernel, one wave per frame boundary: the output position of
//      the boundary bird (its block's base plus the flags before it in the
//      block) gives out_offsets, and neighbouring boundaries give counts.
// Drinker-line proximity: drink_flag_kernel, then drink_counts_kernel, which
// adds each frame's blocks.

#include <climits>

#include "internal.h"

namespace flock {
namespace {

constexpr int kRThreadsR = 256;
constexpr int kRWaves = kRThreadsR / 64;

// Closed polygon test, even-odd rule.  A point outside the polygon's
// bounding box is outside, and edges whose y range excludes the point are
// skipped.  Otherwise an edge on which the point lies decides
// at once (inside), and each edge whose ends lie on different sides of the
// horizontal line through the point (one strictly above it, so that a vertex
// on the line is counted once) toggles the result when it meets the line to
// the right of the point.  Coordinates and vertices are within 2^24 in
// magnitude, so every difference is below 2^25 and the cross product
// ex qy - ey qx below 2^51: exact in fp64 (two exact products, an exact
// difference), one fp64 multiply per product where a 64-bit integer product
// takes several instructions.
__device__ __forceinline__ bool in_box(const RoiArgs &a, int px, int py) {
    return px >= a.bx0 && px <= a.bx1 && py >= a.by0 && py <= a.by1;
}

// The test for a point inside the bounding box.
__device__ __forceinline__ bool in_polygon_boxed(const RoiArgs &a, const int2 *poly, int px, int py) {
    const int n = a.n_vertices;
    bool in = false;
    for (int i = 0; i < n; ++i) {
        const int2 A = poly[i], B = poly[i + 1 == n ? 0 : i + 1];
        // an edge whose y range excludes py neither holds the point nor
        // crosses its line (both ends lie on one side)
        if (py < min(A.y, B.y) || py > max(A.y, B.y)) continue;
        const double ex = (double)(B.x - A.x), ey = (double)(B.y - A.y);
        const double qx = (double)(px - A.x), qy = (double)(py - A.y);
        const double cr = ex * qy - ey * qx;
        if (cr == 0 && px >= min(A.x, B.x) && px <= max(A.x, B.x) && py >= min(A.y, B.y) && py <= max(A.y, B.y))
            return true;
        const bool a_above = A.y > py, b_above = B.y > py;
        if (a_above != b_above) {
            // crossing at x = A.x + qy ex / ey; right of px iff qx ey < qy ex
            // for ey > 0 (reversed for ey < 0); qy ex - qx ey = cr
            const bool right = ey > 0 ? cr > 0 : cr < 0;
            if (right) in = !in;
        }
    }
    return in;
}

__device__ __forceinline__ void load_polygon(const RoiArgs &a, int2 *poly) {
    if ((int)threadIdx.x < a.n_vertices) poly[threadIdx.x] = make_int2(a.vx[threadIdx.x], a.vy[threadIdx.x]);
    __syncthreads();
}

constexpr int kRBlock = kRoiBlock;             // birds per block
constexpr int kRPer = kRBlock / kRThreadsR;    // birds per thread, consecutive chunks of 256

constexpr int kRWaveBirds = kRBlock / kRWaves;  // a wave's share of a block: kRPer chunks of 64
constexpr int kRQueue = 128;                   // queued candidates per wave (part of a batch + one chunk)

// A wave's queue of candidate birds: the cheap test runs on every bird, the
// exact one on batches of 64 candidates, so that whole waves run it instead of
// every wave running it for the few candidates it holds.  Private to the wave
// (its LDS operations stay in order; the fences keep the compiler's too), so
// no barrier is met between a block's loads and its results.
struct WaveQueue {
    int2 pt[kRQueue];
    uint16_t at[kRQueue];  // the bird's index in the wave's share
};

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Queue the lanes with `cand` set (chunk k of the share), and run `exact(pt,
// at)` on 64 queued birds whenever that many wait; `flush` runs it on the rest.
template <class Exact>
struct QueuedTest {
    WaveQueue &q;
    int head, tail;  // positions, taken modulo kRQueue
    Exact exact;
    __device__ __forceinline__ void push(bool cand, int2 pt, int at, int lane) {
        const uint64_t m = __ballot(cand);
        if (m == 0ull) return;  // wave-uniform
        if (cand) {
            const int i = (tail + __popcll(m & ((1ull << lane) - 1ull))) & (kRQueue - 1);
            q.pt[i] = pt;
            q.at[i] = (uint16_t)at;
        }
        tail += __popcll(m);
        if (tail - head >= 64) run(64, lane);
    }
    __device__ __forceinline__ void run(int n, int lane) {
        wave_fence();
        if (lane < n) {
            const int i = (head + lane) & (kRQueue - 1);
            exact(q.pt[i], (int)q.at[i]);
        }
        head += n;
        wave_fence();
    }
    __device__ __forceinline__ void flush(int lane) {
        if (tail > head) run(tail - head, lane);
    }
};
template <class Exact>
__device__ QueuedTest(WaveQueue &, int, int, Exact) -> QueuedTest<Exact>;

// Flags of one block of birds, a bit per bird (64 birds per word), a wave per
// kRWaveBirds of them.  Few birds lie inside the bounding box of a region along
// a wall; those are queued and tested.  The kept birds then go, in input order,
// to the block's staging area (coordinates and input index), for the write
// kernel to copy to their final places without reading every bird again.
// Bound by HBM: 1800 x 5000 birds, 14% kept, move 72 + 1 + 16 MB in 28.8 us
// (27.8 at best); one queue per block between four barriers, with a byte per
// flag, took some 4 us more.
__global__ __launch_bounds__(kRThreadsR) void roi_flag_kernel(RoiArgs a, uint64_t *flag, int32_t *bcount,
                                                             int2 *stage_xy, int32_t *stage_idx) {
    __shared__ int2 poly[kRoiMaxVertices];
    __shared__ WaveQueue s_q[kRWaves];
    __shared__ uint64_t s_bits[kRWaves][kRPer];
    __shared__ int s_tot[kRWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long i0 = (long long)blockIdx.x * kRBlock + wave * kRWaveBirds;  // the wave's first bird
    const int2 *P = reinterpret_cast<const int2 *>(a.xy);
    // all loads first, so that their latencies overlap
    int2 pts[kRPer];
#pragma unroll
    for (int k = 0; k < kRPer; ++k) {
        const long long i = i0 + 64 * k + lane;
        pts[k] = i < a.total ? P[i] : make_int2(INT_MIN, INT_MIN);  // a padding point is outside every box
    }
    if (lane < kRPer) s_bits[wave][lane] = 0ull;
    load_polygon(a, poly);  // holds a barrier
    auto exact = [&](int2 pt, int at) {
        if (in_polygon_boxed(a, poly, pt.x, pt.y))
            atomicOr(reinterpret_cast<uint32_t *>(s_bits[wave]) + (at >> 5), 1u << (at & 31));
    };
    QueuedTest test{s_q[wave], 0, 0, exact};
#pragma unroll
    for (int k = 0; k < kRPer; ++k) test.push(in_box(a, pts[k].x, pts[k].y), pts[k], 64 * k + lane, lane);
    test.flush(lane);
    wave_fence();
    // flags out, and the kept birds' ranks in the block (input order)
    uint64_t m[kRPer];
    int n = 0;
#pragma unroll
    for (int k = 0; k < kRPer; ++k) {
        m[k] = s_bits[wave][k];
        n += __popcll(m[k]);
    }
    if (lane < kRPer && i0 + 64 * lane < a.total) flag[i0 / 64 + lane] = s_bits[wave][lane];
    if (lane == 0) s_tot[wave] = n;
    __syncthreads();
    long long r = (long long)blockIdx.x * kRBlock;
    int all = 0;
#pragma unroll
    for (int w = 0; w < kRWaves; ++w) {
        r += w < wave ? s_tot[w] : 0;
        all += s_tot[w];
    }
#pragma unroll
    for (int k = 0; k < kRPer; ++k) {
        if ((m[k] >> lane) & 1ull) {
            const long long at = r + __popcll(m[k] & ((1ull << lane) - 1ull));
            stage_xy[at] = pts[k];
            stage_idx[at] = (int32_t)(i0 + 64 * k + lane);
        }
        r += __popcll(m[k]);
    }
    if (tid == 0) bcount[blockIdx.x] = all;
}

// bbase[b] = bcount[0] + ... + bcount[b - 1]; bbase[nb] = all kept birds.
__global__ __launch_bounds__(1024) void roi_scan_kernel(const int32_t *bcount, int32_t *bbase, int nb) {
    __shared__ int s_wave[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (nb + 1023) / 1024;
    const int b0 = min(tid * per, nb), b1 = min(b0 + per, nb);
    int sum = 0;
    for (int b = b0; b < b1; ++b) sum += bcount[b];
    int inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    int run = inc - sum;
    for (int w = 0; w < wave; ++w) run += s_wave[w];
    for (int b = b0; b < b1; ++b) {
        bbase[b] = run;
        run += bcount[b];
    }
    if (tid == 1023) bbase[nb] = run;  // the last thread's chunk ends at nb
}

// Each block's kept birds, staged in input order by the flag kernel, go to
// base + rank.  Up to kRSelfScan blocks a block adds up the counts before it
// itself (at most 32 reads a thread, from L2) and leaves its base for the
// counts kernel; beyond that the scan kernel has made the bases.  The whole call
// with own sums and with the scan kernel: 64 blocks 12.3 and 14.3 us, 4096 38.2
// and 41.0, 8192 65.5 and 72.2, 16384 135.6 and 141.0, 24576 226.6 and 212.4 (the
// own sums' work grows with the square of the blocks).
constexpr int kRSelfScan = 8192;

__global__ __launch_bounds__(kRThreadsR) void roi_write_kernel(RoiArgs a, const int32_t *bcount, int32_t *bbase, int nb,
                                                              const int2 *stage_xy, const int32_t *stage_idx) {
    __shared__ int s_sum[kRWaves];
    const int tid = threadIdx.x, b = blockIdx.x;
    int32_t base;
    if (nb <= kRSelfScan) {
        int sum = 0;
        for (int i0 = tid; i0 < b; i0 += kRThreadsR * 8) {
            int c[8];  // in flight together
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = i0 + u * kRThreadsR < b ? bcount[i0 + u * kRThreadsR] : 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += c[u];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if ((tid & 63) == 0) s_sum[tid >> 6] = sum;
        __syncthreads();
        base = 0;
#pragma unroll
        for (int w = 0; w < kRWaves; ++w) base += s_sum[w];
        if (tid == 0) {
            bbase[b] = base;
            if (b == nb - 1) bbase[nb] = base + bcount[b];
        }
    } else {
        base = bbase[b];
    }
    const int n = bcount[b];
    const long long sbase = (long long)b * kRBlock;
    int2 *O = reinterpret_cast<int2 *>(a.out_xy);
    for (int t = tid; t < n; t += kRThreadsR) {
        O[base + t] = stage_xy[sbase + t];
        if (a.out_index) a.out_index[base + t] = stage_idx[sbase + t];
    }
}

// Flagged birds before input bird i (0 <= i <= total) in i's block, from the
// ROI's bits or the drinkers' bytes (wave-uniform calls).
__device__ __forceinline__ int32_t wave_total(int c) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    return c;
}

__device__ __forceinline__ int32_t bits_before(const uint64_t *flag, int32_t i) {
    const int lane = threadIdx.x & 63, n = i % kRBlock - 64 * lane;  // bits of this lane's word
    const uint64_t w = n > 0 ? flag[i / kRBlock * (kRBlock / 64) + lane] : 0ull;  // n > 0: lane < 32
    return wave_total(__popcll(n >= 64 ? w : w & ((1ull << (n & 63)) - 1ull)));
}

__device__ __forceinline__ int32_t bytes_before(const uint8_t *flag, int32_t total, int32_t i) {
    // 16 flags per lane and load (a block is 2048 = 2 x 64 x 16 flags; the
    // flag array is 16-byte aligned), bytes at or past i masked; the last
    // partial word of the array is read byte by byte, never past total
    const int lane = threadIdx.x & 63;
    const int32_t s0 = i / kRBlock * kRBlock;
    int c = 0;
#pragma unroll
    for (int j = 0; j < kRBlock / (64 * 16); ++j) {
        const int32_t base = s0 + 16 * (lane + 64 * j);
        if (base >= i) continue;
        if (base + 16 > total) {
            for (int32_t k = base; k < i; ++k) c += flag[k];
            continue;
        }
        const uint4 w = *reinterpret_cast<const uint4 *>(flag + base);
        const int valid = min(16, i - base);
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int nb = min(max(valid - 4 * q, 0), 4);  // valid bytes in this word
            const uint32_t keep = nb >= 4 ? 0xffffffffu : ((1u << (8 * nb)) - 1u);
            c += (int)(((ws[q] & keep) * 0x01010101u) >> 24);  // bytes are 0 or 1
        }
    }
    return wave_total(c);
}

// Frame boundary g clamped into [0, total] (offsets are only validated with
// FLOCK_VALIDATE; this keeps every read in bounds).
__device__ __forceinline__ int32_t frame_bound(const int32_t *offsets, int32_t n_frames, int32_t total, int g) {
    return g == n_frames ? total : min(max(offsets[g], 0), total);
}

// One wave per frame boundary f = 0 .. n_frames: the CSR offsets of the ROI's
// output and its per-frame counts (bbase has nb + 1 entries, and i = total
// gives block nb at most).
__global__ __launch_bounds__(256) void roi_counts_kernel(RoiArgs a, const uint64_t *flag, const int32_t *bbase) {
    const int f = (int)(((long long)blockIdx.x * 256 + threadIdx.x) >> 6);
    if (f > a.n_frames) return;  // wave-uniform
    auto before = [&](int g) {
        const int32_t i = frame_bound(a.offsets, a.n_frames, a.total, g);
        return bbase[i / kRBlock] + bits_before(flag, i);
    };
    const int32_t v = before(f);
    if ((threadIdx.x & 63) == 0) a.out_offsets[f] = v;
    if (f < a.n_frames) {
        const int32_t v1 = before(f + 1);
        if ((threadIdx.x & 63) == 0) a.counts[f] = max(v1 - v, 0);
    }
}

// One wave per frame: the drinkers' count from the blocks the frame covers
// (whole blocks by their counts, the first and last by their flags), so that no
// scan over all blocks is needed.
__global__ __launch_bounds__(256) void drink_counts_kernel(DrinkArgs a, const int32_t *bcount) {
    const int f = (int)(((long long)blockIdx.x * 256 + threadIdx.x) >> 6);
    if (f >= a.n_frames) return;  // wave-uniform
    const int lane = threadIdx.x & 63;
    const int32_t i0 = frame_bound(a.offsets, a.n_frames, a.total, f);
    const int32_t i1 = frame_bound(a.offsets, a.n_frames, a.total, f + 1);
    if (i1 <= i0) {
        if (lane == 0) a.counts[f] = 0;
        return;
    }
    const int32_t b0 = i0 / kRBlock, b1 = i1 / kRBlock;  // blocks b0 .. b1 - 1 end inside the frame
    int c = 0;
    for (int32_t b = b0 + lane; b < b1; b += 64 * 4) {
        int v[4];  // in flight together
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = b + 64 * u < b1 ? bcount[b + 64 * u] : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) c += v[u];
    }
    const int32_t n = wave_total(c) - bytes_before(a.drinking, a.total, i0) + bytes_before(a.drinking, a.total, i1);
    if (lane == 0) a.counts[f] = n;
}

// ---------------------------------------------------------------------------
// Drinker-line proximity
// ---------------------------------------------------------------------------

// Is (px, py) strictly closer than t to the closed segment s = (ax, ay, bx,
// by)?  The nearest point of the segment is a when the projection of p
// falls before a (or the segment is a point), b when it falls past b, and
// otherwise the foot of the perpendicular, at squared distance
// cross^2 / len2.  Coordinates within 2^24: squared end distances, len2 and
// the projection fit int64, and cross^2 < t^2 len2 is compared as a 128-bit
// product (high and low halves).
__device__ __forceinline__ bool near_segment(int4 s, int px, int py, long long t2) {
    const long long ux = (long long)s.z - s.x, uy = (long long)s.w - s.y;
    const long long wx = (long long)px - s.x, wy = (long long)py - s.y;
    const long long len2 = ux * ux + uy * uy, dot = ux * wx + uy * wy;
    if (len2 == 0 || dot <= 0) return wx * wx + wy * wy < t2;
    if (dot >= len2) {
        const long long vx = (long long)px - s.z, vy = (long long)py - s.w;
        return vx * vx + vy * vy < t2;
    }
    const long long cr = ux * wy - uy * wx;
    const unsigned long long c = (unsigned long long)(cr < 0 ? -cr : cr);
    const unsigned long long ch = __umul64hi(c, c), cl = c * c;
    const unsigned long long lh = __umul64hi((unsigned long long)t2, (unsigned long long)len2),
                             ll = (unsigned long long)t2 * (unsigned long long)len2;
    return ch < lh || (ch == lh && cl < ll);
}

// Flags of one block of birds, a wave per kRWaveBirds of them.  A bird within T
// of a segment lies in the segment's bounding box widened by T on every side,
// so birds outside all widened boxes (most of them, for lines across the frame)
// are not drinking; the others are queued and tested exactly.  The wave's
// results wait in LDS as one byte per bird and leave in full lines.
// Bound by HBM: 1800 x 5000 birds move 72 + 45 MB in 27.9 us (some 3 us more
// with one queue per block and stores by the birds' own lanes).
__global__ __launch_bounds__(kRThreadsR) void drink_flag_kernel(DrinkArgs a, int32_t *bcount) {
    __shared__ int4 seg[kDrinkMaxLines];
    __shared__ int4 box[kDrinkMaxLines];  // x0, y0, x1, y1 widened by T
    __shared__ WaveQueue s_q[kRWaves];
    __shared__ uint64_t s_hit[kRWaves][kRWaveBirds / 8];  // a byte per bird: its segment, 0xff for none
    __shared__ int s_in;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long i0 = (long long)blockIdx.x * kRBlock + wave * kRWaveBirds;  // the wave's first bird
    const int2 *P = reinterpret_cast<const int2 *>(a.xy);
    int2 pts[kRPer];
#pragma unroll
    for (int k = 0; k < kRPer; ++k) {
        const long long i = i0 + 64 * k + lane;
        pts[k] = i < a.total ? P[i] : make_int2(0, 0);
    }
    if (tid == 0) s_in = 0;
    if (tid < a.n_lines) {
        seg[tid] = make_int4(a.ax[tid], a.ay[tid], a.bx[tid], a.by[tid]);
        const int t = a.threshold;  // |coordinates|, T <= 2^24: no overflow
        box[tid] = make_int4(min(a.ax[tid], a.bx[tid]) - t, min(a.ay[tid], a.by[tid]) - t,
                             max(a.ax[tid], a.bx[tid]) + t, max(a.ay[tid], a.by[tid]) + t);
    }
    static_assert(kRWaveBirds == 64 * 8, "eight result bytes per lane");
    s_hit[wave][lane] = ~0ull;
    __syncthreads();
    const long long t2 = (long long)a.threshold * a.threshold;
    bool cands[kRPer];
#pragma unroll
    for (int k = 0; k < kRPer; ++k) cands[k] = false;
    for (int l = 0; l < a.n_lines; ++l) {  // each box read once, for all of the lane's birds
        const int4 b = box[l];
#pragma unroll
        for (int k = 0; k < kRPer; ++k)
            cands[k] |= (pts[k].x > b.x) & (pts[k].x < b.z) & (pts[k].y > b.y) & (pts[k].y < b.w);
    }
    uint8_t *hit = reinterpret_cast<uint8_t *>(s_hit[wave]);
    auto exact = [&](int2 pt, int at) {
        for (int l = 0; l < a.n_lines; ++l)
            if (near_segment(seg[l], pt.x, pt.y, t2)) {
                hit[at] = (uint8_t)l;
                break;
            }
    };
    QueuedTest test{s_q[wave], 0, 0, exact};
#pragma unroll
    for (int k = 0; k < kRPer; ++k)
        test.push(cands[k] & (i0 + 64 * k + lane < a.total), pts[k], 64 * k + lane, lane);
    test.flush(lane);
    wave_fence();
    // eight birds' flags per lane: segments are below 64, so bit 7 tells none
    const uint64_t flags = (~s_hit[wave][lane] >> 7) & 0x0101010101010101ull;
    const long long at = i0 + 8 * lane;
    if (at + 8 <= a.total) {
        *reinterpret_cast<uint64_t *>(a.drinking + at) = flags;
    } else {
        for (int k = 0; k < 8 && at + k < a.total; ++k) a.drinking[at + k] = (uint8_t)(flags >> (8 * k));
    }
    if (a.line) {
#pragma unroll
        for (int k = 0; k < kRPer; ++k) {
            const long long i = i0 + 64 * k + lane;
            if (i < a.total) a.line[i] = (int32_t)(int8_t)hit[64 * k + lane];
        }
    }
    const int cnt = wave_total(__popcll(flags));
    if (lane == 0 && cnt) atomicAdd(&s_in, cnt);
    __syncthreads();
    if (tid == 0) bcount[blockIdx.x] = s_in;
}

}  // namespace

// Workspace: a flag bit per bird; a count and a base per block; per block a
// staging area of kRBlock coordinates and kRBlock input indices.
struct RoiLayout {
    size_t flags, counts, xy, idx, bytes;  // offsets, and the size
};

RoiLayout roi_layout(int32_t total) {
    auto up = [](size_t n) { return (n + 255) & ~(size_t)255; };
    const size_t nb = total > 0 ? ((size_t)total + kRBlock - 1) / kRBlock : 0;
    RoiLayout l;
    l.flags = 0;
    l.counts = up(nb * (kRBlock / 64) * sizeof(uint64_t));
    l.xy = l.counts + up((2 * nb + 1) * sizeof(int32_t));
    l.idx = l.xy + nb * kRBlock * sizeof(int2);
    l.bytes = l.idx + nb * kRBlock * sizeof(int32_t);
    return l;
}

size_t roi_workspace_bytes(int32_t total) { return roi_layout(total).bytes; }

hipError_t launch_roi(const RoiArgs &a, void *workspace, hipStream_t stream) {
    const int nb = (int)(((long long)a.total + kRBlock - 1) / kRBlock);
    const RoiLayout l = roi_layout(a.total);
    char *base = static_cast<char *>(workspace);
    uint64_t *flag = reinterpret_cast<uint64_t *>(base + l.flags);
    int32_t *bcount = reinterpret_cast<int32_t *>(base + l.counts), *bbase = bcount + nb;
    int2 *stage_xy = reinterpret_cast<int2 *>(base + l.xy);
    int32_t *stage_idx = reinterpret_cast<int32_t *>(base + l.idx);
    if (nb > 0)
        hipLaunchKernelGGL(roi_flag_kernel, dim3((unsigned)nb), dim3(kRThreadsR), 0, stream, a, flag, bcount, stage_xy,
                           stage_idx);
    if (nb == 0 || nb > kRSelfScan)
        hipLaunchKernelGGL(roi_scan_kernel, dim3(1), dim3(1024), 0, stream, bcount, bbase, nb);
    if (nb > 0)
        hipLaunchKernelGGL(roi_write_kernel, dim3((unsigned)nb), dim3(kRThreadsR), 0, stream, a, bcount, bbase, nb,
                           stage_xy, stage_idx);
    const long long waves = (long long)a.n_frames + 1;
    hipLaunchKernelGGL(roi_counts_kernel, dim3((unsigned)((waves * 64 + 255) / 256)), dim3(256), 0, stream, a, flag,
                       bbase);
    return hipGetLastError();
}

size_t drink_workspace_bytes(int32_t total) {
    const size_t nb = total > 0 ? ((size_t)total + kRBlock - 1) / kRBlock : 1;
    return ((nb * sizeof(int32_t) + 255) & ~(size_t)255);
}

hipError_t launch_drinkers(const DrinkArgs &a, void *workspace, hipStream_t stream) {
    const int nb = (int)(((long long)a.total + kRBlock - 1) / kRBlock);
    int32_t *bcount = static_cast<int32_t *>(workspace);
    if (nb > 0) hipLaunchKernelGGL(drink_flag_kernel, dim3((unsigned)nb), dim3(kRThreadsR), 0, stream, a, bcount);
    hipLaunchKernelGGL(drink_counts_kernel, dim3((unsigned)(((long long)a.n_frames * 64 + 255) / 256)), dim3(256), 0,
                       stream, a, bcount);
    return hipGetLastError();
}

}  // namespace flock
