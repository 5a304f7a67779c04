/*
 * collide.hip -- collision detection between agents on a wrapped uniform
 * grid (the detection module of Sec. II-A: colliding agents are marked dead
 * and excluded from the simulation).
 *
 * Two alive agents collide when |p_i - p_j|^2 < (r_i + r_j)^2, evaluated in
 * FP32 as d2 = (dx*dx + dy*dy) + dz*dz with dx = x_i - x_j and
 * rr = (r_i + r_j)^2, without contraction, so the decision is the same bit
 * for bit wherever it is taken.  All decisions of one call use the alive set
 * on entry (simultaneous events).
 *
 * Grid: with h = 2.02 r_max (r_max the largest radius), colliding agents are
 * less than h apart along every axis.  A cell is h x 2h x 2h: an agent's
 * partners sit in the 3 cells around it along x, and along y and z in its
 * own cell or in the one on the side of the half that it is in, 12 cells in
 * 4 (y, z) rows.  (Cells of h x h x h have 27 neighbours in 9 rows: the
 * query took 48 us against 31 at 1M agents; where the grid is wrapped, 12
 * buckets also hold fewer candidates than 27.)  Cells map to buckets by their
 * indices wrapped to 2^bx x 2^by x 2^bz, where the bits split the budget
 * 2^k >= 2N by the extent of the alive agents' bounding box (so a flat
 * swarm does not leave the buckets of an unused depth empty); buckets are
 * linear with x fastest, and each x row holds two extra ghost cells (a
 * copy of the last before the first and of the first after the last), so the
 * three x neighbours of any cell are consecutive buckets and an agent's 12
 * cells are 4 contiguous bucket ranges.  Where agents are dense enough to
 * leave bits of the budget over, a cell edge along x is 2 or 4 columns: an
 * agent's range is then 2.5 or 2.25 edges long instead of 3, and its
 * candidates those of 40 or 36 h^3 instead of 48 (27 cells of h: 27 h^3 in 9
 * ranges).  A lattice of 1,048,576 agents 1.05 contact distances apart takes
 * 114 us, close packed at 1.02 129 (one column per edge 128 and 160, cells of
 * h^3 112 and 130); sparse swarms have one column either way.
 * Passes: bounding box (block partials, reduced again by every block of
 * the next kernel, which plans the wrap and stores it); a two-level sort of
 * the items (position and radius or id) into bucket order (per-tile counts
 * of bucket partitions, their scan, the tiles' items written partition by
 * partition, then each window of a partition sorted in LDS, which also
 * writes the bucket starts); query, one thread per sorted slot, over the
 * candidates of its 4 ranges in batches of loads in flight; one block adding
 * up the dead.  At 1M agents (5 per cubic metre) they take 7, 8.5, 6, 12,
 * 16.5, 31 and 3 us, at 20,000 their latencies.  Cells that share a bucket
 * are far apart and fail the distance test; the decision is always the
 * distance test.  Small swarms test every pair instead (k_coll_pairs).  The 1 % margin in h keeps
 * the neighbour property exact for |coordinates| < 2^16 h (about 22 km for
 * 0.17 m radii).
 */
#include <algorithm>
#include <mutex>
#include <vector>

#include "kernels.h"
#include "scan.h"

namespace potato {

/* Candidates whose loads are issued together in the query. */
#ifndef POTATO_QUERY_BATCH
#define POTATO_QUERY_BATCH 8
#endif

namespace {

/* Fewest bits of the ghost-padded x axis: 2^5 columns + 2 ghosts keeps the
 * padding within 1/16 of the bucket budget. */
constexpr int kMinXBits = 5;
constexpr int kMaxSplitBits = 2;

/* Cell index along one axis.  The coordinate in cells is clamped to
 * [-2^24, 2^24] before the conversion, so infinite, NaN (max/min return the
 * other operand) and huge coordinates give a defined index and the
 * neighbour indices +-1 cannot overflow.  Agents beyond the clamp share the
 * edge cells, which only adds candidates; the decision is the distance
 * test, and a NaN or infinite position never passes it. */
__device__ __forceinline__ int32_t cell_index(float x, float inv_h) {
    const float c = fminf(fmaxf(x * inv_h, -16777216.0f), 16777216.0f);
    return (int32_t)floorf(c);
}

/* The cells are two edges wide in y and z: an agent's neighbours along such
 * an axis are its own cell and the one on the side of the half it is in. */
__device__ __forceinline__ int32_t wide_cell(int32_t c) { return c >> 1; }
__device__ __forceinline__ uint32_t near_side(int32_t c) { return (uint32_t)((c & 1) * 2 - 1); }

/* Wrap of the grid: 2^bx x 2^by x 2^bz cells, side = 2^f columns per cell
 * edge, x rows of 2^bx + 2 side buckets. */
struct Wrap {
    int bx, by, bz, f;
    uint32_t mx, my, mz;     /* 2^b - 1 */
    uint32_t side;
    uint32_t row;
    float per_edge;          /* side */
};

/* e >= 1 */
__device__ __forceinline__ int ceil_log2(int64_t e) { return e > 1 ? 64 - __clzll(e - 1) : 0; }

__device__ __forceinline__ Wrap wrap_of(const int32_t* b) {
    Wrap w;
    w.bx = b[0]; w.by = b[1]; w.bz = b[2]; w.f = b[3];
    w.mx = (1u << b[0]) - 1u; w.my = (1u << b[1]) - 1u; w.mz = (1u << b[2]) - 1u;
    w.side = 1u << b[3];
    w.row = (1u << b[0]) + 2u * w.side;
    w.per_edge = (float)w.side;
    return w;
}

/* Bits per axis for bucket budget 2^k from the bounding box (min x, y, z,
 * max x, y, z, in cells): start from the bits that cover each extent, then
 * take bits away, each time from the axis whose extent is the smallest
 * multiple of its halved wrap (it gains the fewest wraps), x not below
 * kMinXBits.  Bits that are left over, as in swarms with several agents per
 * cell, make up to 4 columns of a cell edge: the candidates of an agent then
 * come from 2.5 or 2.25 edges along x instead of 3.  Every block of k_coll_hist computes the same wrap and one
 * stores its bits for the later kernels of the pass. */
__device__ __forceinline__ Wrap plan_wrap(const int32_t* box, int k) {
    int64_t e[3];
    for (int a = 0; a < 3; ++a) {
        const int64_t lo = box[a], hi = box[3 + a];
        e[a] = hi >= lo ? hi - lo + 1 : 1;       /* no alive agent: any wrap */
    }
    int b[4] = {ceil_log2(e[0]), ceil_log2(e[1]), ceil_log2(e[2]), 0};
    if (b[0] < kMinXBits) b[0] = kMinXBits;
    while (b[0] + b[1] + b[2] > k) {
        int best = -1;
        for (int a = 2; a >= 0; --a) {
            if (b[a] == 0 || (a == 0 && b[a] == kMinXBits)) continue;
            /* e[a] / 2^(b[a]-1) < e[best] / 2^(b[best]-1), cross-multiplied */
            if (best < 0 || e[a] * (int64_t(1) << b[best]) < e[best] * (int64_t(1) << b[a])) best = a;
        }
        --b[best];
    }
    b[3] = min(k - (b[0] + b[1] + b[2]), kMaxSplitBits);
    b[0] += b[3];
    return wrap_of(b);
}

/* Bucket of wrapped cell (column col = wrapped x + side, wrapped y, wrapped z). */
__device__ __forceinline__ uint32_t bucket_of(const Wrap& w, uint32_t col, uint32_t wy, uint32_t wz) {
    return col + w.row * (wy | (wz << w.by));
}

/* Bounding box of the alive agents' cells, in two steps: each block of a
 * grid of at most kBoxBlocks reduces its grid-stride share to six partial
 * bounds, then every block of the next kernel reduces the partials itself
 * (one atomic per block on six shared words serialised the first form of
 * this pass: 96 us at 1M agents). */
constexpr int kBoxBlocks = 512;
constexpr int64_t kBoxWords = 6 * 1024;      /* of the workspace, for 6 * kBoxBlocks */
static_assert(6 * kBoxBlocks <= kBoxWords, "partial bounds fit");
constexpr int kBoxThreads = 512;
constexpr int kBoxUnroll = 4;
constexpr int kMaxWaves = 16;

__device__ __forceinline__ int32_t bound_op(int a, int32_t x, int32_t y) { return a < 3 ? min(x, y) : max(x, y); }

/* Block reduction of v[6] (min of 0-2, max of 3-5); the result is valid in
 * thread 0..5 as red[a][0]. */
__device__ __forceinline__ void block_bounds(int32_t v[6], int32_t (*red)[kMaxWaves]) {
    for (int a = 0; a < 6; ++a) {
        int32_t x = v[a];
        for (int off = 32; off > 0; off >>= 1) x = bound_op(a, x, __shfl_xor(x, off));
        v[a] = x;
    }
    if ((threadIdx.x & 63) == 0)
        for (int a = 0; a < 6; ++a) red[a][threadIdx.x / 64] = v[a];
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        int32_t x = red[a][0];
        for (int w = 1; w < (int)(blockDim.x / 64); ++w) x = bound_op(a, x, red[a][w]);
        red[a][0] = x;
    }
}

__global__ void __launch_bounds__(kBoxThreads) k_coll_bounds(const float* rows, int64_t ld, int64_t n,
                                                             const uint8_t* alive, float inv_h, int32_t* partial) {
    __shared__ int32_t red[6][kMaxWaves];
    int32_t v[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
    const int64_t stride = (int64_t)gridDim.x * kBoxThreads;
    for (int64_t i0 = (int64_t)blockIdx.x * kBoxThreads + threadIdx.x; i0 < n; i0 += kBoxUnroll * stride) {
        /* all loads of a round in flight together */
        float x[kBoxUnroll][3];
        bool on[kBoxUnroll];
#pragma unroll
        for (int u = 0; u < kBoxUnroll; ++u) {
            const int64_t i = i0 + u * stride;
            on[u] = i < n;
            if (on[u]) {
                on[u] = alive[i] != 0;
                for (int a = 0; a < 3; ++a) x[u][a] = rows[a * ld + i];
            }
        }
#pragma unroll
        for (int u = 0; u < kBoxUnroll; ++u) {
            if (!on[u]) continue;
            for (int a = 0; a < 3; ++a) {
                const int32_t f = cell_index(x[u][a], inv_h), c = a ? wide_cell(f) : f;
                v[a] = min(v[a], c);
                v[3 + a] = max(v[3 + a], c);
            }
        }
    }
    block_bounds(v, red);
    if (threadIdx.x < 6) partial[threadIdx.x * gridDim.x + blockIdx.x] = red[threadIdx.x][0];
}

/* The bounding box from the partials of k_coll_bounds, in every thread of
 * the block (box_lds: six words of LDS). */
__device__ __forceinline__ void reduce_box(const int32_t* partial, int n_partial, int32_t (*red)[kMaxWaves],
                                           int32_t* box_lds) {
    int32_t v[6] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MIN};
    for (int b = threadIdx.x; b < n_partial; b += blockDim.x)
        for (int a = 0; a < 6; ++a) v[a] = bound_op(a, v[a], partial[a * n_partial + b]);
    block_bounds(v, red);
    if (threadIdx.x < 6) box_lds[threadIdx.x] = red[threadIdx.x][0];
    __syncthreads();
}

/* Blocks are dispatched to the 8 XCDs in turn (block b to XCD b mod 8), and
 * each XCD has its own L2.  Mapping block b to tile xcd * (blocks per XCD) +
 * b / 8 gives each XCD one contiguous eighth of the tiles, so neighbouring
 * tiles, which read the same data, share an L2. */
constexpr uint32_t kXcds = 8;

__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n_blocks) {
    const uint32_t q = n_blocks / kXcds, r = n_blocks % kXcds;
    const uint32_t x = b % kXcds, pos = b / kXcds;
    return x * q + (x < r ? x : r) + pos;
}

/* Wrapped cell of a position. */
__device__ __forceinline__ void wrapped_cell(const Wrap& w, float x, float y, float z, float inv_h, uint32_t& wx,
                                             uint32_t& wy, uint32_t& wz) {
    wx = (uint32_t)cell_index(x, inv_h * w.per_edge) & w.mx;
    wy = (uint32_t)wide_cell(cell_index(y, inv_h)) & w.my;
    wz = (uint32_t)wide_cell(cell_index(z, inv_h)) & w.mz;
}

/* An agent in the first cell edge's columns also sits in the ghost columns
 * after the last, one in the last edge's in those before the first: the
 * bucket offset of its ghost, or 0. */
__device__ __forceinline__ int32_t ghost_offset(const Wrap& w, uint32_t wx) {
    return wx < w.side ? (int32_t)(w.mx + 1) : (wx > w.mx - w.side ? -(int32_t)(w.mx + 1) : 0);
}

/* Bucket of an item: the agent's own bucket, or for a ghost copy (id with
 * the top bit set) the ghost bucket of its edge column. */
__device__ __forceinline__ uint32_t item_bucket(const Wrap& w, const float4& q, int32_t id, float inv_h) {
    uint32_t wx, wy, wz;
    wrapped_cell(w, q.x, q.y, q.z, inv_h, wx, wy, wz);
    const uint32_t b = bucket_of(w, wx + w.side, wy, wz);
    return id < 0 ? (uint32_t)((int32_t)b + ghost_offset(w, wx)) : b;
}

/* An item is (x, y, z, radius) with its id in an array beside it; where all
 * agents have one radius the id takes the radius's place: one scattered
 * store and one gathered load less per item (1M agents: the tiles' pass 19
 * -> 12 us and the windows' 23 -> 16.5, with the wrap kept and the scan by
 * shuffles). */
template <bool ONE_RADIUS>
__device__ __forceinline__ int32_t item_id(const float4& q, const int32_t* ids, int32_t j) {
    return ONE_RADIUS ? __float_as_int(q.w) : ids[j];
}

/* Sort of the items into bucket order.  An item is an alive agent, or the
 * ghost copy of an agent in an edge column.  Two levels:
 *  - the buckets are split into partitions of 2^s consecutive buckets (s the
 *    smallest >= kWindowBits that gives at most kMaxParts partitions) and
 *    the agents into tiles (tiles of one XCD contiguous, as in xcd_tile).
 *    k_coll_hist counts each tile's items per partition in LDS; one
 *    exclusive scan over the counts, laid out partition-major, gives every
 *    (partition, tile) pair its output offset; k_coll_part writes each
 *    tile's items through LDS cursors.  The tiles of one XCD thus write one
 *    contiguous run per partition, which its L2 merges into whole lines.
 *  - k_coll_sort, one block per window of kWindow buckets, counts in LDS the
 *    items of its partition that fall in its window (and those of the
 *    partition's earlier windows), scans the counts into the window's
 *    bucket starts, and places its items within the partition's range.
 * The order of the items of one bucket follows the order of the LDS
 * atomics; no decision of the query depends on it. */
constexpr int kWindowBits = 12;
constexpr int kWindow = 1 << kWindowBits;
constexpr int64_t kMaxParts = 16384;        /* LDS cursors of the tile passes: 64 KB */
constexpr int kTileBlock = 512;
constexpr int kTileUnroll = 4;
constexpr int64_t kTileAgents = kTileBlock * kTileUnroll;
constexpr int64_t kMaxTiles = 2048;

/* Offset of (partition, tile) cell c after the scan in chunks: the chunk's
 * own exclusive scan plus the scanned chunk totals; cell `cells` holds the
 * slot count. */
__device__ __forceinline__ int32_t cell_offset(const int32_t* off, const int32_t* totals, int64_t c, int64_t cells) {
    return c < cells ? off[c] + totals[c / kScanBlock] : off[cells];
}

/* Also reduces the bounding box and plans the wrap. */
__global__ void __launch_bounds__(kTileBlock) k_coll_hist(const float* rows, int64_t ld, int64_t n,
                                                          const uint8_t* alive, float inv_h, const int32_t* partial,
                                                          int n_partial, int32_t* wrap, int k,
                                                          int s, int32_t parts, int64_t tile, int32_t* hist) {
    extern __shared__ int32_t cnt[];
    __shared__ int32_t red[6][kMaxWaves];
    __shared__ int32_t box_lds[6];
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t a0 = (int64_t)t * tile, a1 = a0 + tile < n ? a0 + tile : n;
    float px[kTileUnroll], py[kTileUnroll], pz[kTileUnroll];
    bool on[kTileUnroll];
    auto load = [&](int64_t base) {
#pragma unroll
        for (int r = 0; r < kTileUnroll; ++r) {
            const int64_t i = base + threadIdx.x + r * kTileBlock;
            on[r] = i < a1;
            if (on[r]) {
                on[r] = alive[i] != 0;
                px[r] = rows[i];
                py[r] = rows[ld + i];
                pz[r] = rows[2 * ld + i];
            }
        }
    };
    /* the first round's loads do not depend on the box: in flight during
     * its reduction */
    load(a0);
    reduce_box(partial, n_partial, red, box_lds);
    const Wrap w = plan_wrap(box_lds, k);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        wrap[0] = w.bx;
        wrap[1] = w.by;
        wrap[2] = w.bz;
        wrap[3] = w.f;
    }
    for (int32_t p = threadIdx.x; p < parts; p += kTileBlock) cnt[p] = 0;
    __syncthreads();
    for (int64_t base = a0; base < a1; base += kTileAgents) {
        if (base != a0) load(base);
#pragma unroll
        for (int r = 0; r < kTileUnroll; ++r) {
            if (!on[r]) continue;
            uint32_t wx, wy, wz;
            wrapped_cell(w, px[r], py[r], pz[r], inv_h, wx, wy, wz);
            const uint32_t b = bucket_of(w, wx + w.side, wy, wz);
            atomicAdd(&cnt[b >> s], 1);
            const int32_t g = ghost_offset(w, wx);
            if (g != 0) atomicAdd(&cnt[(uint32_t)((int32_t)b + g) >> s], 1);
        }
    }
    __syncthreads();
    for (int32_t p = threadIdx.x; p < parts; p += kTileBlock) hist[(int64_t)p * gridDim.x + t] = cnt[p];
}

template <bool ONE_RADIUS>
__global__ void __launch_bounds__(kTileBlock) k_coll_part(const float* rows, int64_t ld, int64_t n,
                                                          const uint8_t* alive, const uint8_t* type, int n_types,
                                                          const float* radius, float inv_h, const int32_t* wrap,
                                                          int s, int32_t parts, int64_t tile,
                                                          const int32_t* off, const int32_t* totals, float4* tpos,
                                                          int32_t* tid) {
    extern __shared__ int32_t cur[];
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t a0 = (int64_t)t * tile, a1 = a0 + tile < n ? a0 + tile : n;
    /* all loads of a round first: the stores of the round may alias them as
     * far as the compiler knows; the first round's are in flight while the
     * cursors are read */
    float4 q[kTileUnroll];
    bool on[kTileUnroll];
    auto load = [&](int64_t base) {
#pragma unroll
        for (int r = 0; r < kTileUnroll; ++r) {
            const int64_t i = base + threadIdx.x + r * kTileBlock;
            on[r] = i < a1;
            if (on[r]) {
                on[r] = alive[i] != 0;
                q[r] = make_float4(rows[i], rows[ld + i], rows[2 * ld + i],
                                   ONE_RADIUS ? __int_as_float((int32_t)i)
                                              : radius[type_entry(type, (uint32_t)i, n_types)]);
            }
        }
    };
    load(a0);
    const Wrap w = wrap_of(wrap);
    for (int32_t p = threadIdx.x; p < parts; p += kTileBlock) {
        const int64_t c = (int64_t)p * gridDim.x + t;
        cur[p] = off[c] + totals[c / kScanBlock];
    }
    __syncthreads();
    for (int64_t base = a0; base < a1; base += kTileAgents) {
        if (base != a0) load(base);
#pragma unroll
        for (int r = 0; r < kTileUnroll; ++r) {
            if (!on[r]) continue;
            const int32_t i = (int32_t)(base + threadIdx.x + r * kTileBlock);
            uint32_t wx, wy, wz;
            wrapped_cell(w, q[r].x, q[r].y, q[r].z, inv_h, wx, wy, wz);
            const uint32_t b = bucket_of(w, wx + w.side, wy, wz);
            const int32_t slot = atomicAdd(&cur[b >> s], 1);
            tpos[slot] = q[r];
            if (!ONE_RADIUS) tid[slot] = i;
            const int32_t g = ghost_offset(w, wx);
            if (g != 0) {
                const int32_t gslot = atomicAdd(&cur[(uint32_t)((int32_t)b + g) >> s], 1);
                const int32_t gi = (int32_t)((uint32_t)i | 0x80000000u);
                if (ONE_RADIUS) q[r].w = __int_as_float(gi);
                tpos[gslot] = q[r];
                if (!ONE_RADIUS) tid[gslot] = gi;
            }
        }
    }
}

/* Block b sorts window b (buckets [b kWindow, (b+1) kWindow)) of partition
 * b >> (s - kWindowBits), whose items sit in [off[p tiles], off[(p+1) tiles]).
 * A partition of at most kSortStage items is read once (each thread keeps
 * its items' buckets); the window's order is assembled in LDS as indices
 * into the partition, and the items are then copied out in that order, from
 * the L2, with consecutive stores.  A larger partition (a dense cluster, or
 * one of several windows) is read twice, to count and to place, and placed
 * by scattered stores. */
constexpr int kSortBlock = 512;
constexpr int kSortItems = 8;
constexpr int kSortStage = kSortBlock * kSortItems;
constexpr int kScanItems = kWindow / kSortBlock;
static_assert(kScanItems * kSortBlock == kWindow && kScanItems % 4 == 0, "the scan's share of a thread");
static_assert(kSortStage <= 65536, "staged indices are 16-bit");

template <bool ONE_RADIUS>
__global__ void __launch_bounds__(kSortBlock) k_coll_sort(const float4* tpos, const int32_t* tid,
                                                          const int32_t* off, const int32_t* totals, int64_t tiles,
                                                          int64_t cells, float inv_h, const int32_t* wrap,
                                                          int s, int32_t* start, float4* spos, int32_t* ids) {
    __shared__ int4 cnt4[kWindow / 4];
    int32_t* const cnt = reinterpret_cast<int32_t*>(cnt4);
    __shared__ uint16_t order[kSortStage];
    __shared__ int32_t wsum[kSortBlock / 64];
    const Wrap w = wrap_of(wrap);
    const int64_t b0 = (int64_t)blockIdx.x << kWindowBits;
    const int64_t p = (int64_t)blockIdx.x >> (s - kWindowBits);
    const int32_t lo = cell_offset(off, totals, p * tiles, cells);
    const int32_t hi = cell_offset(off, totals, (p + 1) * tiles, cells);
    const bool staged = hi - lo <= kSortStage;      /* block-uniform */
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int j = threadIdx.x; j < kWindow; j += kSortBlock) cnt[j] = 0;
    __syncthreads();
    /* staged: bucket - b0 of item lo + threadIdx.x + u kSortBlock, or
     * kWindow when it is not in the window */
    int32_t rr[kSortItems];
    int32_t below = 0;
    if (staged) {
#pragma unroll
        for (int u = 0; u < kSortItems; ++u) {
            const int32_t j = lo + (int32_t)threadIdx.x + u * kSortBlock;
            rr[u] = kWindow;
            if (j >= hi) continue;
            const float4 q = tpos[j];
            const int64_t r = (int64_t)item_bucket(w, q, item_id<ONE_RADIUS>(q, tid, j), inv_h) - b0;
            if (r < 0)
                ++below;
            else if (r < kWindow) {
                rr[u] = (int32_t)r;
                atomicAdd(&cnt[r], 1);
            }
        }
    } else {
        for (int32_t j = lo + (int32_t)threadIdx.x; j < hi; j += kSortBlock) {
            const float4 q = tpos[j];
            const int64_t r = (int64_t)item_bucket(w, q, item_id<ONE_RADIUS>(q, tid, j), inv_h) - b0;
            if (r < 0)
                ++below;
            else if (r < kWindow)
                atomicAdd(&cnt[r], 1);
        }
    }
    for (int d = 32; d > 0; d >>= 1) below += __shfl_xor(below, d);
    if (lane == 0) wsum[wave] = below;
    __syncthreads();
    int32_t carry = lo;
    for (int u = 0; u < kSortBlock / 64; ++u) carry += wsum[u];
    const int32_t first = carry;                    /* the window's first slot */
    __syncthreads();
    /* exclusive scan of the window's counts, kScanItems consecutive ones per
     * thread: the bucket starts, and the cursors of the placement below */
    {
        int4 v[kScanItems / 4];
        int32_t sum = 0;
#pragma unroll
        for (int u = 0; u < kScanItems / 4; ++u) {
            v[u] = cnt4[threadIdx.x * (kScanItems / 4) + u];
            sum += v[u].x + v[u].y + v[u].z + v[u].w;
        }
        int32_t x = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        int32_t e = carry + x - sum;
        for (int u = 0; u < kSortBlock / 64; ++u) {
            e += u < wave ? wsum[u] : 0;
            carry += wsum[u];
        }
        int4* const out = reinterpret_cast<int4*>(start + b0);
#pragma unroll
        for (int u = 0; u < kScanItems / 4; ++u) {
            int4 o;
            o.x = e;
            o.y = o.x + v[u].x;
            o.z = o.y + v[u].y;
            o.w = o.z + v[u].z;
            e = o.w + v[u].w;
            cnt4[threadIdx.x * (kScanItems / 4) + u] = o;
            out[threadIdx.x * (kScanItems / 4) + u] = o;
        }
        __syncthreads();
    }
    if (staged) {
        /* the window holds carry - first <= hi - lo <= kSortStage items */
#pragma unroll
        for (int u = 0; u < kSortItems; ++u) {
            if (rr[u] == kWindow) continue;
            order[atomicAdd(&cnt[rr[u]], 1) - first] = (uint16_t)(threadIdx.x + u * kSortBlock);
        }
        __syncthreads();
        for (int32_t j = threadIdx.x; j < carry - first; j += kSortBlock) {
            const int32_t from = lo + order[j];
            spos[first + j] = tpos[from];
            if (!ONE_RADIUS) ids[first + j] = tid[from];
        }
    } else {
        for (int32_t j = lo + (int32_t)threadIdx.x; j < hi; j += kSortBlock) {
            const float4 qj = tpos[j];
            const int32_t ij = item_id<ONE_RADIUS>(qj, tid, j);
            const int64_t r = (int64_t)item_bucket(w, qj, ij, inv_h) - b0;
            if (r >= 0 && r < kWindow) {
                const int32_t slot = atomicAdd(&cnt[r], 1);
                spos[slot] = qj;
                if (!ONE_RADIUS) ids[slot] = ij;
            }
        }
    }
}

/* One thread per sorted real slot (grid-stride; ghost slots are skipped):
 * consecutive lanes hold agents of the same or nearby cells, so the bucket
 * ranges and candidates they read are shared through the caches, and each
 * XCD takes a contiguous range of slots (xcd_tile).  The 4
 * candidate ranges are walked as one sequence, POTATO_QUERY_BATCH loads at
 * a time (indices past a lane's end read its own slot and are masked), and
 * a lane stops once it has found a collision.  (Copying each block's
 * candidate rows to LDS first, with consecutive loads, measured 1.25 times
 * slower at 1M agents: fewer waves per SIMD, a barrier per round, and the
 * L1 already serves most candidate reads.) */
constexpr int kRanges = 4;

template <bool ONE_RADIUS>
__global__ void __launch_bounds__(256) k_coll_query(const float4* spos, const int32_t* ids, const int32_t* start,
                                                    const int32_t* total, const float* radius, float inv_h,
                                                    const int32_t* wrap, uint8_t* alive, int32_t* died_part) {
#pragma clang fp contract(off)
    __shared__ int32_t wave_died[256 / 64];
    int32_t my_died = 0;
    const Wrap w = wrap_of(wrap);
    const float rs1 = radius[0] + radius[0];
    const int64_t slots = *total;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    for (int64_t k0 = tile * blockDim.x; k0 < slots; k0 += stride) {
        /* whole blocks stay in the loop together, so the reduction below
         * sees every lane; slot indices stay below 2^31 (at most two slots
         * per agent, fewer than 2^30 agents) */
        const int32_t k = (int32_t)(k0 + threadIdx.x);
        float4 pk = make_float4(0.0f, 0.0f, 0.0f, __int_as_float(-1));
        if (ONE_RADIUS && k < slots) pk = spos[k];
        const int32_t id = k < slots ? item_id<ONE_RADIUS>(pk, ids, k) : -1;
        bool hit = false;
        if (id >= 0) {
            if (!ONE_RADIUS) pk = spos[k];
            uint32_t wx, wy, wz;
            wrapped_cell(w, pk.x, pk.y, pk.z, inv_h, wx, wy, wz);
            /* the 4 (y, z) rows: bucket range of columns wx .. wx + 2 side (ghost-padded);
             * an axis wrapped to a single cell has no other row */
            const uint32_t ny = (wy + near_side(cell_index(pk.y, inv_h))) & w.my;
            const uint32_t nz = (wz + near_side(cell_index(pk.z, inv_h))) & w.mz;
            int32_t lo[kRanges], hi[kRanges];
#pragma unroll
            for (int r = 0; r < kRanges; ++r) {
                const uint32_t b0 = bucket_of(w, wx, r & 1 ? ny : wy, r & 2 ? nz : wz);
                lo[r] = start[b0];
                hi[r] = start[b0 + 2 * w.side + 1];
            }
            if (w.my == 0) hi[1] = lo[1], hi[3] = lo[3];
            if (w.mz == 0) hi[2] = lo[2], hi[3] = lo[3];
            /* candidate t of the sequence is slot t + d[r] for the last range r
             * whose first candidate number cum[r] is <= t */
            int32_t cum[kRanges], d[kRanges];
            int32_t T = 0;
#pragma unroll
            for (int r = 0; r < kRanges; ++r) {
                cum[r] = T;
                d[r] = lo[r] - T;
                T += hi[r] - lo[r];
            }
            auto collides = [&](const float4& pj) {
                const float ex = pk.x - pj.x, ey = pk.y - pj.y, ez = pk.z - pj.z;
                const float d2 = (ex * ex + ey * ey) + ez * ez;
                const float rs = ONE_RADIUS ? rs1 : pk.w + pj.w;
                return d2 < rs * rs;
            };
            constexpr int B = POTATO_QUERY_BATCH;
            for (int32_t t0 = 0; t0 < T && !hit; t0 += B) {
                float4 pc[B];
                bool use[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const int32_t t = t0 + u;
                    int32_t j = t + d[0];
#pragma unroll
                    for (int r = 1; r < kRanges; ++r) j = t >= cum[r] ? t + d[r] : j;
                    use[u] = t < T && j != k;
                    pc[u] = spos[t < T ? j : k];
                }
#pragma unroll
                for (int u = 0; u < B; ++u) hit |= use[u] && collides(pc[u]);
            }
            /* the query reads positions from the sorted copy only, so the
             * mask is updated in place */
            if (hit) alive[id] = 0;
        }
        my_died += hit ? 1 : 0;
    }
    /* agents marked dead by this block: a partial sum per block, added up by
     * k_coll_died (atomics on one counter serialise across the chip: one per
     * wave took most of the query's 0.21 ms at 1M agents; the last block
     * adding them up after a device-scope fence made the query 3.6 times
     * slower, one L2 write-back per block) */
    if (died_part) {
        int32_t x = my_died;
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
        if ((threadIdx.x & 63) == 0) wave_died[threadIdx.x / 64] = x;
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t sum = 0;
            for (int u = 0; u < (int)(blockDim.x / 64); ++u) sum += wave_died[u];
            died_part[blockIdx.x] = sum;
        }
    }
}

constexpr int kDiedBlock = 1024;

/* *died += the sum of the per-block counts of the query. */
__global__ void __launch_bounds__(kDiedBlock) k_coll_died(const int32_t* died_part, int n_part, unsigned long long* died) {
    __shared__ unsigned long long red[kDiedBlock / 64];
    unsigned long long x = 0;
#pragma unroll 4
    for (int b = threadIdx.x; b < n_part; b += kDiedBlock) x += (unsigned long long)died_part[b];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (int w = 0; w < kDiedBlock / 64; ++w) sum += red[w];
        *died += sum;
    }
}

/* Small swarms: every pair of agents, no grid.  The eight launches of the
 * grid pass cost their latencies, whatever the number of agents (31-33 us
 * from 2,000 to 20,000 agents); all n^2 / 2 pairs of 5,000 agents are 2 us of
 * FP32 work.  A wave holds the agents i of TILES tiles of 64, one per lane
 * and tile, and tests them against a tile of 64 agents j that its block
 * keeps in LDS and every lane reads at the same address.  The blocks cover
 * the tiles j from the block's own agents on, and a wave's ballots give both
 * sides of every pair: the i that collide with some j of the tile, and the j
 * that some i of the wave collides with.  Each is one 64-bit word, stored at
 * hits[tile of the marked agents][other tile]: every word has one writer, so
 * nothing is cleared beforehand, and the alive mask is only read here.
 * k_coll_mark then joins the words of a tile.  A dead agent, and a slot past
 * the end, takes a NaN position, which never passes the distance test.
 *
 * TILES: with one tile the LDS reads take longer than the tests, with two
 * they do not, but a wave then takes twice as long, which shows while the
 * waves do not fill the chip (1,000 / 5,000 / 8,000 / 10,000 / 16,000 agents:
 * 10.4 / 14.4 / 17.9 / 23.8 / 44 us with one, 13.5 / 16.0 / 21.0 / 21.3 / 36
 * with two): two from kPairsOneTile agents on.
 * kPairsMaxAgents: where the pairs' n^2 meets the grid pass's latencies
 * (12,000 agents: 26-28 us against 32; 13,000: 29-32 against 32-33; 14,000:
 * 31-33 against 32-33; 16,000: 36-39 against 32-33). */
constexpr int kPairBlock = 256;
constexpr int kPairWaves = kPairBlock / 64;
constexpr int64_t kPairsOneTile = 9216;
#ifndef POTATO_PAIRS_MAX
#define POTATO_PAIRS_MAX 13312
#endif
constexpr int64_t kPairsMaxAgents = POTATO_PAIRS_MAX;

template <int TILES, bool ONE_RADIUS>
__global__ void __launch_bounds__(kPairBlock) k_coll_pairs(const float* rows, int64_t ld, int32_t n,
                                                           const uint8_t* alive, const uint8_t* type, int n_types,
                                                           const float* radius, int32_t tiles,
                                                           unsigned long long* hits) {
#pragma clang fp contract(off)
    constexpr int kBlockTiles = kPairWaves * TILES;
    __shared__ float4 tile[64];
    const int32_t jt = blockIdx.x;
    const int32_t it0 = (int32_t)blockIdx.y * kBlockTiles;
    if (jt < it0) return;                           /* the pairs of another block */
    auto load = [&](int32_t i) {
        float4 q = make_float4(__builtin_nanf(""), 0.0f, 0.0f, 0.0f);
        if (i < n && alive[i])
            q = make_float4(rows[i], rows[ld + i], rows[2 * ld + i],
                            ONE_RADIUS ? radius[0] : radius[type_entry(type, (uint32_t)i, n_types)]);
        return q;
    };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave == 0) tile[lane] = load(jt * 64 + lane);
    float4 q[TILES];
    int32_t it[TILES];
#pragma unroll
    for (int u = 0; u < TILES; ++u) {
        it[u] = it0 + u * kPairWaves + wave;
        q[u] = load(it[u] * 64 + lane);
    }
    __syncthreads();
    const float rs1 = radius[0] + radius[0];
    const float rr1 = rs1 * rs1;
    unsigned long long row[TILES] = {};
    uint32_t col[TILES][2] = {};
    /* agent j of the tile against the wave's agents; own: the tile of the
     * wave's that j itself is of (an agent does not collide with itself) */
    auto test = [&](int own) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll 8
            for (int j = 0; j < 32; ++j) {
                const float4 p = tile[h * 32 + j];
#pragma unroll
                for (int u = 0; u < TILES; ++u) {
                    const float ex = q[u].x - p.x, ey = q[u].y - p.y, ez = q[u].z - p.z;
                    const float d2 = (ex * ex + ey * ey) + ez * ez;
                    const float rs = q[u].w + p.w;
                    unsigned long long m = __ballot(d2 < (ONE_RADIUS ? rr1 : rs * rs));
                    if (own == u) m &= ~(1ull << (h * 32 + j));
                    row[u] |= m;
                    if (m) col[u][h] |= 1u << j;
                }
            }
    };
    static_assert(TILES <= 2, "one case per tile of the wave");
    if (jt == it[0])
        test(0);
    else if (TILES > 1 && jt == it[TILES - 1])
        test(TILES - 1);
    else
        test(-1);
    if (lane != 0) return;
#pragma unroll
    for (int u = 0; u < TILES; ++u) {
        if (it[u] >= tiles) continue;
        hits[(int64_t)it[u] * tiles + jt] = row[u];
        /* among the block's own tiles every wave tests every tile, so the
         * other side's word is its own wave's */
        if (jt >= it0 + kBlockTiles)
            hits[(int64_t)jt * tiles + it[u]] = (unsigned long long)col[u][1] << 32 | col[u][0];
    }
}

/* One block per tile of 64 agents: joins the tile's words, marks its agents
 * dead and adds their number to *died (at most one atomic per 64 agents). */
__global__ void __launch_bounds__(kPairBlock) k_coll_mark(const unsigned long long* hits, int32_t tiles,
                                                          uint8_t* alive, unsigned long long* died) {
    __shared__ unsigned long long part[kPairBlock / 64];
    const unsigned long long* const words = hits + (int64_t)blockIdx.x * tiles;
    unsigned long long m = 0;
    for (int32_t t = threadIdx.x; t < tiles; t += kPairBlock) m |= words[t];
    for (int off = 32; off > 0; off >>= 1) m |= __shfl_xor(m, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    m = part[0];
#pragma unroll
    for (int u = 1; u < kPairBlock / 64; ++u) m |= part[u];
    if (m >> threadIdx.x & 1ull) alive[(int64_t)blockIdx.x * 64 + threadIdx.x] = 0;
    if (threadIdx.x == 0 && died && m) atomicAdd(died, (unsigned long long)__popcll(m));
}

}  // namespace

namespace {

/* Bucket budget 2^k >= 2N, at least 2^10 (the wrap splits its k bits). */
constexpr int budget_bits(int64_t n) {
    int k = 10;
    while ((int64_t(1) << k) < 2 * n && k < 30) ++k;
    return k;
}

/* Buckets allocated: the budget plus the ghost columns (at most 2 per
 * 2^kMinXBits columns). */
constexpr int64_t buckets_alloc(int64_t n) {
    const int k = budget_bits(n);
    return (int64_t(1) << k) + (int64_t(1) << (k + 1 - kMinXBits));
}

/* Sizes of the two-level sort at N agents. */
struct SortPlan {
    int k;            /* bucket budget bits */
    int s;            /* log2 of the buckets per partition */
    int64_t parts;    /* partitions: parts << s >= m + 1, m the buckets allocated */
    int64_t tile;     /* agents per tile, a multiple of kTileAgents */
    int64_t tiles;    /* at most kMaxTiles */
};

constexpr SortPlan sort_plan(int64_t n) {
    SortPlan q{};
    q.k = budget_bits(n);
    const int64_t m1 = buckets_alloc(n) + 1;
    q.s = kWindowBits;
    while (((m1 + (int64_t(1) << q.s) - 1) >> q.s) > kMaxParts) ++q.s;
    q.parts = (m1 + (int64_t(1) << q.s) - 1) >> q.s;
    const int64_t per = (n + kTileAgents * kMaxTiles - 1) / (kTileAgents * kMaxTiles);
    q.tile = kTileAgents * (per < 1 ? 1 : per);
    q.tiles = (n + q.tile - 1) / q.tile;
    return q;
}

constexpr int64_t workspace_for(int64_t n) {
    const SortPlan q = sort_plan(n);
    const int64_t cells = q.parts * q.tiles;
    const int64_t chunks = (cells + kScanBlock - 1) / kScanBlock;
    /* items (x, y, z, r) in partition order and in bucket order [2n] each
     * first (16-byte aligned: agents and ghosts); their ids [2n] each;
     * bucket starts [parts << s]; partition-tile offsets [parts * tiles + 1];
     * chunk totals of their scan [chunks]; bits of the wrap [4 of 6]; the
     * bounding box's per-block partials [kBoxWords]; the query's per-block counts of dead agents */
    const int64_t blocks = (n + 255) / 256;
    return 16 * 4 * n + 4 * (4 * n + (q.parts << q.s) + cells + 1 + chunks + 6 + kBoxWords + blocks) + 256;
}

/* Workspace of the allocation-free entry point: a file-scope device array
 * sized for the largest swarm it accepts.  Every GPU the library runs on
 * holds its own copy until the process ends; host code reaches it only
 * through the address hipGetSymbolAddress returns for the current device
 * (the array's name in host code is not a device address). */
constexpr int64_t kNoAllocBytes = workspace_for(kNoAllocMaxAgents);

}  // namespace

/* the pairs' words, one per pair of tiles, fit the workspace */
constexpr int64_t kPairTilesMax = (kPairsMaxAgents + 63) / 64;
static_assert(kPairTilesMax * kPairTilesMax * 8 <= workspace_for(kPairsMaxAgents) && workspace_for(1) >= 8,
              "hit words of the pairs pass (n^2 / 512 bytes against more than 80 n)");

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

int64_t collision_workspace_bytes(int64_t n) { return workspace_for(n); }

hipError_t collision_scratch(void** ptr, int64_t* bytes) {
    static std::mutex mu;
    static std::vector<void*> addr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> g(mu);
    if ((size_t)dev >= addr.size()) addr.resize((size_t)dev + 1, nullptr);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = kNoAllocBytes;
    return hipSuccess;
}

hipError_t launch_detect_collisions(const float* rows, int64_t ld, int64_t n, const uint8_t* type, int n_types,
                                    const float* radius_dev, float r_max, uint8_t* alive,
                                    unsigned long long* died, void* workspace, hipStream_t s) {
    if (n <= kPairsMaxAgents) {
        const int32_t tiles = (int32_t)((n + 63) / 64);
        unsigned long long* hits = reinterpret_cast<unsigned long long*>(workspace);
        const int two = n > kPairsOneTile ? 1 : 0;
        const int32_t per_block = kPairWaves << two;
        const dim3 grid((unsigned)tiles, (unsigned)((tiles + per_block - 1) / per_block));
        auto* const fn = two ? (type ? k_coll_pairs<2, false> : k_coll_pairs<2, true>)
                             : (type ? k_coll_pairs<1, false> : k_coll_pairs<1, true>);
        hipLaunchKernelGGL(fn, grid, dim3(kPairBlock), 0, s, rows, ld, (int32_t)n, alive, type, n_types, radius_dev,
                           tiles, hits);
        hipLaunchKernelGGL(k_coll_mark, dim3((unsigned)tiles), dim3(kPairBlock), 0, s, hits, tiles, alive, died);
        return hipGetLastError();
    }
    const SortPlan q = sort_plan(n);
    const int64_t cells = q.parts * q.tiles;
    float4* tpos = reinterpret_cast<float4*>(workspace);
    float4* spos = tpos + 2 * n;
    int32_t* tid = reinterpret_cast<int32_t*>(spos + 2 * n);
    int32_t* ids = tid + 2 * n;
    int32_t* start = ids + 2 * n;
    int32_t* off = start + (q.parts << q.s);
    int32_t* totals = off + cells + 1;
    int32_t* wrap = totals + scan_chunks((uint32_t)cells);
    int32_t* partial = wrap + 6;
    int32_t* died_part = partial + kBoxWords;
    const float inv_h = 1.0f / (2.02f * r_max);
    const unsigned nb = (unsigned)((n + 255) / 256);
    const unsigned nbox = std::min<unsigned>((unsigned)((n + kBoxThreads - 1) / kBoxThreads), kBoxBlocks);
    const size_t lds = (size_t)q.parts * sizeof(int32_t);
    hipLaunchKernelGGL(k_coll_bounds, dim3(nbox), dim3(kBoxThreads), 0, s, rows, ld, n, alive, inv_h, partial);
    hipLaunchKernelGGL(k_coll_hist, dim3((unsigned)q.tiles), dim3(kTileBlock), lds, s, rows, ld, n, alive, inv_h,
                       partial, (int)nbox, wrap, q.k, q.s, (int32_t)q.parts, q.tile, off);
    /* in place, chunk by chunk (the consumers add the chunk totals); the
     * slot count goes to off[cells] */
    launch_exclusive_scan_chunks(off, off, totals, off + cells, (uint32_t)cells, s);
    hipLaunchKernelGGL((type ? k_coll_part<false> : k_coll_part<true>), dim3((unsigned)q.tiles), dim3(kTileBlock), lds,
                       s, rows, ld, n, alive, type, n_types, radius_dev, inv_h, wrap, q.s, (int32_t)q.parts, q.tile,
                       off, totals, tpos, tid);
    hipLaunchKernelGGL((type ? k_coll_sort<false> : k_coll_sort<true>), dim3((unsigned)((q.parts << q.s) >> kWindowBits)),
                       dim3(kSortBlock), 0, s, tpos, tid, off, totals, q.tiles, cells, inv_h, wrap, q.s, start, spos,
                       ids);
    hipLaunchKernelGGL((type ? k_coll_query<false> : k_coll_query<true>), dim3(nb), dim3(256), 0, s, spos, ids, start,
                       off + cells, radius_dev, inv_h, wrap, alive, died ? died_part : nullptr);
    if (died) hipLaunchKernelGGL(k_coll_died, dim3(1), dim3(kDiedBlock), 0, s, died_part, (int)nb, died);
    return hipGetLastError();
}

}  // namespace potato
