// Short-range particle-particle force on gfx950 (Eq. (force), Sec. 3.1).
//
// After binning (sr_bin.hip) the particles sit cell by cell in a float4
// (x, y, z, m) copy.  Each force work item is one cell's chunk of at most 128
// targets, or a sub-item taking a consecutive part of that chunk's stencil
// sources.  One wavefront owns an item:
//   - the 27 neighbour cells are 9 rows of 3 cells that are contiguous in the
//     sorted order, so the source list is at most 18 contiguous pieces (a row
//     splits in two where it wraps around a periodic face; in split
//     coordinates each neighbour cell is a piece of its own);
//   - sources pass by in windows of 64 (sr_item.h) with their periodic image
//     shift applied; those that reach the box of the item's targets are staged
//     in LDS and read back by broadcast;
//   - when a cell holds few targets the 64 lanes are split into S groups that
//     take the staged sources in turn, and the groups' sums are added in a
//     fixed order through LDS at the end;
//   - the targets of dense cells are put in Morton order first (sub_order), so
//     that an item's targets fill a small part of the cell;
//   - a lane may hold two targets, so that every source it reads serves both:
//     an item takes whichever of one or two targets per lane leaves fewer
//     lanes idle (up to 128 targets per item);
//   - the pair loop is plain float32 VALU: one reciprocal square root,
//     the polynomial in registers, the cutoff as a mask on the accumulation
//     (Sec. 3.1 describes select-based filtering inside the force loop).
// Periodic images are made exact: a target in the last cell layer of an axis
// works in a frame shifted by -L there, so every image shift is 0 or -L and is
// only ever applied to coordinates >= L/2, where subtracting L is exact.
//
// Everything runs on a batch of boxes (one box = a batch of one): a work item
// carries its box, whose geometry, inputs and outputs it reads from the
// batch descriptor.  Items may be ordered by decreasing cost bucket (longest
// first) and are either one workgroup each (a workgroup also takes positions
// + k gridDim when sub-items outnumber the grid) or pulled from a counter by
// persistent workgroups; the sub-items' partial sums are then added by
// k_subsum.
#include <climits>
#include <cmath>

#include "sr_internal.h"
#include "sr_item.h"
#include "sr_pair.h"

namespace {

// Position in the item order served by workgroup b: workgroups are dealt to
// the 8 XCDs round-robin, and XCD k serves the chunks of 64 consecutive
// items k, k + 8, k + 16, ..., so each XCD sees the same mix of costs and
// neighbouring cells (shared sources) meet in one L2.  A bijection on
// [0, grid) for grid a multiple of 512.
__device__ __forceinline__ int item_position(int b)
{
    const int xcd = b & 7, j = b >> 3;
    return ((j >> 6) * 8 + xcd) * 64 + (j & 63);
}

// One workgroup per item: the grid covers the chunk bound (a multiple of 512;
// at most kMaskedGrid workgroups in masked passes), and a workgroup also
// serves positions + k gridDim when sub-items make more items than that.
__global__ __launch_bounds__(64, 8) void k_force(Batch B, const int4 *__restrict__ items,
                                                 const int *__restrict__ n_items,
                                                 const float4 *__restrict__ sorted,
                                                 const int *__restrict__ offsets,
                                                 const int *__restrict__ perm,
                                                 const int *__restrict__ mass_mixed, ForceParams fp,
                                                 float *__restrict__ subsums)
{
    __shared__ ItemShared sh;
    const int n = *n_items;
    for (int pos = item_position(blockIdx.x); pos < n; pos += gridDim.x)
        process_item(B, items[pos], sorted, offsets, perm, mass_mixed, fp, sh, threadIdx.x,
                     subsums);
}

// Adds the partial sums of the sub-items of every chunk cut into sub-items
// (heads: each chunk's first sub-item), in sub-item order, and writes the chunk's
// accelerations (passive targets' partials are exact zeros).  One wavefront per
// head (grid-stride), two targets per lane at most.  Latency-bound: the sums of a
// target are all loaded before the first is added; its only scattered accesses
// are the three it writes.
__global__ __launch_bounds__(256) void k_subsum(Batch B, const int4 *__restrict__ heads,
                                                const int *__restrict__ n_heads,
                                                const int *__restrict__ perm,
                                                const float *__restrict__ subsums)
{
    const int n = *n_heads, lane = threadIdx.x & 63;
    for (int h = blockIdx.x * 4 + (threadIdx.x >> 6); h < n; h += gridDim.x * 4) {
        const int4 item = heads[h];
        const int ns = __builtin_amdgcn_readfirstlane(item_nsub(item));
        const BoxDesc &d = box_at(B, item_box(item));
        for (int t = lane; t < item.z; t += 64) {
            const int slot = item.y + t;
            float v[kMaxSrcSplit][3];
#pragma unroll
            for (int k = 0; k < kMaxSrcSplit; ++k)
                if (k < ns)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        v[k][c] = subsums[subsum_at(k, c, B.ntot, slot)];
            const int orig = perm[slot] - d.pbase;
#pragma unroll
            for (int k = 1; k < kMaxSrcSplit; ++k)
                if (k < ns)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        v[0][c] += v[k][c];
            d.ax[orig] = v[0][0];
            d.ay[orig] = v[0][1];
            d.az[orig] = v[0][2];
        }
    }
}

// Persistent variant: a fixed grid of workgroups takes kPersistentGrab
// consecutive items at a time from a counter until none are left (every
// workgroup reaches the exit).  Taking two per atomic halves the traffic on
// the one counter address, which bounded the pass on many-item batches.
constexpr int kPersistentGrab = 2;
__global__ __launch_bounds__(64, 8) void k_force_persistent(Batch B, const int4 *__restrict__ items,
                                                            const int *__restrict__ n_items,
                                                            const float4 *__restrict__ sorted,
                                                            const int *__restrict__ offsets,
                                                            const int *__restrict__ perm,
                                                            const int *__restrict__ mass_mixed,
                                                            ForceParams fp,
                                                            int *__restrict__ queue,
                                                            float *__restrict__ subsums)
{
    __shared__ ItemShared sh;
    __shared__ int next;
    const int n = *n_items;
    for (;;) {
        if (threadIdx.x == 0)
            next = atomicAdd(queue, kPersistentGrab);
        __syncthreads();
        const int p0 = __builtin_amdgcn_readfirstlane(next);
        __syncthreads();
        if (p0 >= n)
            break;
        const int pe = p0 + kPersistentGrab < n ? p0 + kPersistentGrab : n;
        for (int pos = p0; pos < pe; ++pos)
            process_item(B, items[pos], sorted, offsets, perm, mass_mixed, fp, sh, threadIdx.x,
                         subsums);
    }
}

// Useful-pair and candidate counts with the same stencil, chunks and cutoff
// test (one box; a chunk's sub-items, which share its target box, count as one).
__global__ __launch_bounds__(64) void k_pair_stats(Batch B, const int4 *__restrict__ items,
                                                   const int *__restrict__ n_items,
                                                   const float4 *__restrict__ sorted,
                                                   const int *__restrict__ offsets,
                                                   const int *__restrict__ perm, ForceParams fp,
                                                   int *__restrict__ per_target,
                                                   unsigned long long *__restrict__ stats)
{
    __shared__ float4 tile[kTile];
    __shared__ Stencil st;
    const int lane = threadIdx.x;
    const int it = blockIdx.x;
    if (it >= *n_items)
        return;
    const int4 item = items[it];
    const int kb = item.y, nt = item.z;
    const BoxDesc &d = box_at(B, item_box(item));
    const Geom &g = d.g;
    int cx, cy, cz;
    decode_cell(item.x - d.cbase, g, cx, cy, cz);
    const int cc[3] = {cx, cy, cz};
    float F[3];
    frame_shift(g, cc, F);
    build_stencil(st, offsets + d.cbase, g, cx, cy, cz, F, lane);
    // up to 128 targets: lane l counts for targets l and l + 64
    bool act[2], has[2];
    float xi[2], yi[2], zi[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        has[h] = lane + 64 * h < nt;
        const float4 pt = sorted[kb + (has[h] ? lane + 64 * h : 0)];
        act[h] = has[h] && !is_passive(pt, g);
        xi[h] = pt.x + F[0];
        yi[h] = pt.y + F[1];
        zi[h] = pt.z + F[2];
    }
    __syncthreads();
    const int total = st.pbeg[kMaxPieces];
    // the force pass's box test, so that the counts cover exactly the sources
    // it evaluates (and a useful pair it dropped would show in per_target)
    const TargetBox tb = target_box(xi[0], yi[0], zi[0], xi[1], yi[1], zi[1]);
    int cntu[2] = {0, 0};
    int kept = 0;
    int p = 0;
    for (int g0 = 0; g0 < total; g0 += kTile) {
        const int cnt = total - g0 < kTile ? total - g0 : kTile;
        float4 pre[kTile / 64];
        load_tile(pre, st, sorted, g0, cnt, lane, p);
        const int nk = store_tile_kept(tile, pre, tb, fp, lane);
        kept += nk;
        __syncthreads();
        for (int j = 0; j < nk; ++j) {
            const float4 s = tile[j];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float dx = s.x - xi[h], dy = s.y - yi[h], dz = s.z - zi[h];
                const float se = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, fp.eps)));
                cntu[h] += se < fp.rcut ? 1 : 0;
            }
        }
        __syncthreads();
    }
    unsigned long long u = 0ull, c = 0ull;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        cntu[h] = act[h] ? cntu[h] - 1 : 0;  // the target itself is always in its stencil
        if (has[h] && per_target)
            per_target[perm[kb + lane + 64 * h] - d.pbase] = cntu[h];
        u += (unsigned long long)cntu[h];
        c += act[h] ? (unsigned long long)kept : 0ull;
    }
    for (int o = 1; o < 64; o <<= 1) {
        u += __shfl_xor(u, o, 64);
        c += __shfl_xor(c, o, 64);
    }
    if (lane == 0) {
        atomicAdd(&stats[0], u);
        atomicAdd(&stats[1], c);
    }
}

// Work items of a block of kItemCells cells: each of the first kItemCells
// threads takes one cell's chunk and sub-item counts (split: the chunks of
// boxes that box_splits admits, and of any box in masked passes, are cut by
// cell_cut; with target counts, a masked pass, the chunks cover the cell's
// first tcount[c] slots, where its active particles sit), the block
// reserves its item range with one atomic on *n_items, then all threads
// write the block's items, thread j the items j, j + kT, ... (the cell of an
// item found by a binary search over the block's running item counts).  The
// order of the items depends on which block reserves first; no result does:
// every target is summed in a fixed order, by one item or by its chunk's
// sub-items added in order.  The first sub-item of every cut chunk is also
// appended to heads, for k_subsum.  The target slots of cells of more than
// kChunk2 targets are appended to segs, in segments of at most kSegLen, for
// sub_order.
//
// The atomics on the counters (one address, 12 ns each) bound it where there are
// many blocks, the longest block where there are few: passes of kMostCells cells or
// more take 1024 cells per block (100000 particles in 128^3 cells: 100 us with 256,
// 30 with 1024), of kManyCells or more 256 (128^3 lattice, 79507 cells: the pass 585
// us with 64, 574 with 256), others 64 (a halo box of 154003 particles 468 against
// 475 us), by 1024 threads: the cells of a halo's core, with thousands of sub-items,
// sit in one block (that box 460 us with 1024, 469 with 256; an 80^3 halo box 1955
// and 1988).
constexpr int kManyCells = 32768;
constexpr int kMostCells = 1 << 18;
// What k_items cuts: kCutNone whole chunks only, kCutSub chunks and sub-items,
// kCutChunks the same chunks as one item each (sr_pair_stats: the force pass's
// target boxes, with every source counted once).
constexpr int kCutNone = 0, kCutSub = 1, kCutChunks = 2;
constexpr int kSegThreads = 512;  // threads that order a segment
constexpr int kSegRounds = 8;     // slots per thread
constexpr int kSegLen = kSegThreads * kSegRounds;
template <int kItemCells, int kT>
__global__ __launch_bounds__(kT) void k_items(Batch B, const int *__restrict__ offsets,
                                               const int *__restrict__ cell_src,
                                               const unsigned long long *__restrict__ work,
                                               const int *__restrict__ tcount,
                                               const int *__restrict__ partial, int split,
                                               int4 *__restrict__ items,
                                               int *__restrict__ item_cost,
                                               int *__restrict__ n_items,
                                               int4 *__restrict__ heads,
                                               int *__restrict__ n_heads,
                                               int *__restrict__ lpt, int2 *__restrict__ segs,
                                               int *__restrict__ n_segs)
{
    static_assert(kT >= kItemCells, "one cell per thread");
    constexpr int kItemWaves = kItemCells / 64;
    __shared__ int base, sbase;
    __shared__ int s_wave[kItemWaves], s_wseg[kItemWaves];  // items and segments per wavefront
    __shared__ int hist[32];  // the block's items per cost bucket, for the longest-first order
    if (threadIdx.x < 32)
        hist[threadIdx.x] = 0;
    __shared__ int s_end[kItemCells];  // the block's items up to and including each cell
    __shared__ int s_q[kItemCells], s_ns[kItemCells], s_b[kItemCells], s_len[kItemCells];
    __shared__ int s_box[kItemCells], s_full[kItemCells], s_src[kItemCells];
    const int t = threadIdx.x, w = t >> 6;
    int q = 0, ns = 1, box = 0, full = kChunk2, src = 0, b = 0, len = 0, first = 0, seg = 0;
    if (t < kItemCells) {
        const int c = blockIdx.x * kItemCells + t;
        b = c < B.ctot ? offsets[c] : 0;
        // masked passes: the active particles, sorted to the front of the cell
        len = c >= B.ctot ? 0 : (tcount ? tcount[c] : offsets[c + 1] - b);
        if (len > 0) {
            box = find_box(B.cstart, B.nb, c);
            src = cell_src[c];
            if (split != kCutNone && (tcount || box_splits(box_at(B, box).n)))
                ns = cell_cut(len, src, item_pairs(work[box], tcount && *partial), &full);
            if (split == kCutChunks)
                ns = 1;
            q = mesh_chunks(len, full);
        }
        const int nseg = len > kChunk2 ? (len + kSegLen - 1) / kSegLen : 0;
        int tot, all = 0;
        first = wave_exclusive_scan(q * ns, t & 63, &tot);
        if (__any(nseg > 0))
            seg = wave_exclusive_scan(nseg, t & 63, &all);
        if ((t & 63) == 0) {
            s_wave[w] = tot;
            s_wseg[w] = all;
        }
    }
    __syncthreads();
    if (t == 0) {
        int tot = 0, all = 0;
        for (int v = 0; v < kItemWaves; ++v) {
            tot += s_wave[v];
            all += s_wseg[v];
        }
        base = tot > 0 ? atomicAdd(n_items, tot) : 0;
        sbase = all > 0 ? atomicAdd(n_segs, all) : 0;
    }
    if (t < kItemCells) {
        for (int v = 0; v < w; ++v) {
            first += s_wave[v];
            seg += s_wseg[v];
        }
        s_end[t] = first + q * ns;
        s_q[t] = q;
        s_ns[t] = ns;
        s_b[t] = b;
        s_len[t] = len;
        s_box[t] = box;
        s_src[t] = src;
        s_full[t] = full;
    }
    __syncthreads();
    if (t < kItemCells && len > kChunk2)
        for (int k = 0; k * kSegLen < len; ++k)
            segs[sbase + seg + k] =
                make_int2(b + k * kSegLen, len - k * kSegLen < kSegLen ? len - k * kSegLen
                                                                       : kSegLen);
    const int T = s_end[kItemCells - 1];
    for (int j = threadIdx.x; j < T; j += kT) {
        int lo = 0, hi = kItemCells - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_end[mid] > j)
                hi = mid;
            else
                lo = mid + 1;
        }
        const int qq = s_q[lo], nn = s_ns[lo];
        const int r = j - (s_end[lo] - qq * nn);
        const int k = r / nn;
        int bucket;
        const int4 it = cell_item(blockIdx.x * kItemCells + lo, s_box[lo], s_b[lo], s_len[lo], qq,
                                  s_full[lo], k, nn, r - k * nn, s_src[lo], &bucket);
        items[base + j] = it;
        item_cost[base + j] = bucket;
        atomicAdd(&hist[31 - bucket], 1);
        if (nn > 1 && r == k * nn)
            heads[atomicAdd(n_heads, 1)] = it;
    }
    __syncthreads();
    if (threadIdx.x < 32 && hist[threadIdx.x] > 0)
        atomicAdd(&lpt[threadIdx.x], hist[threadIdx.x]);
}

// Longest-first order of the items: a counting sort by decreasing cost
// bucket (key = 31 - bucket).  The kernels that write the items add their key
// counts into 32 global totals; k_lpt_scatter gives key k the range starting at
// the totals of the keys before it, reserves one sub-range per (block, key)
// with an atomic, and places its items there in their original order.  Which
// block gets which sub-range depends on timing, so the item order inside a
// key is not fixed -- results are: every target is summed entirely inside
// one item, in a fixed order, whatever the order of the items.
// lpt[0..31] are the key totals and lpt[32..63] the key cursors, all zero
// before the items are written (the binning pass clears them).
template <int kT>
__device__ __forceinline__ void lpt_scatter(int block, const int4 *__restrict__ items,
                                            const int *__restrict__ item_cost,
                                            const int *__restrict__ n_items,
                                            int *__restrict__ lpt, int4 *__restrict__ out)
{
    __shared__ int run[32];
    __shared__ int hcnt[32];
    __shared__ int wcnt[kT / 64][32];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int n = *n_items;
    if (block * kLptBlock >= n)
        return;
    if (threadIdx.x < 32)
        hcnt[threadIdx.x] = 0;
    __syncthreads();
    for (int k = 0; k < kLptBlock / kT; ++k) {
        const int i = block * kLptBlock + k * kT + threadIdx.x;
        if (i < n)
            atomicAdd(&hcnt[31 - item_cost[i]], 1);
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        int base = 0;
        for (int k = 0; k < (int)threadIdx.x; ++k)
            base += lpt[k];
        const int c = hcnt[threadIdx.x];
        run[threadIdx.x] = c > 0 ? base + atomicAdd(&lpt[32 + threadIdx.x], c) : 0;
    }
    for (int k = 0; k < kLptBlock / kT; ++k) {
        if (threadIdx.x < kT / 2)
            wcnt[threadIdx.x >> 5][threadIdx.x & 31] = 0;
        __syncthreads();
        const int i = block * kLptBlock + k * kT + threadIdx.x;
        const bool live = i < n;
        const int key = live ? 31 - item_cost[i] : 0;
        // lanes of this wavefront with the same key, by 5 ballots
        unsigned long long same = __ballot(live);
#pragma unroll
        for (int bit = 0; bit < 5; ++bit) {
            const unsigned long long v = __ballot(live && ((key >> bit) & 1));
            same &= ((key >> bit) & 1) ? v : ~v;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        if (live && rank == 0)
            wcnt[wid][key] = __popcll(same);
        __syncthreads();
        if (live) {
            int before = run[key];
            for (int w = 0; w < wid; ++w)
                before += wcnt[w][key];
            out[before + rank] = items[i];
        }
        __syncthreads();
        if (threadIdx.x < 32)
#pragma unroll
            for (int w = 0; w < kT / 64; ++w)
                run[threadIdx.x] += wcnt[w][threadIdx.x];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_lpt_scatter(const int4 *__restrict__ items,
                                                     const int *__restrict__ item_cost,
                                                     const int *__restrict__ n_items,
                                                     int *__restrict__ lpt,
                                                     int4 *__restrict__ out)
{
    lpt_scatter<256>(blockIdx.x, items, item_cost, n_items, lpt, out);
}

// Sub-order of a segment of a cell's target slots, len <= kSegLen: a stable
// counting sort of the slots by the Morton code of their eighth (per axis) of
// the segment's own bounding box.  The cell's items take consecutive slots, so
// each one's targets then fill a small part of the cell, and fewer sources pass
// the test against their box (on the 256^3 clustered share 9570 candidates per
// target instead of 10549 in input order, by a CPU model; 9670 with quarters).
// The order depends on the cell's targets alone, so a box gives the same bits
// alone and in a batch.  A masked pass orders the active particles, the front of
// each cell, only: it agrees bitwise with a plain pass when every particle is
// active, else to float32 summation order.  k_force on that share 64.1 -> 57.9
// ms, on an 80^3 halo box 1.99 -> 1.89 ms.  Cells of at most kChunk2 targets are
// one item or few small ones, and stay as they are.
//
// Latency bounds it on small boxes (14 us with 16 slots per thread and 256
// threads on a halo box of 154003 particles, 5 us of them the launch and the item
// order) and its two passes over the slots (20 bytes in, 20 out) on large ones:
// the wavefronts rank their particles with ballots and keep them in registers
// meanwhile.  Segments of 4096 slots at 8 per thread: with 8192 at 16 the share
// gains another 1 % and the box of 154003 loses that.
constexpr int kSegKeys = 512;
constexpr int kSegWaves = kSegThreads / 64;
static_assert(kSegThreads >= kSegKeys, "one key per thread");

struct SegShared {
    float lo[3][kSegWaves], hi[3][kSegWaves];
    int hist[kSegWaves][kSegKeys];  // per wavefront and key: particles, then first slot
    int wsum[kSegKeys / 64];
};

__device__ __forceinline__ int spread3(int v) { return (v & 1) | (v & 2) << 2 | (v & 4) << 4; }

__device__ void sub_order(SegShared &S, float4 *__restrict__ sorted, int *__restrict__ perm, int s0,
                          int len)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // wavefront w holds slots [w 64 R, (w + 1) 64 R), lane by lane in rounds
    const int R = (len + kSegThreads - 1) / kSegThreads, first = w * 64 * R + lane;
    float4 q[kSegRounds];
    int pi[kSegRounds];
    float lo[3] = {3.0e38f, 3.0e38f, 3.0e38f}, hi[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r)
        if (r < R) {
            const int i = first + r * 64;
            const int j = s0 + (i < len ? i : 0);
            q[r] = sorted[j];
            pi[r] = perm[j];
        }
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r)
        if (r < R) {
            // all loads are back before any slot is written
            asm volatile("" : "+v"(q[r].w), "+v"(pi[r]));
            lo[0] = fminf(lo[0], q[r].x);
            lo[1] = fminf(lo[1], q[r].y);
            lo[2] = fminf(lo[2], q[r].z);
            hi[0] = fmaxf(hi[0], q[r].x);
            hi[1] = fmaxf(hi[1], q[r].y);
            hi[2] = fmaxf(hi[2], q[r].z);
        }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, 64));
            hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, 64));
        }
        if (lane == 0) {
            S.lo[d][w] = lo[d];
            S.hi[d][w] = hi[d];
        }
    }
    for (int k = tid; k < kSegKeys; k += kSegThreads)
#pragma unroll
        for (int v = 0; v < kSegWaves; ++v)
            S.hist[v][k] = 0;
    __syncthreads();
    float l[3], inv[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        l[d] = S.lo[d][0];
        float h = S.hi[d][0];
#pragma unroll
        for (int v = 1; v < kSegWaves; ++v) {
            l[d] = fminf(l[d], S.lo[d][v]);
            h = fmaxf(h, S.hi[d][v]);
        }
        inv[d] = h > l[d] ? 8.f / (h - l[d]) : 0.f;
    }
    int kr[kSegRounds];  // key << 16 | rank among the wavefront's particles of the key
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r) {
        kr[r] = 0;
        if (r < R) {
            const bool live = first + r * 64 < len;
            const int cx = (int)fminf(fmaxf((q[r].x - l[0]) * inv[0], 0.f), 7.f);
            const int cy = (int)fminf(fmaxf((q[r].y - l[1]) * inv[1], 0.f), 7.f);
            const int cz = (int)fminf(fmaxf((q[r].z - l[2]) * inv[2], 0.f), 7.f);
            const int key = spread3(cx) | spread3(cy) << 1 | spread3(cz) << 2;
            unsigned long long same = __ballot(live);
#pragma unroll
            for (int bit = 0; bit < 9; ++bit) {
                const unsigned long long v = __ballot((key >> bit) & 1);
                same &= ((key >> bit) & 1) ? v : ~v;
            }
            const int below = __popcll(same & ((1ull << lane) - 1ull));
            int before = 0;
            if (live && below == 0)
                before = atomicAdd(&S.hist[w][key], __popcll(same));
            const int leader = live ? __ffsll(same) - 1 : lane;
            before = __shfl(before, leader, 64);
            kr[r] = key << 16 | (before + below);
        }
    }
    __syncthreads();
    // first slot of each key, then of each wavefront within it
    int t = 0, at = 0;
    if (tid < kSegKeys) {
#pragma unroll
        for (int v = 0; v < kSegWaves; ++v)
            t += S.hist[v][tid];
        int tot;
        at = wave_exclusive_scan(t, lane, &tot);
        if (lane == 0)
            S.wsum[w] = tot;
    }
    __syncthreads();
    if (tid < kSegKeys) {
        for (int v = 0; v < w; ++v)
            at += S.wsum[v];
#pragma unroll
        for (int v = 0; v < kSegWaves; ++v) {
            const int c = S.hist[v][tid];
            S.hist[v][tid] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSegRounds; ++r)
        if (r < R && first + r * 64 < len) {
            const int j = s0 + S.hist[w][kr[r] >> 16] + (kr[r] & 0xffff);
            sorted[j] = q[r];
            perm[j] = pi[r];
        }
    __syncthreads();  // the next segment takes the tables
}

// One launch: the first nseg blocks sub-order the segments in turn, the others
// put the items in longest-first order.
__global__ __launch_bounds__(kSegThreads) void k_order(
    const int2 *__restrict__ segs, const int *__restrict__ n_segs, int nseg,
    float4 *__restrict__ sorted, int *__restrict__ perm, const int4 *__restrict__ items,
    const int *__restrict__ item_cost, const int *__restrict__ n_items, int *__restrict__ lpt,
    int4 *__restrict__ out)
{
    __shared__ SegShared S;
    if ((int)blockIdx.x >= nseg) {
        lpt_scatter<kSegThreads>(blockIdx.x - nseg, items, item_cost, n_items, lpt, out);
        return;
    }
    const int n = *n_segs;
    for (int k = blockIdx.x; k < n; k += nseg)
        sub_order(S, sorted, perm, segs[k].x, segs[k].y);
}

// FP64 sum_i m_i a_i per box.  Box b is cut into R_b = min(kRedBlocks,
// ceil(n_b / 4096)) contiguous chunks, one per block; within a block each
// thread sums a fixed strided subset and the block adds them in a fixed tree
// order.  Blocks past R_b contribute exact zeros, so a box's sum depends on
// that box alone (bitwise the same alone and in a batch).
__global__ __launch_bounds__(256) void k_momentum_partial(Batch B, double *__restrict__ part)
{
    __shared__ double sh[3][256];
    const BoxDesc &d = box_at(B, blockIdx.y);
    int R = (d.n + 4095) / 4096;
    R = R < 1 ? 1 : (R > kRedBlocks ? kRedBlocks : R);
    const int chunk = (d.n + R - 1) / R;
    const int lo = blockIdx.x * chunk;
    const int hi = (int)blockIdx.x < R ? (lo + chunk < d.n ? lo + chunk : d.n) : lo;
    double s[3] = {0.0, 0.0, 0.0};
    for (int i = lo + threadIdx.x; i < hi; i += 256) {
        const double mi = (double)d.m[i];
        s[0] += mi * (double)d.ax[i];
        s[1] += mi * (double)d.ay[i];
        s[2] += mi * (double)d.az[i];
    }
    for (int k = 0; k < 3; ++k)
        sh[k][threadIdx.x] = s[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < 3; ++k)
                sh[k][threadIdx.x] += sh[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k)
            part[(blockIdx.y * kRedBlocks + blockIdx.x) * 3 + k] = sh[k][0];
}

// One block per box: the kRedBlocks partials added in a fixed tree order.
__global__ __launch_bounds__(256) void k_momentum_final(const double *__restrict__ part,
                                                        double *__restrict__ out)
{
    __shared__ double sh[3][256];
    for (int k = 0; k < 3; ++k) {
        double v = 0.0;
        for (int r = threadIdx.x; r < kRedBlocks; r += 256)
            v += part[(blockIdx.x * kRedBlocks + r) * 3 + k];
        sh[k][threadIdx.x] = v;
    }
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < 3; ++k)
                sh[k][threadIdx.x] += sh[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3)
        out[3 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

constexpr unsigned kMaskedGrid = 65536;  // workgroups of a masked pass at most (a multiple of 512)
constexpr unsigned kSubsumGrid = 1024;   // workgroups of k_subsum (256 threads each)

unsigned grid_for_items(int64_t ub)
{
    return (unsigned)((ub + 511) & ~int64_t(511));
}

int lpt_blocks(int64_t ub)
{
    return (int)((ub + kLptBlock - 1) / kLptBlock);
}

// Blocks that sub-order segments: as many as there can be (one per cell of
// more than kChunk2 targets), at most 2 per CU.
int sub_order_blocks(int64_t n)
{
    const int64_t most = n / (kChunk2 + 1);
    return (int)(most < 512 ? most : 512);
}

}  // namespace

int64_t item_bound(int64_t ntot, int64_t ctot, bool split)
{
    int64_t nonempty = ntot < ctot ? ntot : ctot;
    // at most max(ceil(n / 64), n / 16) <= n / 16 + 1 chunks per cell
    // (mesh_chunks_for), each of at most kMaxSrcSplit sub-items when chunks may be cut
    const int64_t chunks = nonempty + ntot / 16 + 1;
    return split ? kMaxSrcSplit * chunks : chunks;
}

void force_layout(Bump &b, int64_t ntot, int64_t ctot, int nb, ForceScratch &s, bool masked,
                  bool split_ok)
{
    size_t nn = (size_t)(ntot > 0 ? ntot : 1);
    const bool split = masked || split_ok;
    const int64_t ub = item_bound(ntot, ctot, split);
    bin_layout(b, ntot, ctot, nb, s.bin);
    s.offsets = b.take<int>((size_t)ctot + 1);
    s.perm = b.take<int>(nn);
    s.sorted = b.take<float4>(nn);
    s.items = b.take<int4>((size_t)ub);
    s.item_cost = b.take<int>((size_t)ub);
    s.items_lpt = b.take<int4>((size_t)ub);
    s.queue = b.take<int>(1);
    s.mom_part = b.take<double>((size_t)(nb > 0 ? nb : 1) * kRedBlocks * 3);
    s.part = split ? b.take<float>(nn * 4 * (kMaxSrcSplit - 1)) : nullptr;
    s.heads = split ? b.take<int4>((size_t)item_bound(ntot, ctot)) : nullptr;
    s.tcount = masked ? b.take<int>((size_t)ctot) : nullptr;
}

int check_force_params(sr_ctx *ctx, float r_max, float eps, const float *poly)
{
    if (!poly)
        return sr_fail(ctx, SR_EINVAL, "poly is NULL");
    for (int k = 0; k < 6; ++k)
        if (!std::isfinite(poly[k]))
            return sr_fail(ctx, SR_EINVAL, "poly[%d] is not finite", k);
    if (!(r_max > 0.f) || !std::isfinite(r_max))
        return sr_fail(ctx, SR_EINVAL, "r_max must be > 0");
    if (!(eps >= 1e-20f) || !std::isfinite(eps))
        return sr_fail(ctx, SR_EINVAL,
                       "eps must be >= 1e-20 (a pair at zero distance must stay finite)");
    return SR_OK;
}

// Validates one box against the cutoff and returns the pair loop's geometry.
int check_box_args(sr_ctx *ctx, const sr_box *box, double cell, float r_max, int xsplit, Geom *g)
{
    int rc = sr_make_geom(ctx, box, cell, g);
    if (rc)
        return rc;
    for (int d = 0; d < 3; ++d) {
        double cs = g->len[d] / g->nc[d];  // chaining cell width
        if ((double)r_max > cs)
            return sr_fail(ctx, SR_EINVAL,
                           "r_max=%g exceeds the cell width %g on axis %d: 27 cells would not "
                           "cover the cutoff",
                           (double)r_max, cs, d);
        if (g->periodic && g->nc[d] < 3)
            return sr_fail(ctx, SR_EINVAL,
                           "periodic box needs >= 3 cells per axis (axis %d has %d)", d,
                           g->nc[d]);
        if (g->periodic && !(2.0 * (double)r_max < g->len[d]))
            return sr_fail(ctx, SR_EINVAL, "periodic box needs 2 r_max < L");
    }
    return sr_make_geom(ctx, box, cell, g, xsplit);
}

ForceParams make_params(float r_max, float eps, const float *poly)
{
    // p(s) = q(s + eps): q_k = sum_{j >= k} C(j, k) c_j (-eps)^(j - k), in FP64
    static const double C[6][6] = {{1, 0, 0, 0, 0, 0},  {1, 1, 0, 0, 0, 0},
                                   {1, 2, 1, 0, 0, 0},  {1, 3, 3, 1, 0, 0},
                                   {1, 4, 6, 4, 1, 0},  {1, 5, 10, 10, 5, 1}};
    const double e = (double)eps;
    double q[6];
    for (int k = 0; k < 6; ++k) {
        double acc = 0.0;
        for (int j = k; j < 6; ++j)
            acc += C[j][k] * (double)poly[j] * std::pow(-e, j - k);
        q[k] = acc;
    }
    ForceParams fp;
    fp.eps = eps;
    fp.rcut = (float)((double)r_max * (double)r_max + e);
    fp.q0 = (float)q[0];
    fp.nq[0] = 0.f;
    for (int k = 1; k < 6; ++k)
        fp.nq[k] = (float)(-q[k]);
    return fp;
}

int lpt_sort_enqueue(sr_ctx *ctx, const int4 *items, const int *item_cost, const int *n_items,
                     int64_t bound, int *lpt, int4 *out)
{
    hipLaunchKernelGGL(k_lpt_scatter, dim3(lpt_blocks(bound)), dim3(256), 0, ctx->stream, items,
                       item_cost, n_items, lpt, out);
    return sr_check_launch(ctx, "k_lpt");
}

// Binning with the per-cell item counts, the work items, then the
// longest-first order when asked for.
static int bin_items_enqueue(sr_ctx *ctx, const Batch &B, const ForceScratch &s, int order,
                             int split)
{
    int rc;
    if ((rc = bin_enqueue(ctx, B, s.bin, s.offsets, s.perm, s.sorted, s.tcount, true)))
        return rc;
    const bool most = B.ctot >= kMostCells, many = B.ctot >= kManyCells;
    const int cells = most ? 1024 : (many ? 256 : 64), threads = many && !most ? 256 : 1024;
    const auto kern = most ? k_items<1024, 1024> : (many ? k_items<256, 256> : k_items<64, 1024>);
    hipLaunchKernelGGL(kern, dim3((B.ctot + cells - 1) / cells), dim3(threads), 0,
                       ctx->stream, B, s.offsets, s.bin.count, s.bin.work, s.tcount, s.bin.partial,
                       split, s.items, s.item_cost, s.bin.n_items, s.heads, s.bin.n_heads,
                       s.bin.lpt, reinterpret_cast<int2 *>(s.bin.tmp), s.bin.n_segs);
    if ((rc = sr_check_launch(ctx, "k_items")))
        return rc;
    const int nseg = sub_order_blocks(B.ntot);
    const int nlpt =
        order == 1 ? lpt_blocks(item_bound(B.ntot, B.ctot, s.part != nullptr)) : 0;
    if (nseg + nlpt == 0)
        return SR_OK;
    hipLaunchKernelGGL(k_order, dim3(nseg + nlpt), dim3(kSegThreads), 0, ctx->stream,
                       reinterpret_cast<const int2 *>(s.bin.tmp), s.bin.n_segs, nseg, s.sorted,
                       s.perm, s.items, s.item_cost, s.bin.n_items, s.bin.lpt, s.items_lpt);
    return sr_check_launch(ctx, "k_order");
}

int force_enqueue(sr_ctx *ctx, const Batch &B, const ForceScratch &s, const ForceParams &fp,
                  int order, int persistent, double *mom, int rec)
{
    int rc;
    sr_timing_mark(ctx, rec, 0);
    if ((rc = bin_items_enqueue(ctx, B, s, order, s.part != nullptr ? kCutSub : kCutNone)))
        return rc;
    sr_timing_mark(ctx, rec, 1);
    const int4 *items = order == 1 ? s.items_lpt : s.items;
    const int *n_items = s.bin.n_items;
    if (B.ntot > 0) {
        if (persistent) {
            int dev_cus = 256;
            (void)hipDeviceGetAttribute(&dev_cus, hipDeviceAttributeMultiprocessorCount,
                                        ctx->device);
            const int64_t ub = item_bound(B.ntot, B.ctot);
            int64_t grid = (int64_t)dev_cus * 24;
            if (grid > ub)
                grid = ub;
            if ((rc = fill_enqueue(ctx, s.queue, 0, 1)))
                return rc;
            hipLaunchKernelGGL(k_force_persistent, dim3((unsigned)grid), dim3(64), 0, ctx->stream,
                               B, items, n_items, s.sorted, s.offsets, s.perm, s.bin.mass_mixed,
                               fp, s.queue, s.part);
        } else {
            // with sub-items the item bound is loose: the grid covers the
            // chunk bound (at most kMaskedGrid workgroups in masked passes,
            // which have few items) and walks the rest
            unsigned grid = grid_for_items(item_bound(B.ntot, B.ctot));
            if (s.tcount && grid > kMaskedGrid)
                grid = kMaskedGrid;
            hipLaunchKernelGGL(k_force, dim3(grid), dim3(64), 0, ctx->stream, B, items, n_items,
                               s.sorted, s.offsets, s.perm, s.bin.mass_mixed, fp, s.part);
        }
        if ((rc = sr_check_launch(ctx, "k_force")))
            return rc;
        // the sub-items' partial sums, added in order
        if (s.part) {
            hipLaunchKernelGGL(k_subsum, dim3(kSubsumGrid), dim3(256), 0, ctx->stream, B,
                               s.heads, s.bin.n_heads, s.perm, s.part);
            if ((rc = sr_check_launch(ctx, "k_subsum")))
                return rc;
        }
    }
    sr_timing_mark(ctx, rec, 2);
    if (mom) {
        hipLaunchKernelGGL(k_momentum_partial, dim3(kRedBlocks, B.nb), dim3(256), 0, ctx->stream,
                           B, s.mom_part);
        hipLaunchKernelGGL(k_momentum_final, dim3(B.nb), dim3(256), 0, ctx->stream, s.mom_part,
                           mom);
        if ((rc = sr_check_launch(ctx, "k_momentum")))
            return rc;
    }
    return SR_OK;
}

int momentum_enqueue(sr_ctx *ctx, const Batch &B, double *part, double *mom)
{
    hipLaunchKernelGGL(k_momentum_partial, dim3(kRedBlocks, B.nb), dim3(256), 0, ctx->stream, B,
                       part);
    hipLaunchKernelGGL(k_momentum_final, dim3(B.nb), dim3(256), 0, ctx->stream, part, mom);
    return sr_check_launch(ctx, "k_momentum");
}

// Batch of one box, by value.
int single_batch(sr_ctx *ctx, const float *x, const float *y, const float *z,
                        const float *mass, int64_t n, const sr_box *box, double cell, float r_max,
                        int xsplit, float *ax, float *ay, float *az, Batch *B)
{
    if (n < 0 || n > INT_MAX)
        return sr_fail(ctx, SR_EINVAL, "n=%lld out of range", (long long)n);
    if (n > 0 && (!x || !y || !z))
        return sr_fail(ctx, SR_EINVAL, "NULL coordinate pointer");
    *B = Batch{};
    int rc = check_box_args(ctx, box, cell, r_max, xsplit, &B->one.g);
    if (rc)
        return rc;
    B->nb = 1;
    B->ntot = (int)n;
    B->ctot = B->one.g.ncell;
    B->one.n = (int)n;
    B->one.x = x;
    B->one.y = y;
    B->one.z = z;
    B->one.m = mass;
    B->one.ax = ax;
    B->one.ay = ay;
    B->one.az = az;
    return SR_OK;
}

// sr_force_split with an optional activity mask (cells without an active
// particle get no work items; their particles' outputs are left as they
// were).  Also the arena bytes such a call uses (bytes != nullptr: sizing
// only, nothing is enqueued).
int force_split_masked(sr_ctx *ctx, const int32_t *cell3, const float *ox, const float *oy,
                       const float *oz, const float *mass, int64_t n, const sr_box *box,
                       double cell, float r_max, float eps, const float poly[6], float *ax,
                       float *ay, float *az, double *momentum3, const unsigned char *active,
                       size_t *bytes)
{
    int rc = check_force_params(ctx, r_max, eps, poly);
    if (rc)
        return rc;
    if (!box || !box->periodic)
        return sr_fail(ctx, SR_EINVAL, "split coordinates need a periodic box");
    const int xs = ctx->xsplit < 3 ? ctx->xsplit : 3;
    Batch B;
    if ((rc = single_batch(ctx, ox, oy, oz, mass, n, box, cell, r_max, xs, ax, ay, az, &B)))
        return rc;
    if (n > 0 && (!cell3 || !mass || !ax || !ay || !az))
        return sr_fail(ctx, SR_EINVAL, "NULL pointer");
    for (int d = 0; d < 3; ++d)
        if (B.one.g.nc[d] / (d == 0 ? xs : 1) > kSplitMaxCells)
            return sr_fail(ctx, SR_EINVAL, "split coordinates allow at most %d cells per axis",
                           kSplitMaxCells);
    B.one.g.split = 1;
    B.one.cell3 = cell3;
    B.one.active = active;
    Bump sz{nullptr, 0, 0};
    ForceScratch s;
    const bool masked = active != nullptr;
    force_layout(sz, n, B.ctot, 1, s, masked, box_splits(n));
    if (bytes) {
        *bytes = sz.off;
        return SR_OK;
    }
    if (hipSetDevice(ctx->device) != hipSuccess)
        return sr_fail(ctx, SR_EDEVICE, "hipSetDevice failed");
    if ((rc = sr_arena_reserve(ctx, sz.off)))
        return rc;
    Bump b{ctx->arena, 0, ctx->arena_cap};
    force_layout(b, n, B.ctot, 1, s, masked, box_splits(n));
    const ForceParams fp = make_params(r_max, eps, poly);
    const int rec = sr_timing_begin(ctx);
    return force_enqueue(ctx, B, s, fp, ctx->order, ctx->persistent, momentum3, rec);
}

extern "C" int sr_force_split(sr_ctx *ctx, const int32_t *cell3, const float *ox, const float *oy,
                              const float *oz, const float *mass, int64_t n, const sr_box *box,
                              double cell, float r_max, float eps, const float poly[6], float *ax,
                              float *ay, float *az, double *momentum3)
{
    if (!ctx)
        return SR_EINVAL;
    ctx->err.clear();
    return force_split_masked(ctx, cell3, ox, oy, oz, mass, n, box, cell, r_max, eps, poly, ax,
                              ay, az, momentum3, nullptr, nullptr);
}

extern "C" int sr_scratch_bytes(const sr_box *box, double cell, int64_t n, int with_force,
                                size_t *bytes)
{
    if (!bytes || n < 0 || n > INT_MAX || with_force < 0 || with_force > 2)
        return SR_EINVAL;
    Geom g;
    // with_force: the largest x split any context may use
    if (sr_make_geom(nullptr, box, cell, &g, with_force ? kMaxXsplit : 1))
        return SR_EINVAL;
    Bump sz{nullptr, 0, 0};
    if (with_force) {
        ForceScratch s;
        force_layout(sz, n, g.ncell, 1, s, with_force == 2, box_splits(n));
        if (with_force == 2) {
            // the multilevel step's levels, activity mask and cell counts
            // (sr_ksk_step lays them out after the force pass)
            Geom g1;
            if (sr_make_geom(nullptr, box, cell, &g1, 1))
                return SR_EINVAL;
            sz.take<unsigned char>((size_t)n);
            sz.take<unsigned char>((size_t)n);
            sz.take<int>((size_t)g1.ncell);
        }
    } else {
        BinScratch s;
        bin_layout(sz, n, g.ncell, 1, s);
    }
    *bytes = sz.off;
    return SR_OK;
}

extern "C" int sr_force(sr_ctx *ctx, const float *x, const float *y, const float *z,
                        const float *mass, int64_t n, const sr_box *box, double cell, float r_max,
                        float eps, const float poly[6], float *ax, float *ay, float *az,
                        double *momentum3)
{
    if (!ctx)
        return SR_EINVAL;
    ctx->err.clear();
    int rc = check_force_params(ctx, r_max, eps, poly);
    if (rc)
        return rc;
    Batch B;
    if ((rc = single_batch(ctx, x, y, z, mass, n, box, cell, r_max, ctx->xsplit, ax, ay, az, &B)))
        return rc;
    if (n > 0 && (!mass || !ax || !ay || !az))
        return sr_fail(ctx, SR_EINVAL, "NULL mass or output pointer");
    if (hipSetDevice(ctx->device) != hipSuccess)
        return sr_fail(ctx, SR_EDEVICE, "hipSetDevice failed");
    Bump sz{nullptr, 0, 0};
    ForceScratch s;
    force_layout(sz, n, B.ctot, 1, s, false, box_splits(n));
    if ((rc = sr_arena_reserve(ctx, sz.off)))
        return rc;
    Bump b{ctx->arena, 0, ctx->arena_cap};
    force_layout(b, n, B.ctot, 1, s, false, box_splits(n));
    const ForceParams fp = make_params(r_max, eps, poly);
    const int rec = sr_timing_begin(ctx);
    return force_enqueue(ctx, B, s, fp, ctx->order, ctx->persistent, momentum3, rec);
}

extern "C" int sr_pair_stats(sr_ctx *ctx, const float *x, const float *y, const float *z,
                             int64_t n, const sr_box *box, double cell, float r_max,
                             int32_t *per_target, int64_t *useful, int64_t *candidates)
{
    if (!ctx)
        return SR_EINVAL;
    ctx->err.clear();
    if (!useful || !candidates)
        return sr_fail(ctx, SR_EINVAL, "NULL result pointer");
    static const float zero_poly[6] = {0, 0, 0, 0, 0, 0};
    Batch B;
    // masses are not needed; the gather reads x in their place
    int rc = single_batch(ctx, x, y, z, x, n, box, cell, r_max, ctx->xsplit, nullptr, nullptr,
                          nullptr, &B);
    if (rc)
        return rc;
    if (hipSetDevice(ctx->device) != hipSuccess)
        return sr_fail(ctx, SR_EDEVICE, "hipSetDevice failed");
    Bump sz{nullptr, 0, 0};
    ForceScratch s;
    force_layout(sz, n, B.ctot, 1, s, false, false);  // no sub-items
    if ((rc = sr_arena_reserve(ctx, sz.off)))
        return rc;
    Bump b{ctx->arena, 0, ctx->arena_cap};
    force_layout(b, n, B.ctot, 1, s, false, false);
    if ((rc = bin_items_enqueue(ctx, B, s, 0, kCutChunks)))
        return rc;
    // eps = 0 so that se = s and the test is s < r_max^2
    ForceParams fp = make_params(r_max, 0.0f, zero_poly);
    unsigned long long *st = (unsigned long long *)ctx->stats;
    if ((rc = fill_enqueue(ctx, (int *)st, 0, 4)))
        return rc;
    if (n > 0) {
        hipLaunchKernelGGL(k_pair_stats, dim3((unsigned)item_bound(n, B.ctot)), dim3(64), 0,
                           ctx->stream, B, s.items, s.bin.n_items, s.sorted, s.offsets,
                           s.perm, fp, per_target, st);
        if ((rc = sr_check_launch(ctx, "k_pair_stats")))
            return rc;
    }
    unsigned long long h[2] = {0, 0};
    if (hipMemcpyAsync(h, st, sizeof h, hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess)
        return sr_fail(ctx, SR_EDEVICE, "reading pair statistics failed");
    *useful = (int64_t)h[0];
    *candidates = (int64_t)h[1];
    return SR_OK;
}
