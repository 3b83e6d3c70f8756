// The pair loop of a chaining-mesh work item (sr_force.hip): one wavefront, at
// most 64 vector registers and 5 KiB of LDS, so that 8 wavefronts share a SIMD.
//
// The stencil's sources pass by in windows of 64, one per lane: each is tested
// against the box of the item's targets (source_kept), and the kept ones are
// appended to a tile in LDS.  When the tile cannot take another window, the S
// lane groups take the whole quanta (2 S sources) it holds in turn, group q
// the sources q, q + S, q + 2 S, ... (consecutive entries at a time, so that the
// groups' reads meet no common LDS bank: with contiguous slices two in five
// LDS cycles of the 128^3 lattice pass were conflicts), and what is left moves
// to its front.  So no source is padding but at the item's end, and only one
// window waits in registers (5 of them) instead of a tile of 256 (16).
//
// What bounds it: FP32 VALU issue.  FMA, multiply, add and subtract issue two
// at a time from different wavefronts (2.2 cycles each per SIMD), compare,
// select, min and max do not (4.1), v_rsq_f32 takes 8.  The more wavefronts
// share a SIMD the more often two are ready: a register-only probe of the loop
// on all 256 CUs reaches 2.41e12 pairs/s at 5 wavefronts per SIMD, 2.83e12 at
// 8, and 2.88e12 at 8 with the cutoff as EXEC mask (pair_masked).
#pragma once

#include "sr_pair.h"

namespace {

constexpr int kSumTile = 64;         // a lane's partial sums close at this many sources,
constexpr int kSumTileLong = 512;    // ... and at this many in items of
constexpr int kLongItem = 1 << 14;   // more stencil sources than this

// The non-empty source pieces of an item's cell: piece k holds the stencil's
// sources [beg[k], beg[k + 1]), source g of it sits in sorted slot g +
// rec[k].off, and its shift is added to its coordinates.  beg past the pieces is
// the number of all sources.
struct PieceRec {
    int off;
    float x, y, z;
};
struct Pieces {
    PieceRec rec[kMaxPieces];
    int beg[kMaxPieces + 2];
};

// Whether the tile of S lane groups holds every entry that item_sources writes
// or reads: before a window it keeps at most stage_hold(S) sources or what a pass
// leaves (less than a quantum), the window adds at most kWindow, and the last
// pass fills its last quantum up.
constexpr bool stage_fits(int S)
{
    const int q = 2 * S;
    const int kept = stage_hold(S) > q - 1 ? stage_hold(S) : q - 1;
    return (kept + kWindow + q - 1) / q * q <= kStage;
}

constexpr bool stages_fit()
{
    for (int S = 1; S <= kMaxSplit; ++S)
        if (!stage_fits(S))
            return false;
    return true;
}
static_assert(stages_fit(), "a window and the padding of a quantum fit in the tile");

// acc: each lane's sums so far, added to once per partial sum, so that they
// hold no registers through the pair loop.
struct ItemShared {
    float4 tile[kStage];
    Pieces st;
    float acc[6][64];
};

// One or two targets of a lane and their partial sums.
struct LaneTargets {
    float xi, yi, zi, xj, yj, zj;
    float tx, ty, tz, ux, uy, uz;
};

// pair_one (sr_pair.h) with the cutoff as EXEC mask on the accumulation: the
// same products and sums for a pair within the cutoff, and nothing added for
// one beyond it, where pair_one adds 0.  One v_cmpx takes the place of v_cmp
// and v_cndmask.  All 64 lanes are active before and after (64-thread
// workgroups, wave-uniform control flow): EXEC is restored to all ones.
template <bool kUniformMass>
__device__ __forceinline__ void pair_masked(const float4 &s, float xi, float yi, float zi,
                                            const ForceParams &w, float rcut, float &tx, float &ty,
                                            float &tz)
{
    const float dx = s.x - xi;
    const float dy = s.y - yi;
    const float dz = s.z - zi;
    const float se = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, w.eps)));
    const float rs = __builtin_amdgcn_rsqf(se);
    const float rs2 = rs * rs;
    const float tt = fmaf(rs2, rs, -w.q0);
    float h = fmaf(w.nq[5], se, w.nq[4]);
    h = fmaf(h, se, w.nq[3]);
    h = fmaf(h, se, w.nq[2]);
    h = fmaf(h, se, w.nq[1]);
    float f = fmaf(h, se, tt);
    if (!kUniformMass)
        f *= s.w;
    asm("v_cmpx_gt_f32 vcc, %6, %7\n\t"
        "v_fmac_f32 %0, %3, %4\n\t"
        "v_fmac_f32 %1, %3, %5\n\t"
        "v_fmac_f32 %2, %3, %8\n\t"
        "s_mov_b64 exec, -1"
        : "+v"(tx), "+v"(ty), "+v"(tz)
        : "v"(f), "v"(dx), "v"(dy), "s"(rcut), "v"(se), "v"(dz)
        : "vcc");
}

// A lane's targets with 2 n sources, src[0], src[S], src[2 S], ...  (n > 0),
// each target summed in source order.  The polynomial's constants sit in vector
// registers: of two instructions issued together one may read a scalar one.
template <bool kTwo, bool kUniformMass>
__device__ __forceinline__ void pair_run(const float4 *src, int S, int n, const ForceParams &fp,
                                         LaneTargets &L)
{
    ForceParams w = fp;
    asm volatile("" : "+v"(w.eps), "+v"(w.q0), "+v"(w.nq[1]), "+v"(w.nq[2]), "+v"(w.nq[3]),
                      "+v"(w.nq[4]), "+v"(w.nq[5]));
    do {
        const float4 a = src[0], b = src[S];
        src += 2 * S;
        pair_masked<kUniformMass>(a, L.xi, L.yi, L.zi, w, fp.rcut, L.tx, L.ty, L.tz);
        if (kTwo)
            pair_masked<kUniformMass>(a, L.xj, L.yj, L.zj, w, fp.rcut, L.ux, L.uy, L.uz);
        pair_masked<kUniformMass>(b, L.xi, L.yi, L.zi, w, fp.rcut, L.tx, L.ty, L.tz);
        if (kTwo)
            pair_masked<kUniformMass>(b, L.xj, L.yj, L.zj, w, fp.rcut, L.ux, L.uy, L.uz);
    } while (--n > 0);
}

// Adds a lane's partial sums to its sums in LDS and clears them.
__device__ __forceinline__ void flush_sums(ItemShared &sh, int lane, LaneTargets &L)
{
    sh.acc[0][lane] += L.tx;
    sh.acc[1][lane] += L.ty;
    sh.acc[2][lane] += L.tz;
    sh.acc[3][lane] += L.ux;
    sh.acc[4][lane] += L.uy;
    sh.acc[5][lane] += L.uz;
    L.tx = L.ty = L.tz = L.ux = L.uy = L.uz = 0.f;
}

// Builds the pieces of target cell (cx, cy, cz) (all lanes call); returns whether
// any is shifted.
__device__ __forceinline__ bool build_pieces(Pieces &st, const int *__restrict__ offsets,
                                             const Geom &g, int cx, int cy, int cz,
                                             const float F[3], int lane)
{
    int len, src, total;
    float sx, sy, sz;
    stencil_piece(offsets, g, cx, cy, cz, F, lane, src, len, sx, sy, sz);
    const int beg = wave_exclusive_scan(len, lane, &total);
    const unsigned long long some = __ballot(len > 0);
    const int k = (int)__builtin_amdgcn_mbcnt_hi(
        (unsigned)(some >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)some, 0u));
    if (len > 0) {
        st.rec[k] = PieceRec{src - beg, sx, sy, sz};
        st.beg[k] = beg;
    }
    const int np = __popcll(some);
    for (int e = np + lane; e < kMaxPieces + 2; e += 64)
        st.beg[e] = total;
    return __any(len > 0 && (sx != 0.f || sy != 0.f || sz != 0.f));
}

// Source gi = g + lane of the stencil, without its shift; far, massless padding
// from `end` on.  p is the piece of the lane's last source and moves on to
// this one's: two pieces at a time, further where pieces are short.
__device__ __forceinline__ float4 load_window(const Pieces &st, const float4 *__restrict__ sorted,
                                              int g, int end, int lane, int &p)
{
    float4 v = make_float4(kFar, kFar, kFar, 0.f);
    const int gi = g + lane;
    if (gi < end) {
        for (;;) {
            const int b1 = st.beg[p + 1], b2 = st.beg[p + 2];
            p += (gi >= b1 ? 1 : 0) + (gi >= b2 ? 1 : 0);
            if (gi < b2)
                break;
        }
        v = sorted[gi + st.rec[p].off];
    }
    return v;
}

// Sources [g0, g1) of the item's stencil.  part: the lane's group, below S.
template <bool kTwo, bool kUniformMass>
__device__ __forceinline__ void item_sources(int S, int part, int g0, int g1, bool shifted,
                                             const float4 *__restrict__ sorted,
                                             const ForceParams &fp, int lane, ItemShared &sh,
                                             LaneTargets &L)
{
    const TargetBox tb = target_box(L.xi, L.yi, L.zi, L.xj, L.yj, L.zj);
    const int quantum = 2 * S, qrecip = kItemTab.srecip[S], hold = kItemTab.hold[S];
    const int close = g1 - g0 > kLongItem ? kSumTileLong : kSumTile;
    int fill = 0, summed = 0, p = 0;
    float4 v = load_window(sh.st, sorted, g0, g1, lane, p);
    for (int g = g0; g < g1; g += kWindow) {
        if (shifted) {
            const PieceRec r = sh.st.rec[p];
            v.x += r.x;
            v.y += r.y;
            v.z += r.z;
        }
        const bool kept = source_kept(v, tb, fp);
        const unsigned long long mask = __ballot(kept);
        if (kept)
            sh.tile[fill + (int)__builtin_amdgcn_mbcnt_hi(
                               (unsigned)(mask >> 32),
                               __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u))] = v;
        fill += __popcll(mask);
        const bool last = g + kWindow >= g1;
        if (!last) {
            v = load_window(sh.st, sorted, g + kWindow, g1, lane, p);
            if (fill <= hold)
                continue;
        }
        // whole quanta: at the end the last one is filled up with far, massless
        // sources, fewer than a quantum, within the tile (stage_fits)
        int n = (fill * qrecip) >> 16;
        if (last && n * quantum < fill) {
            ++n;
            if (fill + lane < n * quantum)
                sh.tile[fill + lane] = make_float4(kFar, kFar, kFar, 0.f);
        }
        if (n == 0)
            continue;
        __syncthreads();
        pair_run<kTwo, kUniformMass>(sh.tile + part, S, n, fp, L);
        const int done = n * quantum;
        fill -= done;
        summed += 2 * n;
        if (fill > 0) {
            const float4 r = sh.tile[done + (lane < fill ? lane : 0)];
            __syncthreads();
            if (lane < fill)
                sh.tile[lane] = r;
        }
        // A sum of N sources in runs of k rounds over k additions and over N / k:
        // k stays near the root of N.  Error against 64 bits: a ragged halo box
        // (a few thousand sources per sub-item) 9.1e-8 with runs of 64, 1.3e-7
        // with 256; the 256^3 share (1e4 to 1e6 per item) 3.8e-7 with 64, 2.4e-7
        // with 256, 2.0e-7 with 512.
        if (summed >= close) {
            summed = 0;
            flush_sums(sh, lane, L);
        }
    }
    flush_sums(sh, lane, L);
}

// The targets of lane `lane` of an item of nt targets: group part of S, t and
// the second one t2 when it holds two (lane t of a group holds targets t and
// t + ln, ln lanes per group).  Lanes past the groups repeat the first ones.
struct ItemLane {
    int ln, part, t, t2;
    bool has, has2;
};

__device__ __forceinline__ ItemLane item_lane(bool two, int nt, int S, int lane)
{
    ItemLane T;
    T.ln = two ? (nt + 1) >> 1 : nt;
    T.part = lane_group(lane, T.ln);
    T.t = lane - T.part * T.ln;
    T.has = T.part < S;
    T.part = T.has ? T.part : 0;
    T.has2 = two && T.has && T.t + T.ln < nt;
    T.t2 = T.has2 ? T.t + T.ln : T.t;
    return T;
}

// Where sub-item sk of a chunk leaves component c of the sum of the target in a
// sorted slot, among the partial sums of all sub-items (s.part).
__device__ __forceinline__ size_t subsum_at(int sk, int c, int ntot, int slot)
{
    return (size_t)(3 * sk + c) * ntot + slot;
}
static_assert(3 * kMaxSrcSplit <= 4 * (kMaxSrcSplit - 1), "s.part holds every sub-item's sums");

// Stores the acceleration of the target in a sorted slot: a whole item writes it
// out, a sub-item leaves its partial sums for k_subsum, in slot order (with
// sub-item 0's sums written out and read back scattered, and 16 bytes per sum, a
// pass over 32 halo boxes of 16^3..96^3 particles took 11204 us here and 312 in
// k_subsum instead of 10952 and 236).
__device__ __forceinline__ void write_target(const BoxDesc &d, const int *__restrict__ perm,
                                             float *__restrict__ subsums, int ntot, bool cut,
                                             int sub, int slot, bool passive, float ax, float ay,
                                             float az)
{
    if (passive)
        ax = ay = az = 0.f;
    if (cut) {
        subsums[subsum_at(sub, 0, ntot, slot)] = ax;
        subsums[subsum_at(sub, 1, ntot, slot)] = ay;
        subsums[subsum_at(sub, 2, ntot, slot)] = az;
    } else {
        const int orig = perm[slot] - d.pbase;
        d.ax[orig] = ax;
        d.ay[orig] = ay;
        d.az[orig] = az;
    }
}

// The pair loop of one work item by one wavefront.
__device__ __forceinline__ void process_item(const Batch &B, const int4 item,
                                             const float4 *__restrict__ sorted,
                                             const int *__restrict__ offsets,
                                             const int *__restrict__ perm,
                                             const int *__restrict__ mass_mixed,
                                             const ForceParams &fp, ItemShared &sh, int lane,
                                             float *__restrict__ subsums)
{
    const int kb = item.y, nt = item.z, S = item_split(item), box = item_box(item);
    const BoxDesc &d = box_at(B, box);
    const Geom &g = d.g;
    const bool two = item_two(item), uniform = mass_mixed[box] == 0;
    ItemLane T = item_lane(two, nt, S, lane);
    float4 pt = sorted[kb + T.t], pt2 = sorted[kb + T.t2];
    const bool work = __any((T.has && !is_passive(pt, g)) || (T.has2 && !is_passive(pt2, g)));
#pragma unroll
    for (int k = 0; k < 6; ++k)
        sh.acc[k][lane] = 0.f;
    if (work) {
        int cx, cy, cz;
        decode_cell(item.x - d.cbase, g, cx, cy, cz);
        const int cc[3] = {cx, cy, cz};
        float F[3];
        frame_shift(g, cc, F);
        const bool shifted =
            build_pieces(sh.st, offsets + d.cbase, g, cx, cy, cz, F, lane);
        __syncthreads();
        // a sub-item takes its part [sk T / ns, (sk + 1) T / ns) of the T sources
        const int ns = item_nsub(item), sk = item_sub(item);
        const int all = __builtin_amdgcn_readfirstlane(sh.st.beg[kMaxPieces]);
        int g0 = 0, g1 = all;
        if (ns > 1) {
            g0 = __builtin_amdgcn_readfirstlane((int)((long long)sk * all / ns));
            g1 = __builtin_amdgcn_readfirstlane((int)((long long)(sk + 1) * all / ns));
        }
        LaneTargets L = {pt.x + F[0], pt.y + F[1], pt.z + F[2], pt2.x + F[0], pt2.y + F[1],
                         pt2.z + F[2], 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (two) {
            if (uniform)
                item_sources<true, true>(S, T.part, g0, g1, shifted, sorted, fp, lane, sh, L);
            else
                item_sources<true, false>(S, T.part, g0, g1, shifted, sorted, fp, lane, sh,
                                          L);
        } else {
            if (uniform)
                item_sources<false, true>(S, T.part, g0, g1, shifted, sorted, fp, lane, sh,
                                          L);
            else
                item_sources<false, false>(S, T.part, g0, g1, shifted, sorted, fp, lane, sh,
                                           L);
        }
        // found and read again instead of held through the pair loop
        asm volatile("" : "+v"(lane));
        T = item_lane(two, nt, S, lane);
        pt = sorted[kb + T.t];
        pt2 = sorted[kb + T.t2];
        __syncthreads();
    }
    // the S group sums of each target in group order, by the first group
    if (lane < T.ln) {
        float a[6];
#pragma unroll
        for (int k = 0; k < 6; ++k)
            a[k] = sh.acc[k][lane];
        for (int q = 1; q < S; ++q)
#pragma unroll
            for (int k = 0; k < 6; ++k)
                a[k] += sh.acc[k][lane + q * T.ln];
        const float m = uniform ? pt.w : 1.f, m2 = uniform ? pt2.w : 1.f;
        const bool cut = item_nsub(item) > 1;
        write_target(d, perm, subsums, B.ntot, cut, item_sub(item), kb + T.t, is_passive(pt, g),
                     a[0] * m, a[1] * m, a[2] * m);
        if (T.has2)
            write_target(d, perm, subsums, B.ntot, cut, item_sub(item), kb + T.t2,
                         is_passive(pt2, g), a[3] * m2, a[4] * m2, a[5] * m2);
    }
    __syncthreads();  // the next item replaces the pieces and the sums
}

}  // namespace
