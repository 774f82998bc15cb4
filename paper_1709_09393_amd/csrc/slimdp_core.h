// Core selection (gfx950): per segment the need parameters first by (score bits descending, index ascending).
// Included only by slimdp.hip, after slimdp_kernels.h.
//
// A radix descent over the 32 score bits in three levels (13 + 12 + 7) in four launches:
//   k_core_build   picks the level-0 bin, sorts every parameter against it (certain bitmap, candidate bitmap, candidate
//                  keys per sub-tile) and counts the candidates' level-1 digits; nothing left to sort where the
//                  scoring pass has already done it against the right bin
//   k_core_hist2   picks the level-1 bin, counts the level-2 digits of the candidates in it
//   k_core_count   picks the level-2 bin: threshold key and tie quota; per tile the certain ones and the ties
//   k_core_emit    the ascending index list, its tile offsets, the public bitmap; clears the histograms for the next use
// A threshold step is cheap (16 KB of histogram from the L2) and its result is needed by every block of the next
// pass, so every block takes it by itself; a segment's core size is known, so one prefix of (certain, ties) inside the
// segment gives every offset; the last pass clears what the first ones count into.  As kernels of their own (a clearing,
// a state, a threshold per level, two scans) these steps made ten to thirteen launches of 2 to 8 us each.  Measured,
// ten launches against four: 200,003 parameters without a context (one launch more: the histogram) 53.8 -> 30.7 us, a
// whole iteration of 10^6 parameters 207 -> 173 us, of 7*10^6 in 57 segments 367 -> 333 us, of 138*10^6 2.39 -> 2.31 ms.
#pragma once
#include "slimdp_kernels.h"
#include "slimdp_split.h"

namespace slimdp {

// What the host knows about a segment: its core size and that of all segments before it.
struct CorePlan { uint32_t need, base; };
// What the passes find out about a segment.  A field is written by one kernel (every block that meets the segment
// writes the same value) and read by later ones.
struct CoreState {
    uint32_t none;                 // nothing is selected here
    uint32_t skip;                 // the scoring pass sorted the whole tiles against the right bin
    uint32_t prefix0, need0;       // level-0 bin, keys still to be taken from it
    uint32_t prefix1, need1;       // the same after level 1 (25 bits)
    uint32_t tau, quota;           // threshold key; how many keys equal to it are taken, lowest index first
};
struct CoreArgs {
    const uint32_t *tile_start, *tile_seg, *seg_first_tile;      // not read for a flat model
    uint64_t n;
    uint32_t T, n_seg, groups;
    uint32_t k_flat;               // flat model: the core size (plan is not read)
    const CorePlan* plan;
    uint32_t* hist;                // [n_seg * H_STRIDE]
    CoreState* state;
    uint32_t *gt_bits, *cand_bits, *cand_keys, *cnt_gt, *cnt_cand;
    uint2* tile_pre;               // [T] (certain, ties) of the tiles before this one in its group and segment
    uint2* group_tail;             // [groups] the same summed over the group's last segment
    uint32_t* flags;
};

__device__ __forceinline__ uint32_t seg_of_tile(const CoreArgs& a, uint32_t t) { return a.n_seg == 1 ? 0u : a.tile_seg[t]; }
__device__ __forceinline__ uint32_t seg_end_tile(const CoreArgs& a, uint32_t seg) { return a.n_seg == 1 ? a.T : a.seg_first_tile[seg + 1]; }
__device__ __forceinline__ uint32_t seg_begin_tile(const CoreArgs& a, uint32_t seg) { return a.n_seg == 1 ? 0u : a.seg_first_tile[seg]; }
__device__ __forceinline__ CorePlan plan_of(const CoreArgs& a, uint32_t seg)
{
    if (a.n_seg == 1) return CorePlan{a.k_flat, 0u};
    return a.plan[seg];
}

// The bin in which the need-th key from the top falls (need >= 1), by the whole block.  sh: 4 words, wtot: 4 words.
// A thread keeps the sums of four bins each and reads the four that matter again: with every bin of its 32 in a register
// k_core_build took 207 registers, two blocks to a compute unit, instead of 125 and four (score and selection of 138*10^6
// parameters without a prediction 663 -> 598 us, selection of any array 414 -> 342 us; 7*10^6 in 57 segments 85.6 -> 77.7 us).
struct BinPick { uint32_t bin, left, total; };
template <int NB>
__device__ __forceinline__ BinPick pick_bin(const uint32_t* __restrict__ hp, uint32_t need, uint32_t* wtot, uint32_t* sh)
{
    constexpr int PER = NB >= BLOCK ? NB / BLOCK : 1, VEC = PER >= 4 ? PER / 4 : 1;
    uint32_t c[VEC], sum = 0;
    const uint32_t low = NB - (threadIdx.x + 1u) * PER;       // this thread's bins low .. low + PER - 1; thread 0 has the largest
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        if constexpr (PER >= 4) {
            const uint4 q = *reinterpret_cast<const uint4*>(hp + low + 4 * v);
            c[v] = (q.x + q.y) + (q.z + q.w);
        } else {
            c[v] = threadIdx.x < (uint32_t)NB ? hp[low] : 0u;
        }
        sum += c[v];
    }
    uint32_t total;
    const uint32_t excl = block_excl_scan<4>(sum, wtot, total);
    if (excl < need && need <= excl + sum) {
        // the four bins (one, with few bins a thread) in which it falls, then the bin among them
        uint32_t run = excl, at = 0, before = 0;
#pragma unroll
        for (int v = VEC - 1; v >= 0; --v) {
            if (run < need && need <= run + c[v]) { at = (uint32_t)v; before = run; }
            run += c[v];
        }
        uint32_t bin = low, left = need - before;
        if constexpr (PER >= 4) {
            const uint4 q = *reinterpret_cast<const uint4*>(hp + low + 4u * at);
            bin = low + 4u * at + 3u;
            if (left > q.w) { left -= q.w; --bin; if (left > q.z) { left -= q.z; --bin; if (left > q.y) { left -= q.y; --bin; } } }
        }
        sh[0] = bin; sh[1] = left;
    }
    __syncthreads();
    const BinPick r{sh[0], sh[1], total};
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------------------------------
// One pass over the score: parameters whose level-0 digit is above the threshold bin are
// certainly in the core (gt bitmap), those in the bin are candidates (bitmap + keys compacted
// per sub-tile) and feed the level-1 histogram.  Bound by reading the score (4 bytes per parameter).
// Every wave owns sub-tile `wid` of each of the block's tiles and needs no block barrier:
// round `it` covers parameters [256*it, 256*it+256) of the sub-tile in index order (lane L
// owns 4L..4L+3), the eight bitmap words of a round are OR-reductions over groups of
// eight lanes, a candidate's place in the key list comes from wave ballots.
// ---------------------------------------------------------------------------------------
// The 1024 scores of sub-tile `wid` of a tile as keys: lane L holds parameters 4L..4L+3 of each round of 256.
__device__ __forceinline__ void core_load_keys(const float* __restrict__ S, uint32_t start, uint32_t len, uint32_t wid,
                                               uint32_t lane, uint32_t key[4][4])
{
    const uint32_t off = wid * SUB;
    const uint32_t sub_len = (len > off) ? ((len - off < SUB) ? len - off : SUB) : 0u;
    const float* src = S + (size_t)start + off;
    if (sub_len == SUB) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const uint4 v = ld4u<NT_BUILD>(reinterpret_cast<const uint32_t*>(src + it * 256 + lane * 4));
            key[it][0] = v.x; key[it][1] = v.y; key[it][2] = v.z; key[it][3] = v.w;
        }
    } else {
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const uint32_t e = (uint32_t)it * 256u + lane * 4u + cc;
                key[it][cc] = (e < sub_len) ? __float_as_uint(src[e]) : 0u;
            }
    }
}

// One sub-tile's keys against the level-0 threshold bin b1: bitmaps, candidate keys, counts, level-1 histogram (LDS).
__device__ __forceinline__ void core_classify(const uint32_t key[4][4], uint32_t t, uint32_t start, uint32_t len, uint32_t wid,
                                              uint32_t lane, uint32_t b1, uint32_t* __restrict__ h, const CoreArgs& a)
{
    const uint32_t off = wid * SUB;
    const uint32_t sub_len = (len > off) ? ((len - off < SUB) ? len - off : SUB) : 0u;
    uint32_t* gwords = a.gt_bits + (size_t)t * TILE_WORDS + wid * SUB_WORDS;
    uint32_t* cwords = a.cand_bits + (size_t)t * TILE_WORDS + wid * SUB_WORDS;
    uint32_t* ckeys = a.cand_keys + (size_t)start + off;
    uint32_t run = 0, ngt = 0;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        uint32_t fg = 0, fc = 0;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            const uint32_t e = (uint32_t)it * 256u + lane * 4u + cc;
            if (e < sub_len) {
                const uint32_t d = key[it][cc] >> CORE_SHIFT0;
                if (d > b1) fg |= 1u << cc;
                else if (d == b1) fc |= 1u << cc;
            }
        }
        const uint32_t vg = or_reduce8(fg << (4u * (lane & 7u))), vc = or_reduce8(fc << (4u * (lane & 7u)));
        if ((lane & 7u) == 0) { gwords[it * 8 + (lane >> 3)] = vg; cwords[it * 8 + (lane >> 3)] = vc; }
        ngt += __popc(fg);
        uint32_t below = 0, total = 0;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            const unsigned long long bal = __ballot((fc >> cc) & 1u);
            below += __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            total += (uint32_t)__popcll(bal);
        }
        if (fc) {
            uint32_t pos = run + below;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
                if ((fc >> cc) & 1u) {
                    ckeys[pos++] = key[it][cc];
                    atomicAdd(&h[(key[it][cc] >> CORE_SHIFT1) & (CORE_NB1 - 1u)], 1u);
                }
        }
        run += total;
    }
    ngt = wave_sum(ngt);
    if (lane == 0) { a.cnt_cand[(size_t)t * SUBS + wid] = run; a.cnt_gt[(size_t)t * SUBS + wid] = ngt; }
}

// Level-0 histogram of a score array that did not come from a scoring pass (any bit pattern).  Flat model: the array
// in one run of 16-byte loads; otherwise contiguous tile ranges.  grid: any (segmented: at most T blocks).
__global__ __launch_bounds__(BLOCK) void k_core_hist0(const float* __restrict__ S, CoreArgs a)
{
    __shared__ uint32_t h[CORE_NB0];
    for (uint32_t b = threadIdx.x; b < CORE_NB0; b += BLOCK) h[b] = 0;
    __syncthreads();
    const uint32_t* keys = reinterpret_cast<const uint32_t*>(S);
    if (a.n_seg == 1) {
        const uint64_t n4 = a.n / 4, stride = (uint64_t)gridDim.x * BLOCK;
        for (uint64_t x = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; x < n4; x += stride) {
            const uint4 v = ld4u<0>(keys + 4 * x);
            atomicAdd(&h[v.x >> CORE_SHIFT0], 1u); atomicAdd(&h[v.y >> CORE_SHIFT0], 1u);
            atomicAdd(&h[v.z >> CORE_SHIFT0], 1u); atomicAdd(&h[v.w >> CORE_SHIFT0], 1u);
        }
        for (uint64_t i = 4 * n4 + (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < a.n; i += stride) atomicAdd(&h[keys[i] >> CORE_SHIFT0], 1u);
        __syncthreads();
        flush_hist(h, CORE_NB0, a.hist + H_L0);
        return;
    }
    uint32_t t = (uint32_t)((uint64_t)a.T * blockIdx.x / gridDim.x);
    const uint32_t t1 = (uint32_t)((uint64_t)a.T * (blockIdx.x + 1) / gridDim.x);
    while (t < t1) {
        const uint32_t seg = a.tile_seg[t], seg_t1 = min(t1, a.seg_first_tile[seg + 1]);
        const uint32_t i1 = a.tile_start[seg_t1];
        for (uint32_t i = a.tile_start[t] + threadIdx.x; i < i1; i += BLOCK) atomicAdd(&h[keys[i] >> CORE_SHIFT0], 1u);
        __syncthreads();
        flush_hist(h, CORE_NB0, a.hist + (size_t)seg * H_STRIDE + H_L0);
        __syncthreads();
        t = seg_t1;
    }
}

// The segments' core sizes, written once and kept while they stay the same.
constexpr int PLAN_CHUNK = 256;
struct CorePlanChunk { CorePlan s[PLAN_CHUNK]; };
__global__ __launch_bounds__(PLAN_CHUNK) void k_core_plan(CorePlan* __restrict__ plan, CorePlanChunk chunk, uint32_t seg0, uint32_t count)
{
    if (threadIdx.x < count) plan[seg0 + threadIdx.x] = chunk.s[threadIdx.x];
}

// used (flat model): the level-0 bin against which the scoring pass has already sorted every whole tile, if check is
// set.  The pass counted the level-1 digits of its candidates in region H_L1; this kernel's own counts go there if
// that bin was the right one (only the ragged tile is missing then) and to region H_L1B otherwise.
// half: the histogram comes from a scoring pass, whose significances have a clear sign bit.
// zero_bits: public bitmap of a model whose tiles may start inside a word: the words that two tiles share are
// cleared here and filled with atomics by k_core_emit.
__global__ __launch_bounds__(BLOCK) void k_core_build(const float* __restrict__ S, CoreArgs a, const uint32_t* __restrict__ used,
                                                      int check, int half, int strided, uint32_t* __restrict__ zero_bits)
{
    __shared__ uint32_t h[CORE_NB1];
    __shared__ uint32_t wtot[4], sh[4];
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    if (zero_bits) {
        for (uint32_t t = blockIdx.x * BLOCK + threadIdx.x; t <= a.T; t += gridDim.x * BLOCK) {
            const uint32_t i = (t < a.T) ? a.tile_start[t] : (uint32_t)(a.n - 1u);
            if (t == a.T || (i & 31u)) zero_bits[i >> 5] = 0;
        }
    }
    // a contiguous range of tiles, or (flat model) every gridDim.x-th tile: see k_score
    uint32_t t = strided ? blockIdx.x : (uint32_t)((uint64_t)a.T * blockIdx.x / gridDim.x);
    const uint32_t t1 = strided ? a.T : (uint32_t)((uint64_t)a.T * (blockIdx.x + 1) / gridDim.x);
    const uint32_t tstep = strided ? gridDim.x : 1u;
    if (t >= t1) return;
    for (uint32_t b = threadIdx.x; b < CORE_NB1; b += BLOCK) h[b] = 0;
    // one segment of the block's range after the other (flat model: once)
    while (t < t1) {
        const uint32_t seg = seg_of_tile(a, t);
        const uint32_t seg_t1 = strided ? t1 : min(t1, seg_end_tile(a, seg));
        const CorePlan plan = plan_of(a, seg);
        CoreState* st = a.state + seg;
        uint32_t* hs = a.hist + (size_t)seg * H_STRIDE;
        if (plan.need == 0) {
            if (threadIdx.x == 0) { st->none = 1; st->skip = 0; }
            t = seg_t1;
            continue;
        }
        const BinPick p = half ? pick_bin<(int)CORE_NB0 / 2>(hs + H_L0, plan.need, wtot, sh)
                               : pick_bin<(int)CORE_NB0>(hs + H_L0, plan.need, wtot, sh);
        const bool ok = p.total >= plan.need;            // fewer counted than asked for: the histogram is not of this score
        const bool skip = ok && check && used[seg] == p.bin;
        if (threadIdx.x == 0) {
            st->none = ok ? 0u : 1u; st->skip = skip ? 1u : 0u;
            st->prefix0 = p.bin; st->need0 = p.left;
            if (!ok) atomicOr(&a.flags[1], 2u);
        }
        uint32_t tt = t, te = seg_t1;
        if (skip) {                                      // a ragged last tile at most; one block looks at it, whatever its own range
            tt = a.T - 1u;
            te = (blockIdx.x == 0 && (a.n % TILE) != 0) ? a.T : tt;
        }
        if (!ok) te = tt;
        // two tiles a turn: the scores of both are requested before either is worked on
        for (; tt < te; tt += 2 * tstep) {
            const uint32_t tB = tt + tstep;
            const bool two = tB < te;
            const TileRef A = tile_ref(tt, a.n_seg, a.n, a.tile_start, a.tile_seg);
            const TileRef B = two ? tile_ref(tB, a.n_seg, a.n, a.tile_start, a.tile_seg) : TileRef{0u, 0u, 0u};
            uint32_t keyA[4][4], keyB[4][4];
            core_load_keys(S, A.start, A.len, wid, lane, keyA);
            if (two) core_load_keys(S, B.start, B.len, wid, lane, keyB);
            core_classify(keyA, tt, A.start, A.len, wid, lane, p.bin, h, a);
            if (two) core_classify(keyB, tB, B.start, B.len, wid, lane, p.bin, h, a);
        }
        __syncthreads();
        flush_hist(h, CORE_NB1, hs + (skip ? H_L1 : H_L1B));
        __syncthreads();
        t = seg_t1;
    }
}

// ---------------------------------------------------------------------------------------
// Level-2 histogram of the candidates whose first 25 bits are the threshold's.  One wave per tile of the block's
// group, 16 lanes per sub-tile list.  grid: groups.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_core_hist2(CoreArgs a)
{
    __shared__ uint32_t h2[CORE_NB2];
    __shared__ uint32_t wtot[4], sh[4];
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    uint32_t t = group_first(blockIdx.x, a.T, a.groups);
    const uint32_t t1 = group_first(blockIdx.x + 1, a.T, a.groups);
    while (t < t1) {
        const uint32_t seg = seg_of_tile(a, t), seg_t1 = min(t1, seg_end_tile(a, seg));
        CoreState* st = a.state + seg;
        if (st->none) { t = seg_t1; continue; }
        uint32_t* hs = a.hist + (size_t)seg * H_STRIDE;
        const uint32_t prefix0 = st->prefix0, need0 = st->need0, region = st->skip ? H_L1 : H_L1B;
        if (threadIdx.x < CORE_NB2) h2[threadIdx.x] = 0;
        const BinPick p = pick_bin<(int)CORE_NB1>(hs + region, need0, wtot, sh);
        const uint32_t prefix = (prefix0 << 12) | p.bin;
        if (threadIdx.x == 0) { st->prefix1 = prefix; st->need1 = p.left; }
        for (uint32_t tt = t + wid; tt < seg_t1; tt += 4) {
            const TileRef tr = tile_ref(tt, a.n_seg, a.n, a.tile_start, a.tile_seg);
            const uint32_t* keys = a.cand_keys + (size_t)tr.start + (lane >> 4) * SUB;
            const uint32_t c = a.cnt_cand[(size_t)tt * SUBS + (lane >> 4)];
            uint32_t kv[CORE_KPL];
            load_sublists<CORE_KPL>(a.cand_keys + (size_t)tr.start, lane, kv);
#pragma unroll
            for (int i = 0; i < CORE_KPL; ++i)
                if ((lane & 15u) + 16u * i < c && (kv[i] >> CORE_SHIFT1) == prefix) atomicAdd(&h2[kv[i] & (CORE_NB2 - 1u)], 1u);
            for (uint32_t j = (lane & 15u) + 16u * CORE_KPL; j < c; j += 16) {
                const uint32_t k = keys[j];
                if ((k >> CORE_SHIFT1) == prefix) atomicAdd(&h2[k & (CORE_NB2 - 1u)], 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x < CORE_NB2 && h2[threadIdx.x]) atomicAdd(&hs[H_L2 + threadIdx.x], h2[threadIdx.x]);
        __syncthreads();
        t = seg_t1;
    }
}

// ---------------------------------------------------------------------------------------
// Threshold key and tie quota; per tile the number of keys certainly taken (above the bin, or candidates above the
// threshold) and of those equal to it, as prefixes inside the block's group and segment.  What a tile emits is
// then certain + min(quota, ties before and in it) - min(quota, ties before it): one prefix of the pair is enough.
// The block that holds a segment's first tile also leaves the prediction of the next threshold's bin, the verdict
// on the capture of the scoring pass and the next capture bound.  grid: groups.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_core_count(CoreArgs a, SpecTau sp, uint32_t* __restrict__ pred)
{
    __shared__ uint2 cnt[GROUP_MAX];
    __shared__ uint32_t wtot[4], sh[4];
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    const uint32_t g0 = group_first(blockIdx.x, a.T, a.groups);
    uint32_t t = g0;
    const uint32_t t1 = group_first(blockIdx.x + 1, a.T, a.groups);
    uint2 tail = make_uint2(0u, 0u);
    while (t < t1) {
        const uint32_t seg = seg_of_tile(a, t), seg_t1 = min(t1, seg_end_tile(a, seg));
        CoreState* st = a.state + seg;
        const bool owner = threadIdx.x == 0 && t == seg_begin_tile(a, seg), none = st->none != 0;
        if (none) {
            if (owner) {
                st->tau = NONE; st->quota = 0;
                if (pred) pred[seg] = NONE;
                if (sp.next) { sp.fail[seg] = 0; sp.next[seg] = NONE; }      // nothing selected, nothing to capture
            }
            for (uint32_t tt = t + threadIdx.x; tt < seg_t1; tt += BLOCK) a.tile_pre[tt] = make_uint2(0u, 0u);
            tail = make_uint2(0u, 0u);
            t = seg_t1;
            continue;
        }
        const BinPick p = pick_bin<(int)CORE_NB2>(a.hist + (size_t)seg * H_STRIDE + H_L2, st->need1, wtot, sh);
        const uint32_t tau = (st->prefix1 << CORE_SHIFT1) | p.bin;
        if (owner) {
            st->tau = tau; st->quota = p.left;
            if (pred) pred[seg] = tau >> CORE_SHIFT0;
            if (sp.next) {
                sp.fail[seg] = (tau < sp.cur[seg]) ? 1u : 0u;
                sp.next[seg] = tau > SPEC_MARGIN ? tau - SPEC_MARGIN : 0u;
            }
        }
        for (uint32_t tt = t + wid; tt < seg_t1; tt += 4) {
            const TileRef tr = tile_ref(tt, a.n_seg, a.n, a.tile_start, a.tile_seg);
            const uint32_t* keys = a.cand_keys + (size_t)tr.start + (lane >> 4) * SUB;
            const uint32_t c = a.cnt_cand[(size_t)tt * SUBS + (lane >> 4)];
            const uint32_t gt = a.cnt_gt[(size_t)tt * SUBS + (lane >> 4)];
            uint32_t kv[CORE_KPL];
            load_sublists<CORE_KPL>(a.cand_keys + (size_t)tr.start, lane, kv);
            uint32_t sel = (lane & 15u) == 0 ? gt : 0u, tie = 0;
#pragma unroll
            for (int i = 0; i < CORE_KPL; ++i)
                if ((lane & 15u) + 16u * i < c) { sel += (kv[i] > tau) ? 1u : 0u; tie += (kv[i] == tau) ? 1u : 0u; }
            for (uint32_t j = (lane & 15u) + 16u * CORE_KPL; j < c; j += 16) {
                const uint32_t k = keys[j];
                sel += (k > tau) ? 1u : 0u;
                tie += (k == tau) ? 1u : 0u;
            }
            const uint32_t both = wave_sum(sel | (tie << 16));       // a tile holds at most 4096 of either
            if (lane == 0) cnt[tt - g0] = make_uint2(both & 0xFFFFu, both >> 16);
        }
        __syncthreads();
        if (wid == 0) {
            uint2 run = make_uint2(0u, 0u);
            for (uint32_t x0 = t; x0 < seg_t1; x0 += 64) {
                const uint32_t x = x0 + lane;
                const uint2 v = (x < seg_t1) ? cnt[x - g0] : make_uint2(0u, 0u);
                const uint32_t is = wave_incl_scan(v.x), it = wave_incl_scan(v.y);
                if (x < seg_t1) a.tile_pre[x] = make_uint2(run.x + is - v.x, run.y + it - v.y);
                run.x += last_lane(is); run.y += last_lane(it);
            }
            tail = run;
        }
        __syncthreads();
        t = seg_t1;
    }
    if (threadIdx.x == 0) a.group_tail[blockIdx.x] = tail;
}

// ---------------------------------------------------------------------------------------
// Ordered emission.  One wave per tile, each lane owning two consecutive bitmap words: decide every candidate
// against tau, hand out the tie quota in index order, write the tile's chosen indices at its offset and its
// bits to the public bitmap.  Each group of tiles is served by per_group blocks.  The core size of a segment is known,
// so only the tiles of the own segment come before: those of earlier groups through the groups' tails.
// Clears the histograms on the way.  grid: groups * per_group.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_core_emit(CoreArgs a, uint32_t per_group, uint32_t* __restrict__ out_idx,
                                                     uint32_t* __restrict__ out_off, uint32_t* __restrict__ pub_bits, uint32_t expected)
{
    __shared__ uint32_t kb[4][SUBS * 16 * CORE_KPL];
    __shared__ uint16_t stage[4][EMIT_STAGE];
    __shared__ uint2 part[4];
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    const uint32_t g = blockIdx.x / per_group, r = blockIdx.x % per_group;
    const uint32_t g0 = group_first(g, a.T, a.groups), g1 = group_first(g + 1, a.T, a.groups);
    const uint32_t t0 = g0 + (g1 - g0) * r / per_group, t1 = g0 + (g1 - g0) * (r + 1) / per_group;
    for (uint64_t x = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; x < (uint64_t)a.n_seg * (H_STRIDE / 4); x += (uint64_t)gridDim.x * BLOCK)
        reinterpret_cast<uint4*>(a.hist)[x] = make_uint4(0u, 0u, 0u, 0u);
    if (t0 >= t1) return;
    // the first segment of the group may have begun in an earlier one
    const uint32_t seg0 = seg_of_tile(a, g0), f0 = seg_begin_tile(a, seg0);
    uint2 carry = make_uint2(0u, 0u);
    if (f0 < g0) {
        uint2 s = make_uint2(0u, 0u);
        for (uint32_t x = group_of(f0, a.T, a.groups) + threadIdx.x; x < g; x += BLOCK) { const uint2 v = a.group_tail[x]; s.x += v.x; s.y += v.y; }
        s.x = wave_sum(s.x); s.y = wave_sum(s.y);
        if (lane == 0) part[wid] = s;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) { carry.x += part[w].x; carry.y += part[w].y; }
    }
    uint32_t* kbw = kb[wid];
    for (uint32_t t = t0 + wid; t < t1; t += 4) {
        // everything the tile needs is requested here, before any of it is used
        const TileRef tr = tile_ref(t, a.n_seg, a.n, a.tile_start, a.tile_seg);
        const uint2 g2 = *reinterpret_cast<const uint2*>(a.gt_bits + (size_t)t * TILE_WORDS + 2 * lane);
        const uint2 c2 = *reinterpret_cast<const uint2*>(a.cand_bits + (size_t)t * TILE_WORDS + 2 * lane);
        uint32_t kv[CORE_KPL];
        load_sublists<CORE_KPL>(a.cand_keys + (size_t)tr.start, lane, kv);
        uint2 pre = a.tile_pre[t];
        const CoreState* st = a.state + tr.seg;
        const uint32_t none = st->none, tau = st->tau, quota = st->quota;
        const uint32_t base = plan_of(a, tr.seg).base;
        if (tr.seg == seg0) { pre.x += carry.x; pre.y += carry.y; }
        const uint32_t* keys = a.cand_keys + (size_t)tr.start;
        uint32_t cw[2] = {0u, 0u}, gw[2] = {0u, 0u};
        if (!none) { cw[0] = c2.x; cw[1] = c2.y; gw[0] = g2.x; gw[1] = g2.y; }
        wave_sync();
#pragma unroll
        for (int i = 0; i < CORE_KPL; ++i) kbw[(lane >> 4) * (16 * CORE_KPL) + (lane & 15u) + 16 * i] = kv[i];
        wave_sync();
        const uint32_t pos = sublist_pos(lane, __popc(cw[0]) + __popc(cw[1]));
        const uint32_t sub = pos >> 10;
        uint32_t j = pos & (SUB - 1u);
        uint32_t selmask[2] = {0u, 0u}, tiemask[2] = {0u, 0u};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t m = cw[h];
            while (m) {
                const uint32_t p = __ffs(m) - 1;
                m &= m - 1;
                const uint32_t k = (j < 16u * CORE_KPL) ? kbw[sub * (16 * CORE_KPL) + j] : keys[sub * SUB + j];
                ++j;
                if (k > tau) selmask[h] |= 1u << p;
                else if (k == tau) tiemask[h] |= 1u << p;
            }
        }
        const uint32_t tcnt = __popc(tiemask[0]) + __popc(tiemask[1]);
        uint32_t taken[2] = {0u, 0u};
        if (__ballot(tcnt != 0)) {
            const uint32_t tbase = pre.y + wave_incl_scan(tcnt) - tcnt;
            uint32_t take = (quota > tbase) ? quota - tbase : 0u;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t m = tiemask[h];
                while (m && take) { const uint32_t low = m & (0u - m); taken[h] |= low; m ^= low; --take; }
            }
        }
        const uint32_t fm0 = gw[0] | selmask[0] | taken[0], fm1 = gw[1] | selmask[1] | taken[1];
        const uint32_t ocnt = __popc(fm0) + __popc(fm1);
        const uint32_t first = base + pre.x + min(quota, pre.y);
        const uint32_t oincl = wave_incl_scan(ocnt);
        if (lane == 0) out_off[t] = first;
        if (t == a.T - 1 && lane == 63) {
            out_off[a.T] = first + oincl;
            if (first + oincl != expected) atomicOr(&a.flags[1], 1u);
        }
        emit_indices(fm0, fm1, oincl, tr.start, first, expected, stage[wid], out_idx);
        // the public bitmap: whole words directly; words shared with a neighbouring tile (cleared by k_core_build) by OR
        const uint32_t sft = tr.start & 31u;
        uint32_t* pb = pub_bits + (tr.start >> 5) + 2 * lane;
        if (sft == 0) {
            const uint32_t i0 = lane * 64u;
            if (i0 < tr.len) { if (a.n_seg == 1 || i0 + 32u <= tr.len) pb[0] = fm0; else if (fm0) atomicOr(&pb[0], fm0); }
            if (i0 + 32u < tr.len) { if (a.n_seg == 1 || i0 + 64u <= tr.len) pb[1] = fm1; else if (fm1) atomicOr(&pb[1], fm1); }
        } else {
            uint32_t prev = __shfl_up(fm1, 1, 64);
            if (lane == 0) prev = 0;
            const uint32_t w0 = (fm0 << sft) | (prev >> (32u - sft)), w1 = (fm1 << sft) | (fm0 >> (32u - sft));
            // word 2 * lane + j covers positions 64 * lane + 32 * j - sft .. + 31 of the tile
            const int p0 = (int)(lane * 64u) - (int)sft, end = (int)tr.len;
            if (p0 >= 0 && p0 + 32 <= end) pb[0] = w0; else if (w0) atomicOr(&pb[0], w0);
            if (p0 + 64 <= end) pb[1] = w1; else if (w1) atomicOr(&pb[1], w1);
            if (lane == 63 && (fm1 >> (32u - sft))) atomicOr(&pb[2], fm1 >> (32u - sft));
        }
    }
}

}  // namespace slimdp
