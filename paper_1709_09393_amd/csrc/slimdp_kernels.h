// Kernels of libslimdp (gfx950).  Included only by slimdp.hip.
//
// Shared structure: the index range is cut into tiles of <= 4096 parameters (never across a segment).  The core
// selection is in slimdp_core.h, the explorer's (what follows the draw) in slimdp_explore.h.  In both, the parameters
// in doubt ("candidates") are a per-tile bitmap plus the keys of each 1024-parameter sub-tile compacted in index
// order at cand_keys[tile_start + 1024*s ...] with their number in cnt_cand[4*tile + s] (a sub-tile is what one wave
// handles on its own, without block barriers).
#pragma once
#include "slimdp_device.h"

// Cache policy of the streaming accesses, per kernel (0 = default, 1 = non-temporal).  Measured on the VGG-16-sized
// workload: each switch alone moves its kernel by 0 to 5 %, all together take 0.07 ms off the 2.75 ms step.
#ifndef NT_BUILD
#define NT_BUILD 1
#endif
#ifndef NT_MERGE_LD
#define NT_MERGE_LD 1
#endif
#ifndef NT_MERGE_ST
#define NT_MERGE_ST 1
#endif
#ifndef NT_MERGE_VAL
#define NT_MERGE_VAL 1
#endif
#ifndef NT_PACKS
#define NT_PACKS 1
#endif
#ifndef NT_PACKC_LD
#define NT_PACKC_LD 1
#endif
#ifndef NT_PACKC_ST
#define NT_PACKC_ST 1
#endif
#ifndef NT_EXPLG
#define NT_EXPLG 1
#endif

namespace slimdp {

// ---------------------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, uint64_t count, uint32_t v)
{
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (uint64_t)gridDim.x * 256)
        p[i] = v;
}

// ---------------------------------------------------------------------------------------
// K4: the explorer draw of one (worker, sub-tile), by ONE wave with no block barrier: the
// Philox word r of each parameter, sorted into two zones chosen on the host so that the
// m-th smallest word of the segment falls into the second one:
//   sure zone       r <= sure_m1 (if has_sure): one bit in the "sure" bitmap; such a
//                   parameter is taken unless it turns out to be in the core;
//   candidate zone  sure_m1 < r <= bound_m1: one bit in the candidate bitmap plus the key
//                   bound_m1 - r (the smallest words are the largest keys), the keys of a
//                   sub-tile compacted in index order.
// The draw does not look at the core; a later pass applies it, so the same routine serves
// inside the scoring kernel (core not known yet) and stand-alone.
// PAIRS = 1 (every segment's candidate zone is narrow): no candidate bitmap; the sub-tile's
// slot holds (key, offset inside the sub-tile) pairs, at most PAIR_CAP of them: the count still
// reports any beyond, which the gathering pass turns into the exact rerun.
// ---------------------------------------------------------------------------------------
struct PhiloxKey { uint32_t seed_lo, seed_hi, it_lo, it_hi; };
// PAIRS = 1: a sub-tile's (key, offset) pairs live in a slot of PAIR_SLOT words at
// cand_keys[(tile * SUBS + sub-tile) * PAIR_SLOT]: PAIR_CAP pairs, about a hundred times the expected number.
constexpr uint32_t PAIR_CAP = 16, PAIR_SLOT = 2 * PAIR_CAP;
struct DrawOut {                 // per batch (worker) base pointers
    uint32_t* sure_bits;         // [T * TILE_WORDS]
    uint32_t* cand_bits;         // [T * TILE_WORDS]
    uint32_t* cand_keys;         // [keys_stride]
    uint32_t* cnt_cand;          // [T * SUBS]
};

// LDS traffic between the lanes of one wave: the hardware keeps a wave's LDS operations in
// order, this keeps the compiler from moving them across the hand-over point.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_wave_barrier();
}

// Which of a lane's four parameters e0 .. e0+3 lie inside a ragged sub-tile of sub_len parameters.
__device__ __forceinline__ uint32_t inside_mask(uint32_t e0, uint32_t sub_len)
{
    const uint32_t left = (e0 < sub_len) ? sub_len - e0 : 0u;
    return (left >= 4u) ? 15u : ((1u << left) - 1u);
}

// No LDS: round `it` covers the 256 parameters [256*it, 256*it+256) of the sub-tile in index order (lane L owns
// parameters 4L..4L+3 of the round: one Philox block), so a candidate's place in the key list is the number of
// candidates in earlier rounds plus a wave ballot count.  Bound by the vector unit: 15 wide multiplications and 17
// exclusive ors for four words, then a subtraction whose borrow is the sure flag and an addition with carry that files it
// for each of them; the four rounds' flags become bitmap words together (transpose_flags): 51 instructions a round and worker,
// the vector units busy all the time when it runs alone.  With every worker's words from the beginning, masks and a reduction for each
// round's words (67 instructions): 138*10^6 parameters, 8 workers 535 -> 407 us, 20*10^6 and 3 workers 38 -> 33 us.
// MIS = 1: tiles may begin inside a Philox block (segmented models).  Everything above then counts from the start of that
// block, mis = start mod 4 positions earlier; the bitmaps are shifted down by mis at the end, and the block that holds the
// sub-tile's last mis parameters is computed apart, from wave-uniform values, that is by the scalar unit beside the
// vector one.  (As a fifth round through LDS bitmaps the draw of 7*10^6 parameters for 4 workers took 36 us.)
// What a lane's four blocks share between the workers (philox_common): the caller keeps it, for as many workers as it draws.
struct DrawLanes {
    PhiloxCommon c[4];
    __device__ __forceinline__ PhiloxCommon operator()(int it) const { return c[it]; }
};
struct ParkedLanes {             // the same in LDS: [round][lane], written and read by one wave
    const uint4* at;
    __device__ __forceinline__ PhiloxCommon operator()(int it) const
    {
        const uint4 v = at[it * 64 + (int)lane_id()];
        return PhiloxCommon{v.x, v.y, v.z, v.w};
    }
};
__device__ __forceinline__ DrawLanes draw_lanes(uint32_t start, uint32_t sub, const PhiloxKey& pk)
{
    DrawLanes d;
    const uint32_t g = ((start + sub * SUB) >> 2) + lane_id();
#pragma unroll
    for (uint32_t it = 0; it < 4; ++it) d.c[it] = philox_common(g + it * 64u, pk.it_lo, pk.it_hi, pk.seed_lo, pk.seed_hi);
    return d;
}
__device__ __forceinline__ void park_lanes(uint4* at, const DrawLanes& d)
{
    wave_sync();
#pragma unroll
    for (int it = 0; it < 4; ++it) at[it * 64 + (int)lane_id()] = make_uint4(d.c[it].x, d.c[it].y, d.c[it].z, d.c[it].d);
    wave_sync();
}
template <int PAIRS, int MIS, class LANES>
__device__ __forceinline__ void explore_subtile(uint32_t worker, uint32_t t, uint32_t sub, uint32_t start, uint32_t len,
                                                uint32_t bound_m1, uint32_t sure_m1, uint32_t has_sure, uint32_t skip,
                                                const DrawOut& out, const PhiloxKey& pk, const PhiloxRoundKeys& keys, const LANES& lanes)
{
    const uint32_t lane = lane_id();
    const uint32_t off = sub * SUB;
    const uint32_t sub_len = (len > off) ? ((len - off < SUB) ? len - off : SUB) : 0u;
    // the sub-tile's bitmap words and count through descriptors (t and sub are the same for the whole wave): scalar bases,
    // no per-lane 64-bit addresses that a caller's loop over workers would have to carry along
    const __amdgpu_buffer_rsrc_t rc = buffer_of(out.cand_bits + (size_t)t * TILE_WORDS + sub * SUB_WORDS, SUB_WORDS * 4u);
    const __amdgpu_buffer_rsrc_t rs = buffer_of(out.sure_bits + (size_t)t * TILE_WORDS + sub * SUB_WORDS, SUB_WORDS * 4u);
    const __amdgpu_buffer_rsrc_t rn = buffer_of(out.cnt_cand + (size_t)t * SUBS + sub, 4u);
    if (sub_len == 0 || skip) {                                   // uniform over the wave
        if (lane < SUB_WORDS) {
            if (!PAIRS) buffer_store1(rc, lane * 4u, 0u);
            buffer_store1(rs, lane * 4u, 0u);
        }
        if (lane == 0) buffer_store1(rn, 0u, 0u);
        return;
    }
    const uint32_t base = start + off, mis = MIS ? base & 3u : 0u;
    const uint32_t end = sub_len + mis;                              // positions mis .. end - 1 belong to the sub-tile
    uint32_t* ckeys = PAIRS ? out.cand_keys + ((size_t)t * SUBS + sub) * PAIR_SLOT : out.cand_keys + (size_t)base;
    const uint32_t sure_excl = has_sure ? sure_m1 + 1u : 0u;         // sure_m1 < bound_m1: no overflow
    const uint32_t width_m1 = bound_m1 - sure_excl;                  // candidate words are sure_excl .. bound_m1
    const uint64_t v = philox_worker(worker, pk.it_lo, pk.seed_lo);
    uint32_t run = 0, sure = 0, cand = 0;                            // flags of the rounds so far, the last one lowest
    // a candidate's key and place, by the lane that owns it
    auto put = [&](uint32_t pos, uint32_t word, uint32_t e) {
        if (!PAIRS) ckeys[pos] = bound_m1 - word;
        else if (pos < PAIR_CAP) { ckeys[2u * pos] = bound_m1 - word; ckeys[2u * pos + 1u] = e - mis; }
    };
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint32_t e0 = (uint32_t)it * 256u + lane * 4u;      // first of this lane's four positions
        uint32_t r[4], d[4];
        philox_words(lanes(it), v, keys, r);
        sub4_borrow(r, sure_excl, d, sure);        // a word inside the sure zone wraps to a huge distance
        // candidate zone sure_excl <= word <= bound: one test for the four; the per-parameter work only when some lane of
        // the wave has one, which is rare with a narrow zone
        const uint32_t dmin = min(min(d[0], d[1]), min(d[2], d[3]));
        uint32_t fc = 0;
        if (__ballot(dmin <= width_m1) != 0ull) {                     // uniform
            fc = (d[0] <= width_m1 ? 1u : 0u) | (d[1] <= width_m1 ? 2u : 0u) | (d[2] <= width_m1 ? 4u : 0u) |
                 (d[3] <= width_m1 ? 8u : 0u);
            if (MIS || end != SUB) {                                  // a ragged or shifted sub-tile
                fc &= inside_mask(e0, end);
                if (MIS && it == 0 && lane == 0) fc &= ~((1u << mis) - 1u);
            }
            // place in the list: candidates of lower lanes in this round, all four components
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
                    if ((fc >> cc) & 1u) put(pos++, r[cc], e0 + cc);
            }
            run += total;
        }
        if (!PAIRS) cand |= fc << (4 * it);
    }
    sure = __brev(sure) >> 16;                                       // bit 4 * round + component
    if (MIS || end != SUB) {
        uint32_t in = 0;
#pragma unroll
        for (int it = 0; it < 4; ++it) in |= inside_mask((uint32_t)it * 256u + lane * 4u, end) << (4 * it);
        if (MIS && lane == 0) in &= ~((1u << mis) - 1u);
        sure &= in;
    }
    // the block beyond the four rounds: positions SUB .. end - 1, at most three (uniform)
    uint32_t xs = 0, xc = 0;
    if (MIS && end > SUB) {
        uint32_t r[4];
        philox4x32_10((base >> 2) + SUB / 4u, worker, pk.it_lo, pk.it_hi, pk.seed_lo, pk.seed_hi, r);
#pragma unroll
        for (uint32_t cc = 0; cc < 3; ++cc) {
            if (SUB + cc >= end) break;
            if (r[cc] < sure_excl) xs |= 1u << cc;
            else if (r[cc] - sure_excl <= width_m1) {
                xc |= 1u << cc;
                if (lane == 0) put(run, r[cc], SUB + cc);
                ++run;
            }
        }
    }
    // the 32 bitmap words of the sub-tile in one store of one whole line by lanes 0..31 in address order (scattered
    // words make the memory side read the line first): word 8 * round + j sits in lane 8 * j + 2 * round
    const int src = (int)(8u * (lane & 7u) + 2u * ((lane >> 3) & 3u));
    auto store = [&](const __amdgpu_buffer_rsrc_t& dst, uint32_t flags, uint32_t extra) {
        uint32_t w = __shfl(transpose_flags(flags), src, 64);
        if (MIS && mis) {                                              // uniform
            uint32_t next = __shfl_down(w, 1, 64);
            if (lane == SUB_WORDS - 1u) next = extra;
            w = (w >> mis) | (next << ((32u - mis) & 31u));          // mis is 1 to 3
        }
        if (lane < SUB_WORDS) buffer_store1(dst, lane * 4u, w);
    };
    store(rs, sure, xs);
    if (!PAIRS) store(rc, cand, xc);
    if (lane == 0) buffer_store1(rn, 0u, run);
}

// ---------------------------------------------------------------------------------------
// K1: significance of every parameter + level-0 histogram of its bits (per segment).
// Reads w and the W updates once, writes the score once: 4n(W+2) bytes.
// With DENSE = 1 (the iteration before a reselection, algorithm 1 / section 3.3 steps
// 3 and 6: every worker pushed its whole update) the model is first updated with all of them,
// w_new = fma(-lr, (+0 + g_0) + g_1 + ..., w), written to w_new (which may be w itself), and
// the significance is that of the new model: 4n(W+3) bytes.
// Persistent blocks over contiguous tile ranges keep the level-0 histogram in LDS.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void flush_hist(uint32_t* lds, uint32_t nb, uint32_t* __restrict__ g)
{
    for (uint32_t b = threadIdx.x; b < nb; b += BLOCK) {
        const uint32_t v = lds[b];
        if (v) { atomicAdd(&g[b], v); lds[b] = 0; }
    }
}

// PRE != 0 additionally draws the explorer zones of pre.nw workers for every tile
// (explore_subtile): integer work that runs while other waves wait for memory.
// Explorer capture (flat models, narrow zones, speculative packing): the update values of the parameters in the sure zones,
// kept by the scoring pass for the pack.  A sub-tile has PreArgs::slots values for each worker scored, in the order of
// the parameters' blocks of four: the first sure parameter of every block that has one.  Which those are is told by the
// sure bitmap as the draw left it.
constexpr uint32_t EXPL_SLOTS_FEW = 32, EXPL_SLOTS_MAX = 48;        // whole lines for two workers and more
struct PreArgs {
    uint32_t nw, worker0, n_seg;
    const SegState* states;
    uint32_t* sure_bits;
    uint32_t* cand_bits;
    uint32_t* cand_keys;
    uint32_t* cnt_cand;
    uint64_t keys_stride;
    PhiloxKey pk;
    float* vals;             // explorer capture (see above); slots: entries a sub-tile and worker, 0: none
    uint32_t slots;
};

// SPEC = 1 (speculative packing, WT != 0 only) keeps, for every parameter of a whole
// tile whose significance reaches spec.lo[segment] - a little below the core threshold of
// the previous selection -, the W update values while they are in registers: one bit in
// spec.bits (beside each bitmap word: the entry number of its first parameter), and one
// entry of W consecutive values in spec.vals.  The entries of a sub-tile
// follow each other in index order from entry (tile start + 1024 * sub-tile); each round of
// 256 parameters starts on a 128-byte line and its last line is filled up, so that every
// line is written whole and at once (a line written in parts minutes apart leaves the cache
// in between and costs a read-modify-write in memory).
// If the coming selection's threshold is not below spec.lo, every core parameter is among
// them and the pack need not read the updates again.
struct SpecArgs {
    const uint32_t* lo;      // [n_seg] lowest captured significance (as bits)
    uint2* bits;             // [T * TILE_WORDS] x = the bits, y = number of the word's first entry inside its sub-tile
    float* vals;             // [entries][W]
};
// A sub-tile's entries live at spec.vals[(tile * SUBS + sub-tile) * SPEC_CAP * W]; entries beyond SPEC_CAP (a quarter
// of the sub-tile: two and a half times a 10 % core) are not kept (the descriptor's range drops their stores) and
// the pack reads those parameters from the update vectors.
constexpr uint32_t SPEC_CAP = SUB / 4;
__host__ __device__ constexpr uint32_t spec_align(uint32_t W) { return (W == 0u || W >= 32u) ? 1u : 32u / W; }   // entries per 128-byte line

#ifndef SCORE_MINB
#define SCORE_MINB 4
#endif
#ifndef SCORE_LD_AUX
#define SCORE_LD_AUX 2          // cache policy of the general scoring kernel's loads: non-temporal (the stress workload scores 4 % faster)
#endif
template <int WT, int PRE, int SPEC, int DENSE, int STRIDED>
__global__ __launch_bounds__(BLOCK, SCORE_MINB) void k_score(const float* __restrict__ w, PtrTab g, int Wrt, float c,
                                                 float* __restrict__ S, const uint32_t* __restrict__ tile_start,
                                                 const uint32_t* __restrict__ tile_seg, uint32_t T,
                                                 uint32_t* __restrict__ hist, PreArgs pre, SpecArgs spec,
                                                 float* __restrict__ w_new, float lr)
{
    static_assert(!SPEC || WT != 0, "capture needs the update values in registers");
    static_assert(!(SPEC && DENSE), "a dense update is never followed by a pack of the same updates");
    // a significance is never negative: its sign bit is clear and the upper half of the level-0 bins stays empty
    constexpr uint32_t NB = CORE_NB0 / 2;
    __shared__ uint32_t h[NB];
    const int W = WT ? WT : Wrt;
    // the wave's number as a scalar: addresses below are then a scalar base plus a small per-lane offset
    const uint32_t lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lane16 = lane * 16u;      // byte offset of the lane's sixteen bytes inside a round
    for (uint32_t b = threadIdx.x; b < NB; b += BLOCK) h[b] = 0;
    __syncthreads();
    // A block's tiles: a contiguous range (few segment changes, each of which flushes the histogram), or - flat model,
    // STRIDED - every gridDim.x-th tile, so that at any moment the whole chip streams through one window of each
    // array instead of a thousand separate places (fewer DRAM rows open at a time).  A compile-time choice: with the
    // step in a register the 16-worker variant spills more and loses 0.3 ms.
    const uint32_t t0 = STRIDED ? blockIdx.x : (uint32_t)((uint64_t)T * blockIdx.x / gridDim.x);
    const uint32_t t1 = STRIDED ? T : (uint32_t)((uint64_t)T * (blockIdx.x + 1) / gridDim.x);
    const uint32_t tstep = STRIDED ? gridDim.x : 1u;
    if (t0 >= t1) return;
    uint32_t cur_seg = tile_seg[t0];
    // Every wave owns sub-tile `wid` of each tile and runs through the block's tiles on its
    // own; the block only meets at a segment change and at the end (histogram flush).
    for (uint32_t t = t0; t < t1; t += tstep) {
        const uint32_t seg = tile_seg[t];
        if (seg != cur_seg) {
            __syncthreads();
            flush_hist(h, NB, hist + (size_t)cur_seg * H_STRIDE + H_L0);
            __syncthreads();
            cur_seg = seg;
        }
        const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
        // the candidate bound depends on the segment only (every worker draws the same number)
        uint32_t pre_bound = 0, pre_sure = 0, pre_has_sure = 0, pre_skip = 1;
        if (PRE) {
            const SegState* st = &pre.states[seg];
            pre_bound = st->bound_m1; pre_sure = st->sure_m1; pre_has_sure = st->has_gt; pre_skip = st->need0 == 0;
        }
        // Sixteen bytes at a time wherever a tile begins: three of four segments do not begin on a multiple of four, and by single
        // floats, uncaptured besides, they kept an iteration of 7*10^6 parameters in 57 segments at 216 us (195 now).
        const bool vec = len == TILE;
        uint32_t spec_lo = 0xFFFFFFFFu, spec_run = 0;
        if (SPEC) spec_lo = spec.lo[seg];
        if (!vec) {
            const uint32_t lo = wid * SUB, hi = (lo + SUB < len) ? lo + SUB : len;
            for (uint32_t l = lo + lane; l < hi; l += 64) {
                const size_t e = (size_t)start + l;
                float a = static_cast<const float*>(g.p[0])[e];
                for (int k = 1; k < W; ++k) a = a + static_cast<const float*>(g.p[k])[e];
                float we = w[e];
                if (DENSE) { we = __builtin_fmaf(-lr, a + 0.0f, we); w_new[e] = we; }      // dense update first
                const float sc = significance(we, a, c);
                S[e] = sc;
                atomicAdd(&h[(__float_as_uint(sc) >> CORE_SHIFT0) & (NB - 1u)], 1u);
            }
        }
        if (!vec && !PRE) continue;
        // the tile through buffer descriptors (scalar base per array, one 32-bit lane offset for all of them)
        const __amdgpu_buffer_rsrc_t rw = buffer_of(w + start, TILE * 4u);
        const __amdgpu_buffer_rsrc_t rS = buffer_of(S + start, TILE * 4u);
        const __amdgpu_buffer_rsrc_t rn = buffer_of(DENSE ? w_new + start : S + start, TILE * 4u);
        __amdgpu_buffer_rsrc_t rg[WT ? WT : 1];
        if (WT) {
#pragma unroll
            for (int k = 0; k < WT; ++k) rg[k] = buffer_of(static_cast<const float*>(g.p[k]) + start, TILE * 4u);
        }
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
            const size_t e0 = (size_t)start + (size_t)wid * SUB + (size_t)r * 256;      // uniform over the wave
            const uint32_t lane_bytes = (wid * SUB + (uint32_t)r * 256u) * 4u + lane16;  // of the lane's float4 inside the tile
            float4 wv = make_float4(0.f, 0.f, 0.f, 0.f);
            float4 x[WT ? WT : 1];
            if (vec) {          // request this round's lines first ...
                wv = buffer_load4_aux<SCORE_LD_AUX>(rw, lane_bytes);
                if (WT) {
#pragma unroll
                    for (int k = 0; k < WT; ++k) x[k] = buffer_load4_aux<SCORE_LD_AUX>(rg[k], lane_bytes);
                }
            }
            if (PRE && (uint32_t)r < pre.nw) {          // ... do this round's share of the integer work while they fly ...
                const DrawLanes lanes = draw_lanes(start, wid, pre.pk);
                const PhiloxRoundKeys rk = philox_round_keys<false>(pre.pk.seed_lo, pre.pk.seed_hi);
#pragma unroll 1
                for (uint32_t b = (uint32_t)r; b < pre.nw; b += 4) {
                    DrawOut out;
                    out.sure_bits = pre.sure_bits + (size_t)b * T * TILE_WORDS;
                    out.cand_bits = pre.cand_bits + (size_t)b * T * TILE_WORDS;
                    out.cand_keys = pre.cand_keys + (size_t)b * pre.keys_stride;
                    out.cnt_cand = pre.cnt_cand + (size_t)b * T * SUBS;
                    explore_subtile<(PRE == 2) ? 1 : 0, 1>(pre.worker0 + b, t, wid, start, len, pre_bound, pre_sure,
                                                             pre_has_sure, pre_skip, out, pre.pk, rk, lanes);
                }
            }
            if (vec) {          // ... then score them
                float4 a;
                if (WT) {
                    a = x[0];
#pragma unroll
                    for (int k = 1; k < WT; ++k) { a.x = a.x + x[k].x; a.y = a.y + x[k].y; a.z = a.z + x[k].z; a.w = a.w + x[k].w; }
                } else {
                    a = ld4<0>(static_cast<const float*>(g.p[0]) + e0 + 4u * lane);
                    for (int k = 1; k < W; ++k) {
                        const float4 y = ld4<0>(static_cast<const float*>(g.p[k]) + e0 + 4u * lane);
                        a.x = a.x + y.x; a.y = a.y + y.y; a.z = a.z + y.z; a.w = a.w + y.w;
                    }
                }
                if (DENSE) {        // the server's dense update first (its sum starts from +0), then the new model's score
                    wv.x = __builtin_fmaf(-lr, a.x + 0.0f, wv.x); wv.y = __builtin_fmaf(-lr, a.y + 0.0f, wv.y);
                    wv.z = __builtin_fmaf(-lr, a.z + 0.0f, wv.z); wv.w = __builtin_fmaf(-lr, a.w + 0.0f, wv.w);
                    buffer_store4(rn, lane_bytes, 0u, wv);
                }
                float4 sc;
                sc.x = significance(wv.x, a.x, c); sc.y = significance(wv.y, a.y, c);
                sc.z = significance(wv.z, a.z, c); sc.w = significance(wv.w, a.w, c);
                buffer_store4(rS, lane_bytes, 0u, sc);
                atomicAdd(&h[(__float_as_uint(sc.x) >> CORE_SHIFT0) & (NB - 1u)], 1u);
                atomicAdd(&h[(__float_as_uint(sc.y) >> CORE_SHIFT0) & (NB - 1u)], 1u);
                atomicAdd(&h[(__float_as_uint(sc.z) >> CORE_SHIFT0) & (NB - 1u)], 1u);
                atomicAdd(&h[(__float_as_uint(sc.w) >> CORE_SHIFT0) & (NB - 1u)], 1u);
                if (SPEC) {
                    const uint32_t f = (__float_as_uint(sc.x) >= spec_lo ? 1u : 0u) | (__float_as_uint(sc.y) >= spec_lo ? 2u : 0u) |
                                       (__float_as_uint(sc.z) >= spec_lo ? 4u : 0u) | (__float_as_uint(sc.w) >= spec_lo ? 8u : 0u);
                    const uint32_t v = or_reduce8(f << (4u * (lane & 7u)));      // lanes 8j..8j+7 make bitmap word j of this round
                    uint32_t below = 0, total = 0;
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) {
                        const unsigned long long bal = __ballot((f >> cc) & 1u);
                        below += __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                        total += (uint32_t)__popcll(bal);
                    }
                    // lane 8j holds word j of the round and the number of captured parameters before it
                    if ((lane & 7u) == 0)
                        spec.bits[(size_t)t * TILE_WORDS + wid * SUB_WORDS + r * 8 + (lane >> 3)] = make_uint2(v, spec_run + below);
                    constexpr uint32_t A = spec_align(WT);
                    const uint32_t padded = (total + A - 1u) & ~(A - 1u);
                    // the sub-tile's entries through a descriptor: the entry number is the lane's part
                    const __amdgpu_buffer_rsrc_t rv = buffer_of(spec.vals + ((size_t)t * SUBS + wid) * SPEC_CAP * WT, SPEC_CAP * WT * 4u);
                    if (f) {
                        uint32_t pos = spec_run + below;
#pragma unroll
                        for (int cc = 0; cc < 4; ++cc) {
                            if ((f >> cc) & 1u) {
                                if (WT >= 4) {
#pragma unroll
                                    for (int k = 0; k < WT; k += 4) {
                                        float4 o;
                                        o.x = cc == 0 ? x[k].x : cc == 1 ? x[k].y : cc == 2 ? x[k].z : x[k].w;
                                        o.y = cc == 0 ? x[k + 1].x : cc == 1 ? x[k + 1].y : cc == 2 ? x[k + 1].z : x[k + 1].w;
                                        o.z = cc == 0 ? x[k + 2].x : cc == 1 ? x[k + 2].y : cc == 2 ? x[k + 2].z : x[k + 2].w;
                                        o.w = cc == 0 ? x[k + 3].x : cc == 1 ? x[k + 3].y : cc == 2 ? x[k + 3].z : x[k + 3].w;
                                        buffer_store4(rv, (pos * WT + k) * 4u, 0u, o);
                                    }
                                } else {
#pragma unroll
                                    for (int k = 0; k < WT; ++k)
                                        buffer_store1(rv, (pos * WT + k) * 4u,
                                                      __float_as_uint(cc == 0 ? x[k].x : cc == 1 ? x[k].y : cc == 2 ? x[k].z : x[k].w));
                                }
                                ++pos;
                            }
                        }
                    }
                    if (lane < padded - total) {          // fill the round's last line
#pragma unroll
                        for (int k = 0; k < WT; ++k) buffer_store1(rv, ((spec_run + total + lane) * WT + k) * 4u, 0u);
                    }
                    spec_run += padded;
                }
            }
        }
    }
    __syncthreads();
    flush_hist(h, NB, hist + (size_t)cur_seg * H_STRIDE + H_L0);
}

// ---------------------------------------------------------------------------------------
// K1 for a flat model whose arrays are 16-byte aligned: the same results as k_score, with
// the loads of the NEXT round of 256 parameters per wave (the next tile's first round after
// a tile's last) requested before the current round is worked on, so that a wave always has
// two rounds of W + 1 16-byte loads in flight, also while it draws explorer zones.  Whole
// arrays are addressed by a scalar base (the stores by a descriptor) and one 32-bit lane offset
// for all of them (n < 2^30 parameters: byte offsets fit); block b takes the whole tiles b, b + gridDim.x, ...; the ragged last tile, if any,
// goes to one block after its loop, element by element.
// 1 to 8 and 16 workers come here (16 with two parts of capture staging and no round keys in registers), because a
// selection then finds its candidates sorted: k_core_build falls from 209 to 14 us at 138*10^6 parameters and 16 workers
// (scoring with draws and capture itself 2,558 -> 2,190 us), from 50 to 12 us at 20*10^6 and 3 workers (94 -> 82 us).
// 9 to 15 would fit as well: they have no instantiation (six each, in a library that takes over a minute to compile) and
// pay for it with k_score and a second pass over the scores (20*10^6 parameters: 308 us with 9 workers, 304 here with
// 16).  More than 16 do not fit: two rounds of 18 vectors alone are 144 registers beside the ones the pass needs.
// ---------------------------------------------------------------------------------------
#ifndef SCOREF_MINB
#define SCOREF_MINB 2
#endif
#ifndef SCOREF_LD_AUX
#define SCOREF_LD_AUX 2
#endif
#ifndef SCOREF_ST_AUX
#define SCOREF_ST_AUX 2
#endif
#ifndef SCOREF_CAP_AUX
#define SCOREF_CAP_AUX 2
#endif
// cls.pred[0] != NONE: every whole tile is also sorted against that predicted level-0 threshold bin, exactly as
// k_core_build would do it once the bin is known (certain bitmap, candidate bitmap, candidate keys compacted per
// sub-tile, counts): if the histogram then confirms the bin, the selection need not read the scores again.
struct ClsArgs {
    const uint32_t* pred;
    uint32_t* used;          // [0]: the bin this launch classified against (NONE: it did not)
    int mode;                // 1: pred[0]; test switches: 0 never classify, 2 take the bin above the prediction (always wrong)
    uint32_t *gt_bits, *cand_bits, *cand_keys, *cnt_gt, *cnt_cand;
};
template <int WT, int PRE, int SPEC, int DENSE>
__global__ __launch_bounds__(BLOCK, SCOREF_MINB) void k_score_flat(const float* __restrict__ w, PtrTab g, float c,
                                                                   float* __restrict__ S, uint64_t n, uint32_t* __restrict__ hist,
                                                                   PreArgs pre, SpecArgs spec, ClsArgs cls, float* __restrict__ w_new, float lr)
{
    static_assert(WT >= 1 && WT <= 16, "two rounds of W + 1 vectors must fit the registers");
    constexpr uint32_t STAGED = WT <= 8 ? 256 : 128;      // captured entries staged at a time: two blocks share a unit's LDS
    static_assert(!(SPEC && DENSE), "a dense update is never followed by a pack of the same updates");
    constexpr uint32_t NB = CORE_NB0 / 2;
    __shared__ uint32_t h[NB];
    __shared__ __align__(16) float stage[SPEC ? 4 * STAGED * WT : 4];
    __shared__ uint32_t h1[CORE_NB1];                // level-1 digits of the candidates of the predicted bin
    const uint32_t lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t T_full = (uint32_t)(n / TILE), T = (uint32_t)((n + TILE - 1) / TILE);
    for (uint32_t b = threadIdx.x; b < NB; b += BLOCK) h[b] = 0;
    for (uint32_t b = threadIdx.x; b < CORE_NB1; b += BLOCK) h1[b] = 0;
    __syncthreads();
    const uint32_t bytes = (uint32_t)(n * 4u);
    const __amdgpu_buffer_rsrc_t rS = buffer_of(S, bytes), rn = buffer_of(DENSE ? w_new : S, bytes);
    uint32_t pre_bound = 0, pre_sure = 0, pre_has_sure = 0, pre_skip = 1;
    if (PRE) {
        const SegState* st = &pre.states[0];
        pre_bound = st->bound_m1; pre_sure = st->sure_m1; pre_has_sure = st->has_gt; pre_skip = st->need0 == 0;
    }
    uint32_t spec_lo = 0xFFFFFFFFu;
    if (SPEC) spec_lo = spec.lo[0];
    uint32_t b1 = cls.mode ? cls.pred[0] : NONE;     // predicted threshold bin, NONE: no prediction
    if (cls.mode == 2 && b1 != NONE) b1 += 1u;
    if (blockIdx.x == 0 && threadIdx.x == 0) cls.used[0] = b1;
    uint32_t crun = 0, ngt = 0, gw[4], cw[4];
    // byte offset of this lane's vector in round r of this wave's sub-tile of tile t
    auto voff = [&](uint32_t t, uint32_t r) { return (t * TILE + wid * SUB + r * 256u) * 4u + lane * 16u; };
    // a scalar base and a 32-bit lane offset (whole arrays are below 2^32 bytes): a descriptor would take four scalar registers
    // of each array, and they are short here
    auto fetch = [&](float4 (&x)[WT + 1], uint32_t t, uint32_t r) {
        const uint32_t o = voff(t, r);
        x[WT] = ld4<1>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(w) + o));
#pragma unroll
        for (int k = 0; k < WT; ++k) x[k] = ld4<1>(reinterpret_cast<const float*>(static_cast<const char*>(g.p[k]) + o));
    };
    // PRE = 3 (pre.slots is not zero): a round draws its own 256 parameters for every worker, so that the flags meet the update
    // values in registers; otherwise a round draws the whole sub-tile for its share of the workers
    constexpr bool KEEP_EXPL = PRE == 3;
    constexpr int PAIRS_W = (WT + 1) / 2;
    constexpr bool PACK_FILL = WT > 8;           // the workers' fill counts as bytes: registers are short there
    __shared__ __align__(16) float estage[KEEP_EXPL ? 4 * WT * EXPL_SLOTS_MAX : 4];
    uint32_t esure[KEEP_EXPL ? PAIRS_W : 1], efill[KEEP_EXPL ? (PACK_FILL ? WT / 4 : WT) : 1];
    uint32_t ecount = 0;                         // lane b: candidates of worker b in this sub-tile
    // 14 and 16 registers from a tile's first round to its last; with 16 workers' rounds beside them they would spill: the
    // keys are computed anew and the lanes' part waits in LDS
    constexpr bool HELD = WT <= 8;
    __shared__ uint4 parked[PRE && !HELD && !KEEP_EXPL ? 4 : 1][PRE && !HELD && !KEEP_EXPL ? 256 : 1];
    PhiloxRoundKeys rkeys;
    DrawLanes lanes;
    if constexpr (PRE && HELD) rkeys = philox_round_keys<true>(pre.pk.seed_lo, pre.pk.seed_hi);
    auto out_of = [&](uint32_t b) {
        DrawOut out;
        out.sure_bits = pre.sure_bits + (size_t)b * T * TILE_WORDS;
        out.cand_bits = pre.cand_bits + (size_t)b * T * TILE_WORDS;
        out.cand_keys = pre.cand_keys + (size_t)b * pre.keys_stride;
        out.cnt_cand = pre.cnt_cand + (size_t)b * T * SUBS;
        return out;
    };
    auto draw = [&](uint32_t t, uint32_t len, uint32_t r) {      // this round's share of the announced draws
        if (PRE && r < pre.nw) {
            PhiloxKey pk = pre.pk;
            if constexpr (!HELD) {
                asm volatile("" : "+s"(pk.seed_lo), "+s"(pk.seed_hi));
                rkeys = philox_round_keys<false>(pk.seed_lo, pk.seed_hi);
            }
            if (r == 0) {
                const DrawLanes d = draw_lanes(t * TILE, wid, pk);
                if constexpr (HELD) lanes = d;
                else park_lanes(parked[wid], d);
            }
#pragma unroll 1
            for (uint32_t b = r; b < pre.nw; b += 4) {
                const DrawOut out = out_of(b);
                if constexpr (HELD)
                    explore_subtile<(PRE >= 2) ? 1 : 0, 0>(pre.worker0 + b, t, wid, t * TILE, len, pre_bound, pre_sure,
                                                             pre_has_sure, pre_skip, out, pk, rkeys, lanes);
                else
                    explore_subtile<(PRE >= 2) ? 1 : 0, 0>(pre.worker0 + b, t, wid, t * TILE, len, pre_bound, pre_sure,
                                                             pre_has_sure, pre_skip, out, pk, rkeys, ParkedLanes{parked[wid]});
            }
        }
    };
    // One round of a whole tile for every worker that is scored.  A lane with a sure parameter among its four leaves the
    // first one's update value in the worker's line of the wave's stage, lanes in order: about 20 values a sub-tile at the
    // paper's ratio; 3 % of the sure ones are not the first in their lane and are not kept.  Two workers at a time: the
    // chains of multiplications are long, and eight waves to a unit leave little else to fill them with.  (One worker, the only
    // odd number that has a capture, is kept for by option "explore_keep" = 2 alone.)
    auto draw_round = [&](float4 (&x)[WT + 1], uint32_t t, uint32_t r) {
        PhiloxKey pk = pre.pk;
        uint32_t worker0 = pre.worker0;
        asm volatile("" : "+s"(worker0));                        // the workers' scalars are computed anew, not kept
        if constexpr (!HELD) {
            asm volatile("" : "+s"(pk.seed_lo), "+s"(pk.seed_hi));
            rkeys = philox_round_keys<false>(pk.seed_lo, pk.seed_hi);
        }
        const PhiloxCommon c = philox_common(((t * TILE + wid * SUB) >> 2) + r * 64u + lane, pk.it_lo, pk.it_hi, pk.seed_lo, pk.seed_hi);
        const uint32_t sure_excl = pre_has_sure ? pre_sure + 1u : 0u, width_m1 = pre_bound - sure_excl;
        float* es = estage + wid * (WT * EXPL_SLOTS_MAX);
        auto candidates = [&](int b, const uint32_t (&d)[4]) {      // rare
            uint32_t* slot = pre.cand_keys + (size_t)b * pre.keys_stride + ((size_t)t * SUBS + wid) * PAIR_SLOT;
            uint32_t e0 = d[0], e1 = d[1], e2 = d[2], e3 = d[3];
#pragma unroll 1
            for (uint32_t k = 0; k < 4; ++k) {
                const uint64_t bal = __ballot(e0 <= width_m1);
                const uint32_t before = __builtin_amdgcn_readlane(ecount, b);
                const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, before));
                if (e0 <= width_m1 && pos < PAIR_CAP) { slot[2u * pos] = width_m1 - e0; slot[2u * pos + 1u] = r * 256u + lane * 4u + k; }
                if (lane == (uint32_t)b) ecount += (uint32_t)__popcll(bal);
                e0 = e1; e1 = e2; e2 = e3;
            }
        };
        auto keep = [&](int b, const Masks4& m) {
            const uint64_t any = (m.m0 | m.m1) | (m.m2 | m.m3);
            const uint32_t fill = PACK_FILL ? (efill[b / 4] >> (8 * (b % 4))) & 0xFFu : efill[b];
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, fill));
            const float v = first_masked(x[b], m);
            if (__builtin_amdgcn_inverse_ballot_w64(any) && at < pre.slots) es[(uint32_t)b * EXPL_SLOTS_MAX + at] = v;
            uint32_t& f = efill[PACK_FILL ? b / 4 : b];
            f += (uint32_t)__popcll(any) << (PACK_FILL ? 8 * (b % 4) : 0);
            asm("" : "+v"(f));                                    // in a vector register: the scalar ones are short
        };
#pragma unroll
        for (int p = 0; p < PAIRS_W; ++p) {
            const int A = 2 * p, B = 2 * p + 1 < WT ? 2 * p + 1 : A;
            if (r == 0) {
                esure[p] = 0;
                if (PACK_FILL) { if (p % 2 == 0) efill[p / 2] = 0; }
                else { efill[A] = 0; efill[B] = 0; }
            }
            uint32_t wa[4], wb[4], da[4], db[4];
            philox_words(c, philox_worker(worker0 + A, pk.it_lo, pk.seed_lo), rkeys, wa);
            philox_words(c, philox_worker(worker0 + B, pk.it_lo, pk.seed_lo), rkeys, wb);
            const Masks4 ma = sub4_borrow(wa, sure_excl, da, esure[p]);
            uint32_t dmin = min(min(da[0], da[1]), min(da[2], da[3]));
            Masks4 mb = ma;
            if (B != A) {
                mb = sub4_borrow(wb, sure_excl, db, esure[p]);
                dmin = min(dmin, min(min(db[0], db[1]), min(db[2], db[3])));
            } else esure[p] <<= 4;
            if (__ballot(dmin <= width_m1) != 0ull) {             // uniform
                candidates(A, da);
                if (B != A) candidates(B, db);
            }
            // Always so; as a branch, which sets these steps apart from the products of the next pair: 138*10^6 parameters, 8 workers
            // 1,202 us, 1,213 without, but 64*10^6, 2 234 and 227, 32*10^6, 4 172 and 168; 16 alike.
            if (WT < 8 || pre.slots != 0) {
                keep(A, ma);
                if (B != A) keep(B, mb);
            }
        }
        if (r == 3) {
            // every worker's 32 bitmap words through the wave's (now idle) stage of the core capture: whole lines
            uint32_t* sb = reinterpret_cast<uint32_t*>(stage + wid * (STAGED * WT));
            wave_sync();
#pragma unroll
            for (int p = 0; p < PAIRS_W; ++p) {
                const uint32_t v = __brev(esure[p]);             // bit 8 * round + 4 * (second worker) + component
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (2 * p + h >= WT) continue;
                    const uint32_t word = transpose_spread((v >> (4 * h)) & 0x0F0F0F0Fu);
                    if ((lane & 1u) == 0) sb[(2 * p + h) * SUB_WORDS + 4u * (lane & 6u) + (lane >> 3)] = word;      // word 8 * round + j
                }
            }
            wave_sync();
#pragma unroll
            for (int p = 0; p < PAIRS_W; ++p) {
                const uint32_t b = 2u * p + (lane >> 5);
                if (b < (uint32_t)WT) pre.sure_bits[((size_t)b * T + t) * TILE_WORDS + wid * SUB_WORDS + (lane & 31u)] = sb[p * 64 + lane];
            }
            if (lane < (uint32_t)WT) pre.cnt_cand[((size_t)lane * T + t) * SUBS + wid] = ecount;
            ecount = 0;
            const __amdgpu_buffer_rsrc_t rv = buffer_of(pre.vals + ((size_t)t * SUBS + wid) * WT * pre.slots, WT * pre.slots * 4u);
            const bool few = pre.slots == EXPL_SLOTS_FEW;         // 16-byte pieces: the worker and the piece of its line
            for (uint32_t k = lane; k < WT * pre.slots / 4u; k += 64) {
                const uint32_t b = few ? k / (EXPL_SLOTS_FEW / 4u) : k / (EXPL_SLOTS_MAX / 4u);
                buffer_store4_aux<SCOREF_CAP_AUX>(rv, k * 16u, *reinterpret_cast<const float4*>(es + b * EXPL_SLOTS_MAX + (k - b * (pre.slots / 4u)) * 4u));
            }
            wave_sync();
        }
    };
    uint32_t spec_run = 0;
    uint2 bw[4];
    auto work = [&](float4 (&x)[WT + 1], uint32_t t, uint32_t r) {
        const uint32_t o = voff(t, r);
        float4 a = x[0];
#pragma unroll
        for (int k = 1; k < WT; ++k) { a.x = a.x + x[k].x; a.y = a.y + x[k].y; a.z = a.z + x[k].z; a.w = a.w + x[k].w; }
        float4 wv = x[WT];
        if (DENSE) {
            wv.x = __builtin_fmaf(-lr, a.x + 0.0f, wv.x); wv.y = __builtin_fmaf(-lr, a.y + 0.0f, wv.y);
            wv.z = __builtin_fmaf(-lr, a.z + 0.0f, wv.z); wv.w = __builtin_fmaf(-lr, a.w + 0.0f, wv.w);
            buffer_store4_aux<0>(rn, o, wv);
        }
        float4 sc;
        sc.x = significance(wv.x, a.x, c); sc.y = significance(wv.y, a.y, c);
        sc.z = significance(wv.z, a.z, c); sc.w = significance(wv.w, a.w, c);
        buffer_store4_aux<SCOREF_ST_AUX>(rS, o, sc);
        atomicAdd(&h[(__float_as_uint(sc.x) >> CORE_SHIFT0) & (NB - 1u)], 1u);
        atomicAdd(&h[(__float_as_uint(sc.y) >> CORE_SHIFT0) & (NB - 1u)], 1u);
        atomicAdd(&h[(__float_as_uint(sc.z) >> CORE_SHIFT0) & (NB - 1u)], 1u);
        atomicAdd(&h[(__float_as_uint(sc.w) >> CORE_SHIFT0) & (NB - 1u)], 1u);
        if (b1 != NONE) {                            // uniform
            if (r == 0) { crun = 0; ngt = 0; }
            const uint32_t d0 = __float_as_uint(sc.x) >> CORE_SHIFT0, d1 = __float_as_uint(sc.y) >> CORE_SHIFT0,
                           d2 = __float_as_uint(sc.z) >> CORE_SHIFT0, d3 = __float_as_uint(sc.w) >> CORE_SHIFT0;
            const uint32_t fg = (d0 > b1 ? 1u : 0u) | (d1 > b1 ? 2u : 0u) | (d2 > b1 ? 4u : 0u) | (d3 > b1 ? 8u : 0u);
            const uint32_t fc = (d0 == b1 ? 1u : 0u) | (d1 == b1 ? 2u : 0u) | (d2 == b1 ? 4u : 0u) | (d3 == b1 ? 8u : 0u);
            gw[r] = or_reduce8(fg << (4u * (lane & 7u)));
            cw[r] = or_reduce8(fc << (4u * (lane & 7u)));
            ngt += __popc(fg);
            if (__ballot(fc != 0u) != 0ull) {
                uint32_t below = 0, total = 0;
#pragma unroll
                for (int cc = 0; cc < 4; ++cc) {
                    const unsigned long long bal = __ballot((fc >> cc) & 1u);
                    below += __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                    total += (uint32_t)__popcll(bal);
                }
                if (fc) {
                    const __amdgpu_buffer_rsrc_t rk = buffer_of(cls.cand_keys + (size_t)t * TILE + wid * SUB, SUB * 4u);
                    uint32_t pos = crun + below;
                    if (fc & 1u) { buffer_store1(rk, 4u * pos++, __float_as_uint(sc.x)); atomicAdd(&h1[(__float_as_uint(sc.x) >> CORE_SHIFT1) & (CORE_NB1 - 1u)], 1u); }
                    if (fc & 2u) { buffer_store1(rk, 4u * pos++, __float_as_uint(sc.y)); atomicAdd(&h1[(__float_as_uint(sc.y) >> CORE_SHIFT1) & (CORE_NB1 - 1u)], 1u); }
                    if (fc & 4u) { buffer_store1(rk, 4u * pos++, __float_as_uint(sc.z)); atomicAdd(&h1[(__float_as_uint(sc.z) >> CORE_SHIFT1) & (CORE_NB1 - 1u)], 1u); }
                    if (fc & 8u) { buffer_store1(rk, 4u * pos, __float_as_uint(sc.w)); atomicAdd(&h1[(__float_as_uint(sc.w) >> CORE_SHIFT1) & (CORE_NB1 - 1u)], 1u); }
                }
                crun += total;
            }
            if (r == 3) {          // the sub-tile's 32 + 32 bitmap words as whole lines, its two counts
                const int src = (int)(8u * (lane & 7u));
                uint32_t og = 0, oc = 0;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const uint32_t xg = __shfl(gw[rr], src, 64), xc = __shfl(cw[rr], src, 64);
                    if ((lane >> 3) == (uint32_t)rr) { og = xg; oc = xc; }
                }
                const size_t wbase = (size_t)t * TILE_WORDS + wid * SUB_WORDS;
                if (lane < SUB_WORDS) { cls.gt_bits[wbase + lane] = og; cls.cand_bits[wbase + lane] = oc; }
                const uint32_t ng = wave_sum(ngt);
                if (lane == 0) { cls.cnt_cand[(size_t)t * SUBS + wid] = crun; cls.cnt_gt[(size_t)t * SUBS + wid] = ng; }
            }
        }
        if (SPEC) {
            if (r == 0) spec_run = 0;
            const uint32_t f = (__float_as_uint(sc.x) >= spec_lo ? 1u : 0u) | (__float_as_uint(sc.y) >= spec_lo ? 2u : 0u) |
                               (__float_as_uint(sc.z) >= spec_lo ? 4u : 0u) | (__float_as_uint(sc.w) >= spec_lo ? 8u : 0u);
            const uint32_t v = or_reduce8(f << (4u * (lane & 7u)));
            uint32_t below = 0, total = 0;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const unsigned long long bal = __ballot((f >> cc) & 1u);
                below += __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                total += (uint32_t)__popcll(bal);
            }
            // bitmap words with their entry numbers: lane 8j holds word j of this round; after the sub-tile's last
            // round lanes 0..31 write all 32 of them at once (two whole lines)
            bw[r] = make_uint2(v, spec_run + below);
            if (r == 3) {
                const int src = (int)(8u * (lane & 7u));
                uint2 o = make_uint2(0u, 0u);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const uint32_t ox = __shfl(bw[rr].x, src, 64), oy = __shfl(bw[rr].y, src, 64);
                    if ((lane >> 3) == (uint32_t)rr) o = make_uint2(ox, oy);
                }
                if (lane < SUB_WORDS) spec.bits[(size_t)t * TILE_WORDS + wid * SUB_WORDS + lane] = o;
            }
            constexpr uint32_t A = spec_align(WT);
            const uint32_t padded = (total + A - 1u) & ~(A - 1u);
            // the round's entries go through the wave's staging area in LDS, so that every 128-byte line of the capture is
            // written by one store instruction, whole (a line written piecewise by several instructions can leave the
            // cache half-written and costs a read-modify-write in memory)
            float* stf = stage + wid * (STAGED * WT);
            auto part = [&](uint32_t eb) {            // entries eb .. eb + STAGED - 1 of the round
                if (f) {
                    uint32_t pos = below - eb;
#pragma unroll
                    for (int cc = 0; cc < 4; ++cc) {
                        if ((f >> cc) & 1u) {
                            if (STAGED < 256 && pos >= STAGED) {
                                // in another part
                            } else if (WT >= 4 && WT % 4 == 0) {
#pragma unroll
                                for (int k = 0; k < WT; k += 4) {
                                    float4 q;
                                    q.x = cc == 0 ? x[k].x : cc == 1 ? x[k].y : cc == 2 ? x[k].z : x[k].w;
                                    q.y = cc == 0 ? x[k + 1].x : cc == 1 ? x[k + 1].y : cc == 2 ? x[k + 1].z : x[k + 1].w;
                                    q.z = cc == 0 ? x[k + 2].x : cc == 1 ? x[k + 2].y : cc == 2 ? x[k + 2].z : x[k + 2].w;
                                    q.w = cc == 0 ? x[k + 3].x : cc == 1 ? x[k + 3].y : cc == 2 ? x[k + 3].z : x[k + 3].w;
                                    *reinterpret_cast<float4*>(stf + pos * WT + k) = q;
                                }
                            } else {
#pragma unroll
                                for (int k = 0; k < WT; ++k)
                                    stf[pos * WT + k] = cc == 0 ? x[k].x : cc == 1 ? x[k].y : cc == 2 ? x[k].z : x[k].w;
                            }
                            ++pos;
                        }
                    }
                }
                if (lane < padded - total && (STAGED == 256 || total + lane - eb < STAGED)) {      // fill the round's last line
#pragma unroll
                    for (int k = 0; k < WT; ++k) stf[(total + lane - eb) * WT + k] = 0.0f;
                }
                wave_sync();
                const __amdgpu_buffer_rsrc_t rv = buffer_of(spec.vals + ((size_t)t * SUBS + wid) * SPEC_CAP * WT, SPEC_CAP * WT * 4u);
                const uint32_t nchunk = min(padded - eb, STAGED) * WT / 4u;          // 16-byte pieces: a multiple of 8 (whole lines)
                for (uint32_t cidx = lane; cidx < nchunk; cidx += 64)
                    buffer_store4_aux<SCOREF_CAP_AUX>(rv, (spec_run + eb) * WT * 4u + cidx * 16u, *reinterpret_cast<const float4*>(stf + cidx * 4u));
                wave_sync();
            };
            part(0);
            if (STAGED < 256 && padded > STAGED) part(STAGED);       // uniform
            spec_run += padded;
        }
    };
    float4 xa[WT + 1], xb[WT + 1];
    uint32_t t = blockIdx.x;
    if (t < T_full) fetch(xa, t, 0);
#pragma unroll 1
    for (; t < T_full; t += gridDim.x) {
        const uint32_t tn = t + gridDim.x;
        if constexpr (KEEP_EXPL) {
            fetch(xb, t, 1); draw_round(xa, t, 0); work(xa, t, 0);
            fetch(xa, t, 2); draw_round(xb, t, 1); work(xb, t, 1);
            fetch(xb, t, 3); draw_round(xa, t, 2); work(xa, t, 2);
            if (tn < T_full) fetch(xa, tn, 0);
            draw_round(xb, t, 3); work(xb, t, 3);
        } else {
            fetch(xb, t, 1); draw(t, TILE, 0); work(xa, t, 0);
            fetch(xa, t, 2); draw(t, TILE, 1); work(xb, t, 1);
            fetch(xb, t, 3); draw(t, TILE, 2); work(xa, t, 2);
            if (tn < T_full) fetch(xa, tn, 0);
            draw(t, TILE, 3); work(xb, t, 3);
        }
    }
    // the ragged last tile
    if (T != T_full && blockIdx.x == T_full % gridDim.x) {
        const uint32_t start = T_full * TILE, len = (uint32_t)(n - start);
        const uint32_t lo = wid * SUB, hi = (lo + SUB < len) ? lo + SUB : len;
        for (uint32_t l = lo + lane; l < hi; l += 64) {
            const size_t e = (size_t)start + l;
            float a = static_cast<const float*>(g.p[0])[e];
#pragma unroll
            for (int k = 1; k < WT; ++k) a = a + static_cast<const float*>(g.p[k])[e];
            float we = w[e];
            if (DENSE) { we = __builtin_fmaf(-lr, a + 0.0f, we); w_new[e] = we; }
            const float sc = significance(we, a, c);
            S[e] = sc;
            atomicAdd(&h[(__float_as_uint(sc) >> CORE_SHIFT0) & (NB - 1u)], 1u);
        }
        if constexpr (!KEEP_EXPL)
            for (uint32_t r = 0; r < 4; ++r) draw(T_full, len, r);
    }
    // the ragged tile, and workers announced beyond those scored: a whole sub-tile of a worker at a time, nothing kept
    if constexpr (KEEP_EXPL) {
        const PhiloxRoundKeys rk = philox_round_keys<false>(pre.pk.seed_lo, pre.pk.seed_hi);
        for (uint32_t tt = pre.nw > (uint32_t)WT ? blockIdx.x : (blockIdx.x == T_full % gridDim.x ? T_full : T); tt < T; tt += gridDim.x) {
            const DrawLanes d = draw_lanes(tt * TILE, wid, pre.pk);
            const uint32_t len = tt < T_full ? TILE : (uint32_t)(n - (uint64_t)T_full * TILE);
#pragma unroll 1
            for (uint32_t b = tt < T_full ? (uint32_t)WT : 0u; b < pre.nw; ++b)
                explore_subtile<1, 0>(pre.worker0 + b, tt, wid, tt * TILE, len, pre_bound, pre_sure, pre_has_sure, pre_skip, out_of(b), pre.pk, rk, d);
        }
    }
    __syncthreads();
    flush_hist(h, NB, hist + H_L0);
    if (b1 != NONE) flush_hist(h1, CORE_NB1, hist + H_L1);
}

// ---------------------------------------------------------------------------------------
// Capture bound without an earlier selection (flat model): a sample of the significances about
// to be computed gives an estimate of the coming threshold.  k_sample_keys scores SAMPLE_PER
// consecutive parameters of every full tile, at a tile-dependent offset; k_sample_bound (one
// block) finds the sample's need-th largest key by a two-level radix descent (12 + 12 bits:
// 2^7 units in the last place) and writes it, less a margin, as the capture bound.  An
// estimate that turns out too high is caught by the selection's own verdict (the pack then
// gathers); one that is too low only makes the capture larger.
// ---------------------------------------------------------------------------------------
constexpr uint32_t SAMPLE_PER = 2;
constexpr uint32_t SAMPLE_MARGIN = 1u << 18;
__global__ __launch_bounds__(256) void k_sample_keys(const float* __restrict__ w, PtrTab g, int W, float c, uint32_t T_full,
                                                     uint32_t* __restrict__ keys)
{
    const uint32_t x = blockIdx.x * 256 + threadIdx.x;
    if (x >= T_full * SAMPLE_PER) return;
    const uint32_t t = x / SAMPLE_PER, j = x % SAMPLE_PER;
    const uint32_t off = ((t * 0x9E3779B1u) >> 21) * SAMPLE_PER;       // 0 .. 4094 in steps of 2: inside the tile
    const size_t i = (size_t)t * TILE + off + j;
    float a = static_cast<const float*>(g.p[0])[i];
    for (int k = 1; k < W; ++k) a = a + static_cast<const float*>(g.p[k])[i];
    keys[x] = __float_as_uint(significance(w[i], a, c));
}

// bias: test switch, added to the bound (in units of the last place, clamped).
__global__ __launch_bounds__(1024) void k_sample_bound(const uint32_t* __restrict__ keys, uint32_t N, uint32_t need,
                                                       long long bias, uint32_t* __restrict__ lo, uint32_t* __restrict__ pred)
{
    __shared__ uint32_t h[4096];
    __shared__ uint32_t wtot[16];
    __shared__ uint32_t sh[2];
    const uint32_t tid = threadIdx.x;
    if (need == 0 || need > N) { if (tid == 0) { lo[0] = NONE; pred[0] = NONE; } return; }   // nothing to estimate, nothing captured
    uint32_t prefix = 0, want = need;
#pragma unroll 1
    for (int level = 0; level < 2; ++level) {
        for (uint32_t b = tid; b < 4096; b += 1024) h[b] = 0;
        __syncthreads();
        for (uint32_t x = tid; x < N; x += 1024) {
            const uint32_t key = keys[x];
            if (level == 0) atomicAdd(&h[(key >> 19) & 4095u], 1u);
            else if ((key >> 19) == prefix) atomicAdd(&h[(key >> 7) & 4095u], 1u);
        }
        __syncthreads();
        // four bins per thread, from the largest digit down
        uint32_t cnt[4], sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) { cnt[e] = h[4095u - (tid * 4u + e)]; sum += cnt[e]; }
        uint32_t total;
        const uint32_t excl = block_excl_scan<16>(sum, wtot, total);
        if (excl < want && want <= excl + sum) {
            uint32_t run = excl;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (run < want && want <= run + cnt[e]) { sh[0] = 4095u - (tid * 4u + e); sh[1] = want - run; }
                run += cnt[e];
            }
        }
        __syncthreads();
        prefix = (level == 0) ? sh[0] : ((prefix << 12) | sh[0]);
        want = sh[1];
        __syncthreads();
    }
    if (tid == 0) {
        const long long tau = (long long)(prefix << 7);
        long long b = tau - (long long)SAMPLE_MARGIN + bias;
        if (b < 0) b = 0;
        if (b > 0x7FFFFFFFll) b = 0x7FFFFFFFll;
        lo[0] = (uint32_t)b;
        pred[0] = prefix >> 12;          // the level-0 bin of the estimated threshold
    }
}

// With speculative packing on (next != nullptr) the last step of a core selection tells per segment whether the threshold
// fell below what the scoring pass captured (fail, against cur), and next becomes the capture bound of the next scoring
// pass: the new threshold less 2^17 units in the last place (0.8 % to 1.6 %).
struct SpecTau { const uint32_t* cur; uint32_t* next; uint32_t* fail; };
constexpr uint32_t SPEC_MARGIN = 1u << 17;

// Stand-alone draw over every (worker, tile); each wave owns one sub-tile of the block's tiles and draws it for per_group
// workers in turn.  grid (blocks, ceil(n_workers / per_group)).
template <int MIS, int PAIRS>
__global__ __launch_bounds__(BLOCK) void k_explore_keys(const uint32_t* __restrict__ tile_start,
                                                        const uint32_t* __restrict__ tile_seg, uint32_t T,
                                                        uint32_t n_seg, const SegState* __restrict__ states,
                                                        uint32_t* __restrict__ sure_bits, uint32_t* __restrict__ cand_bits,
                                                        uint32_t* __restrict__ cand_keys, uint32_t* __restrict__ cnt_cand,
                                                        uint64_t keys_stride, uint32_t worker0, uint32_t n_workers, uint32_t per_group,
                                                        PhiloxKey pk)
{
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b0 = blockIdx.y * per_group, b1 = min(b0 + per_group, n_workers);
    const uint32_t t0 = (uint32_t)((uint64_t)T * blockIdx.x / gridDim.x);
    const uint32_t t1 = (uint32_t)((uint64_t)T * (blockIdx.x + 1) / gridDim.x);
    const PhiloxRoundKeys rk = philox_round_keys<true>(pk.seed_lo, pk.seed_hi);
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t seg = (n_seg == 1) ? 0u : tile_seg[t];
        const SegState* st = &states[seg];                 // the same for every worker
        const uint32_t bound_m1 = st->bound_m1;
        const uint32_t sure_m1 = st->sure_m1, has_sure = st->has_gt;
        const uint32_t skip = st->need0 == 0;
        const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
        const DrawLanes lanes = draw_lanes(start, wid, pk);
#pragma unroll 1
        for (uint32_t b = b0; b < b1; ++b) {
            DrawOut out;
            out.sure_bits = sure_bits + (size_t)b * T * TILE_WORDS;
            out.cand_bits = cand_bits + (size_t)b * T * TILE_WORDS;
            out.cand_keys = cand_keys + (size_t)b * keys_stride;
            out.cnt_cand = cnt_cand + (size_t)b * T * SUBS;
            explore_subtile<PAIRS, MIS>(worker0 + b, t, wid, start, len, bound_m1, sure_m1, has_sure, skip, out, pk, rk, lanes);
        }
    }
}

// A wave walks one tile's candidates with every lane owning two bitmap words; the 16 lanes
// of a sub-tile find their place in that sub-tile's key list by a prefix inside the group.
__device__ __forceinline__ uint32_t sublist_pos(uint32_t lane, uint32_t my_count)
{
    const uint32_t excl = wave_incl_scan(my_count) - my_count;
    const uint32_t group0 = __shfl(excl, (int)(lane & ~15u), 64);
    return (lane >> 4) * SUB + (excl - group0);
}

// Where a tile is.  Flat model: no table look-ups, so that every load a tail kernel needs
// can be requested at once.
struct TileRef { uint32_t seg, start, len; };
__device__ __forceinline__ TileRef tile_ref(uint32_t t, uint32_t n_seg, uint64_t n, const uint32_t* __restrict__ tile_start,
                                            const uint32_t* __restrict__ tile_seg)
{
    TileRef r;
    if (n_seg == 1) {
        r.seg = 0; r.start = t * TILE;
        const uint64_t rest = n - (uint64_t)r.start;
        r.len = rest < TILE ? (uint32_t)rest : TILE;
    } else {
        r.seg = tile_seg[t]; r.start = tile_start[t]; r.len = tile_start[t + 1] - r.start;
    }
    return r;
}

// The first 16*KPL keys of each of a tile's four sub-lists, requested without waiting for
// the lists' lengths (the slots exist whatever the length; the unused ones are ignored):
// lane (s = lane/16, r = lane%16) holds entries r, r+16, ... of sub-list s.
template <int KPL>
__device__ __forceinline__ void load_sublists(const uint32_t* __restrict__ keys_tile, uint32_t lane, uint32_t kv[KPL])
{
    const uint32_t* p = keys_tile + (lane >> 4) * SUB + (lane & 15u);
#pragma unroll
    for (int i = 0; i < KPL; ++i) kv[i] = p[16 * i];
}

constexpr int CORE_KPL = 4;

// Bits [i0, i0 + 64) of a bitmap over all n parameters (i0 need not be word aligned).
__device__ __forceinline__ void bitmap_window(const uint32_t* __restrict__ bits, uint32_t n_words, uint32_t i0, uint32_t out[2])
{
    const uint32_t sh = i0 & 31u, wi = i0 >> 5;
    const uint32_t a0 = (wi < n_words) ? bits[wi] : 0u;
    const uint32_t a1 = (wi + 1 < n_words) ? bits[wi + 1] : 0u;
    const uint32_t a2 = (sh && wi + 2 < n_words) ? bits[wi + 2] : 0u;
    out[0] = sh ? ((a0 >> sh) | (a1 << (32u - sh))) : a0;
    out[1] = sh ? ((a1 >> sh) | (a2 << (32u - sh))) : a1;
}

// One tile's chosen parameters (two consecutive bitmap words a lane) as ascending indices at out[first] .., by one wave.
// Up to EMIT_STAGE of them are put in order in LDS (stage: half words, private to the wave) and leave as consecutive stores;
// written straight from the bits, a store instruction touched a line for every two to four lanes.  Core of 138*10^6
// parameters, 10 %: 55 -> 41 us; explorers of 20*10^6 for 3 workers, 17 %: 41 -> 17 us.
// Of a fuller tile every lane in turn shows its 64 bits to the wave, whose lanes write the positions set, side by side:
// 64 short steps, where a lane that walks its own bits takes up to 64 dependent ones for each of four fills of the stage.
// Explorer request of 138*10^6, 2 workers, 50 %: 942 us with a store per lane and bit, 543 through the stage, 537 so; of
// 10^6, 4 workers, 80 %: 163, 126, 107 us.
// limit: never beyond the caller's list.  All lanes call; incl: inclusive prefix of the lanes' numbers.
constexpr uint32_t EMIT_STAGE = 1024;
__device__ __forceinline__ void emit_indices(uint32_t w0, uint32_t w1, uint32_t incl, uint32_t start, uint32_t first, uint32_t limit,
                                             uint16_t* stage, uint32_t* __restrict__ out)
{
    const uint32_t lane = lane_id();
    const uint32_t total = last_lane(incl), excl = incl - __popc(w0) - __popc(w1);
    if (total > EMIT_STAGE) {                         // uniform
#pragma unroll 4
        for (uint32_t l = 0; l < 64; ++l) {
            const uint32_t lo = __builtin_amdgcn_readlane(w0, l), hi = __builtin_amdgcn_readlane(w1, l);
            const uint32_t at = first + __builtin_amdgcn_readlane(excl, l) + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
            if (((((uint64_t)hi << 32) | lo) >> lane) & 1u) { if (at < limit) out[at] = start + l * 64u + lane; }
        }
        return;
    }
    const uint32_t w[2] = {w0, w1};
    uint32_t o = excl;
    wave_sync();                                     // the previous tile's positions have been read
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
        uint32_t m = w[h];
        while (m) {
            const uint32_t p = __ffs(m) - 1;
            m &= m - 1;
            stage[o++] = (uint16_t)(lane * 64u + h * 32u + p);
        }
    }
    wave_sync();
    const uint32_t n_out = first < limit ? min(total, limit - first) : 0u;
    for (uint32_t x = lane; x < n_out; x += 64) out[first + x] = start + stage[x];
}

// Segmented models: the public bitmap is built from the index list (tiles may start inside a word).
__global__ __launch_bounds__(256) void k_bits_from_idx(const uint32_t* __restrict__ idx, uint64_t count, uint64_t n,
                                                       uint32_t* __restrict__ bits)
{
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < count; j += (uint64_t)gridDim.x * 256) {
        const uint32_t i = idx[j];
        if (i < n) atomicOr(&bits[i >> 5], 1u << (i & 31u));
    }
}

// ---------------------------------------------------------------------------------------
// Tile offsets of an ascending index list by binary search.  One thread per tile boundary.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tile_offsets(const uint32_t* __restrict__ idx, uint64_t count,
                                                      const uint32_t* __restrict__ tile_start, uint32_t T, uint64_t n,
                                                      uint32_t* __restrict__ off)
{
    const uint32_t t = blockIdx.x * 256 + threadIdx.x;
    if (t > T) return;
    const uint64_t target = (t == T) ? n : tile_start[t];
    uint64_t lo = 0, hi = count;                 // first position with idx >= target
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if ((uint64_t)idx[mid] < target) lo = mid + 1; else hi = mid;
    }
    off[t] = (uint32_t)lo;
}

// ---------------------------------------------------------------------------------------
// K5: pack (src_is_w == 0: the workers' updates) and the read half of pull (one shared
// source).  One block per tile; the tile's slice of every list is a short contiguous run,
// and the gathered lines of the source are shared by the core and explorer reads.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_gather(PtrTab src, int shared_src, uint32_t nw, uint64_t n,
                                                  const uint32_t* __restrict__ core_idx, const uint32_t* __restrict__ core_off,
                                                  PtrTab expl_idx, PtrTab expl_off, MutPtrTab core_val, MutPtrTab expl_val,
                                                  MutPtrTab scatter_dst)
{
    __shared__ uint32_t elo[MAXW], ecn[MAXW];
    const uint32_t t = blockIdx.x;
    // the tile's slices of all explorer lists are requested first, in one go (one list after the other would wait
    // for memory three times per worker)
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        const uint32_t lo = eo[t];
        elo[threadIdx.x] = lo;
        ecn[threadIdx.x] = eo[t + 1] - lo;
    }
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    for (uint32_t j = c0 + threadIdx.x; j < c1; j += BLOCK) {
        const uint32_t i = core_idx[j];
        if (i >= n) continue;
        if (shared_src) {
            const float v = static_cast<const float*>(src.p[0])[i];
            for (uint32_t q = 0; q < nw; ++q) {
                static_cast<float*>(core_val.p[q])[j] = v;
                if (scatter_dst.p[q]) static_cast<float*>(scatter_dst.p[q])[i] = v;
            }
        } else {
            for (uint32_t q0 = 0; q0 < nw; q0 += 8) {          // eight workers' loads together
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = (q0 + u < nw) ? static_cast<const float*>(src.p[q0 + u])[i] : 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) if (q0 + u < nw) static_cast<float*>(core_val.p[q0 + u])[j] = v[u];
            }
        }
    }
    __syncthreads();
    uint32_t E = 0;
    for (uint32_t q = 0; q < nw; ++q) E += ecn[q];
    for (uint32_t x0 = 0; x0 < E; x0 += 2 * BLOCK) {            // two entries per thread in flight
        uint32_t qq[2], jj[2], ii[2];
        float vv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t x = x0 + u * BLOCK + threadIdx.x;
            qq[u] = 0; jj[u] = 0; ii[u] = 0xFFFFFFFFu;
            if (x < E) {
                uint32_t q = 0, run = 0;
                while (q + 1 < nw && run + ecn[q] <= x) { run += ecn[q]; ++q; }
                qq[u] = q; jj[u] = elo[q] + (x - run);
                ii[u] = static_cast<const uint32_t*>(expl_idx.p[q])[jj[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            vv[u] = (ii[u] < n) ? static_cast<const float*>(src.p[shared_src ? 0 : qq[u]])[ii[u]] : 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (ii[u] >= n) continue;
            static_cast<float*>(expl_val.p[qq[u]])[jj[u]] = vv[u];
            float* sd = static_cast<float*>(scatter_dst.p[qq[u]]);
            if (sd) sd[ii[u]] = vv[u];
        }
    }
}

// ---------------------------------------------------------------------------------------
// Pack after a scoring pass that captured the update values of every parameter at or above
// spec_lo (k_score<.., SPEC = 1>): the core values of a captured tile come from the compact
// capture (rank of the parameter among the captured ones of its sub-tile), not from the
// update vectors.  Tiles that were not captured (ragged ones, or those of a segment whose
// threshold fell below the capture bound) gather from the update vectors.
// One wave per tile, all workers (the rank is the same for all); ceil(T/4) blocks.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void pack_core_spec(uint32_t block, const PtrTab& g, uint32_t nw, uint64_t n,
                                               const uint32_t* __restrict__ tile_start,
                                               const uint32_t* __restrict__ tile_seg, uint32_t T,
                                               const uint32_t* __restrict__ core_idx,
                                               const uint32_t* __restrict__ core_off,
                                               const uint2* __restrict__ spec_bits,
                                               const float* __restrict__ spec_vals,
                                               const uint32_t* __restrict__ spec_fail, const MutPtrTab& core_val)
{
    __shared__ uint32_t wd[4][TILE_WORDS], pre[4][TILE_WORDS];
    const uint32_t wid = threadIdx.x >> 6, t = block * 4 + wid, lane = lane_id();
    if (t >= T) return;
    const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
    const uint32_t j0 = core_off[t], j1 = core_off[t + 1];
    if (j0 >= j1) return;
    const bool captured = len == TILE && spec_fail[tile_seg[t]] == 0;
    if (captured) {
        // entry number of every captured parameter inside its sub-tile: lanes 4r..4r+3 hold the eight bitmap
        // words of round r (16 rounds a tile, 4 a sub-tile); a round's entries start on a multiple of A
        const uint32_t A = spec_align(nw);
        const uint4 w4 = *reinterpret_cast<const uint4*>(spec_bits + (size_t)t * TILE_WORDS + 2 * lane);
        const uint2 w2 = make_uint2(w4.x, w4.z);
        const uint32_t pc = __popc(w2.x) + __popc(w2.y);
        const uint32_t incl = wave_incl_scan(pc);
        const uint32_t round0 = __shfl(incl - pc, (int)(lane & ~3u), 64);                     // captured before this round
        const uint32_t round_total = __shfl(incl, (int)(lane | 3u), 64) - round0;
        const uint32_t round_padded = (round_total + A - 1u) & ~(A - 1u);
        const uint32_t pin = wave_incl_scan((lane & 3u) == 0 ? round_padded : 0u);            // padded rounds up to this one
        const uint32_t sub0 = __shfl(pin - ((lane & 3u) == 0 ? round_padded : 0u), (int)(lane & ~15u), 64);
        const uint32_t first = (__shfl(pin, (int)(lane & ~3u), 64) - round_padded) - sub0 + (incl - pc - round0);
        wd[wid][2 * lane] = w2.x; wd[wid][2 * lane + 1] = w2.y;
        pre[wid][2 * lane] = first; pre[wid][2 * lane + 1] = first + __popc(w2.x);
        wave_sync();
        // four list entries per lane and pass: all their index loads are requested first, then all their values
        constexpr int U = 4;
        for (uint32_t jb = j0; jb < j1; jb += 64 * U) {
            uint32_t e[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = jb + u * 64 + lane;
                e[u] = (j < j1) ? core_idx[j] - start : 0xFFFFFFFFu;       // beyond the tile: the caller's lists are inconsistent
            }
            if ((nw & 3u) == 0) {
                for (uint32_t q = 0; q < nw; q += 4) {
                    float4 v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (e[u] < TILE) {
                            const uint32_t entry = pre[wid][e[u] >> 5] + __popc(wd[wid][e[u] >> 5] & mask_below(e[u] & 31u));
                            if (entry < SPEC_CAP)
                                v[u] = *reinterpret_cast<const float4*>(spec_vals + (((size_t)t * SUBS + (e[u] >> 10)) * SPEC_CAP + entry) * nw + q);
                            else {
                                const size_t i = (size_t)start + e[u];
                                v[u].x = static_cast<const float*>(g.p[q])[i]; v[u].y = static_cast<const float*>(g.p[q + 1])[i];
                                v[u].z = static_cast<const float*>(g.p[q + 2])[i]; v[u].w = static_cast<const float*>(g.p[q + 3])[i];
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t j = jb + u * 64 + lane;
                        if (e[u] < TILE) {
                            static_cast<float*>(core_val.p[q])[j] = v[u].x; static_cast<float*>(core_val.p[q + 1])[j] = v[u].y;
                            static_cast<float*>(core_val.p[q + 2])[j] = v[u].z; static_cast<float*>(core_val.p[q + 3])[j] = v[u].w;
                        }
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t j = jb + u * 64 + lane;
                    if (e[u] >= TILE) continue;
                    const uint32_t entry = pre[wid][e[u] >> 5] + __popc(wd[wid][e[u] >> 5] & mask_below(e[u] & 31u));
                    const float* src = spec_vals + (((size_t)t * SUBS + (e[u] >> 10)) * SPEC_CAP + entry) * nw;
                    for (uint32_t q = 0; q < nw; ++q)
                        static_cast<float*>(core_val.p[q])[j] = (entry < SPEC_CAP) ? src[q] : static_cast<const float*>(g.p[q])[(size_t)start + e[u]];
                }
            }
        }
    } else {
        for (uint32_t j = j0 + lane; j < j1; j += 64) {
            const uint32_t i = core_idx[j];
            if (i >= n) continue;
            for (uint32_t q = 0; q < nw; ++q) static_cast<float*>(core_val.p[q])[j] = static_cast<const float*>(g.p[q])[i];
        }
    }
}

// The same for a flat model, one thread per list entry: the tile and the bitmap word follow
// from the index itself, the word's first entry number is stored beside the word.  Every wave
// writes 64 consecutive list positions per worker (whole, aligned lines: a store that covers
// a line only in part makes the memory side read it first).  Any number of blocks.
__device__ __forceinline__ void pack_core_flat(uint32_t block, uint32_t blocks, const PtrTab& g, uint32_t nw, uint64_t n, uint32_t T_full,
                                               const uint32_t* __restrict__ core_idx, uint32_t k,
                                               const uint2* __restrict__ spec_bits,
                                               const float* __restrict__ spec_vals,
                                               const uint32_t* __restrict__ spec_fail, const MutPtrTab& core_val)
{
    constexpr int U = 4;
    const bool ok = spec_fail[0] == 0;
    const uint32_t stride = blocks * 256u;
    for (uint32_t jb = block * 256u + threadIdx.x; jb < k; jb += U * stride) {
        uint32_t i[U];
#pragma unroll
        for (int u = 0; u < U; ++u) i[u] = (jb + u * stride < k) ? core_idx[jb + u * stride] : 0xFFFFFFFFu;
        uint2 bp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bp[u] = make_uint2(0u, 0u);
            if (i[u] < n && ok && (i[u] >> 12) < T_full) bp[u] = spec_bits[i[u] >> 5];      // tile * 128 + word in tile
        }
        if ((nw & 3u) == 0) {
            // eight workers (two 16-byte pieces of an entry) per turn, all loads of a turn requested before any store
            for (uint32_t q = 0; q < nw; q += 8) {
                float4 v[U][2];
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        v[u][h] = make_float4(0.f, 0.f, 0.f, 0.f);
                        const uint32_t qq = q + 4u * h;
                        if (i[u] >= n || qq >= nw) continue;
                        const uint32_t entry = bp[u].y + __popc(bp[u].x & mask_below(i[u] & 31u));
                        if (ok && (i[u] >> 12) < T_full && entry < SPEC_CAP) {
                            v[u][h] = ld4<NT_PACKC_LD>(spec_vals + ((size_t)(i[u] >> 10) * SPEC_CAP + entry) * nw + qq);
                        } else {
                            v[u][h].x = static_cast<const float*>(g.p[qq])[i[u]]; v[u][h].y = static_cast<const float*>(g.p[qq + 1])[i[u]];
                            v[u][h].z = static_cast<const float*>(g.p[qq + 2])[i[u]]; v[u][h].w = static_cast<const float*>(g.p[qq + 3])[i[u]];
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t j = jb + u * stride;
                    if (i[u] >= n) continue;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t qq = q + 4u * h;
                        if (qq >= nw) continue;
                        st1<NT_PACKC_ST>(static_cast<float*>(core_val.p[qq]) + j, v[u][h].x);
                        st1<NT_PACKC_ST>(static_cast<float*>(core_val.p[qq + 1]) + j, v[u][h].y);
                        st1<NT_PACKC_ST>(static_cast<float*>(core_val.p[qq + 2]) + j, v[u][h].z);
                        st1<NT_PACKC_ST>(static_cast<float*>(core_val.p[qq + 3]) + j, v[u][h].w);
                    }
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = jb + u * stride;
                if (i[u] >= n) continue;
                const uint32_t entry = bp[u].y + __popc(bp[u].x & mask_below(i[u] & 31u));
                if (ok && (i[u] >> 12) < T_full && entry < SPEC_CAP) {
                    const float* src = spec_vals + ((size_t)(i[u] >> 10) * SPEC_CAP + entry) * nw;
                    for (uint32_t q = 0; q < nw; ++q) static_cast<float*>(core_val.p[q])[j] = src[q];
                } else {
                    for (uint32_t q = 0; q < nw; ++q) static_cast<float*>(core_val.p[q])[j] = static_cast<const float*>(g.p[q])[i[u]];
                }
            }
        }
    }
}

// Explorer values by gathering from the update vectors: block `block` of `blocks` of worker q.
struct CountTab { uint32_t c[MAXW]; };
__device__ __forceinline__ void pack_expl_gather(uint32_t block, uint32_t blocks, uint32_t q, const PtrTab& g, uint64_t n, const PtrTab& expl_idx,
                                                 const CountTab& m_w, const MutPtrTab& expl_val)
{
    const uint32_t cnt = m_w.c[q];
    const float* src = static_cast<const float*>(g.p[q]);
    const uint32_t* idx = static_cast<const uint32_t*>(expl_idx.p[q]);
    float* out = static_cast<float*>(expl_val.p[q]);
    const uint32_t stride = blocks * 256u;
    for (uint32_t j = block * 256u + threadIdx.x; j < cnt; j += 4u * stride) {
        uint32_t i[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) i[u] = (j + u * stride < cnt) ? idx[j + u * stride] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = (j + u * stride < cnt && i[u] < n) ? ld1<NT_EXPLG>(src + i[u]) : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) if (j + u * stride < cnt) out[j + u * stride] = v[u];
    }
}

// Core values from the capture (the first core_blocks blocks) and explorer values by gathering (expl_blocks blocks a worker):
// either alone, or both in one launch where nothing has to be waited for in between.
template <int FLAT>
__global__ __launch_bounds__(BLOCK) void k_pack_spec(uint32_t core_blocks, uint32_t expl_blocks, PtrTab g, uint32_t nw, uint64_t n,
                                                     const uint32_t* __restrict__ tile_start, const uint32_t* __restrict__ tile_seg, uint32_t T,
                                                     const uint32_t* __restrict__ core_idx, const uint32_t* __restrict__ core_off, uint32_t k,
                                                     const uint2* __restrict__ spec_bits, const float* __restrict__ spec_vals,
                                                     const uint32_t* __restrict__ spec_fail, MutPtrTab core_val,
                                                     PtrTab expl_idx, CountTab m_w, MutPtrTab expl_val)
{
    if (blockIdx.x < core_blocks) {
        if (FLAT) pack_core_flat(blockIdx.x, core_blocks, g, nw, n, (uint32_t)(n / TILE), core_idx, k, spec_bits, spec_vals, spec_fail, core_val);
        else pack_core_spec(blockIdx.x, g, nw, n, tile_start, tile_seg, T, core_idx, core_off, spec_bits, spec_vals, spec_fail, core_val);
    } else {
        const uint32_t x = blockIdx.x - core_blocks;
        pack_expl_gather(x % expl_blocks, expl_blocks, x / expl_blocks, g, n, expl_idx, m_w, expl_val);
    }
}

// Explorer values from the scoring pass's capture.  A list entry is looked up by its own index: a parameter that is set in the
// draw's sure bitmap, is the first such of its block of four and lies within the slots was kept, whatever list names it;
// the others are gathered: of 2 % of the parameters 3.0 % that are not the first of their block and 0.03 % beyond the slots, 0.4 %
// chosen candidates, and the ragged tile.  A later request may have marked
// chosen candidates in the bitmap (or be about to): the slots of the draw's candidates name those bits, and they are taken out.
// One wave per tile and four workers, every load of a step requested for all four before any is used: a chain of three
// trips to memory.  grid (ceil(T / 4), ceil(nw / 4)).
constexpr int PEXP = 4;
__global__ __launch_bounds__(BLOCK) void k_pack_expl_spec(PtrTab g, uint32_t nw, uint64_t n, uint32_t T, uint32_t T_full, PtrTab expl_idx,
                                                          PtrTab expl_off, CountTab m_w, const uint32_t* __restrict__ sure_bits,
                                                          const uint32_t* __restrict__ pairs, uint64_t pair_stride,
                                                          const uint32_t* __restrict__ cnt_cand, const float* __restrict__ vals,
                                                          uint32_t slots, MutPtrTab expl_val)
{
    __shared__ uint32_t wd[4][PEXP][TILE_WORDS];
    __shared__ uint16_t pre[4][PEXP][TILE_WORDS];
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
    const uint32_t t = blockIdx.x * 4 + wid, q0 = blockIdx.y * PEXP;
    if (t >= T) return;
    const uint32_t start = t * TILE;
    uint32_t lo[PEXP], hi[PEXP], i0[PEXP], i1[PEXP], cc[PEXP];
    uint2 w2[PEXP];
#pragma unroll
    for (int u = 0; u < PEXP; ++u) {
        const uint32_t q = q0 + u;
        lo[u] = hi[u] = 0; w2[u] = make_uint2(0u, 0u); cc[u] = 0;
        if (q < nw) {
            const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[q]);
            lo[u] = eo[t]; hi[u] = min(eo[t + 1], m_w.c[q]);
            if (t < T_full) {
                w2[u] = *reinterpret_cast<const uint2*>(sure_bits + ((size_t)q * T + t) * TILE_WORDS + 2 * lane);
                cc[u] = cnt_cand[((size_t)q * T + t) * SUBS + (lane >> 4)];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < PEXP; ++u) {
        const uint32_t q = q0 + u, j = lo[u] + lane;
        i0[u] = i1[u] = 0xFFFFFFFFu;
        if (j < hi[u]) i0[u] = static_cast<const uint32_t*>(expl_idx.p[q])[j];
        if (j + 64u < hi[u]) i1[u] = static_cast<const uint32_t*>(expl_idx.p[q])[j + 64u];
        // a candidate of sub-tile lane / 16, if it has so many
        if ((lane & 15u) < cc[u]) cc[u] = (lane >> 4) * SUB + pairs[(size_t)q * pair_stride + ((size_t)t * SUBS + (lane >> 4)) * PAIR_SLOT + 2u * (lane & 15u) + 1u];
        else cc[u] = 0xFFFFFFFFu;
    }
#pragma unroll
    for (int u = 0; u < PEXP; ++u) *reinterpret_cast<uint2*>(&wd[wid][u][2 * lane]) = w2[u];
    wave_sync();
#pragma unroll
    for (int u = 0; u < PEXP; ++u)
        if (cc[u] < TILE) atomicAnd(&wd[wid][u][cc[u] >> 5], ~(1u << (cc[u] & 31u)));
    wave_sync();
    auto blocks_of = [](uint32_t w) { w |= w >> 1; w |= w >> 2; return w & 0x11111111u; };        // blocks of four with a bit set
#pragma unroll
    for (int u = 0; u < PEXP; ++u) {
        const uint2 w = *reinterpret_cast<const uint2*>(&wd[wid][u][2 * lane]);
        const uint32_t a = __popc(blocks_of(w.x)), s = a + __popc(blocks_of(w.y));
        const uint32_t excl = wave_incl_scan(s) - s, group0 = __shfl(excl, (int)(lane & ~15u), 64);
        pre[wid][u][2 * lane] = (uint16_t)(excl - group0);
        pre[wid][u][2 * lane + 1] = (uint16_t)(excl - group0 + a);
    }
    wave_sync();
    auto source = [&](int u, uint32_t i) -> const float* {
        const uint32_t q = q0 + u, pos = i - start;
        const float* src = static_cast<const float*>(g.p[q]) + i;
        if (pos < TILE) {
            const uint32_t w = wd[wid][u][pos >> 5], bit = pos & 31u;
            const uint32_t at = pre[wid][u][pos >> 5] + __popc(blocks_of(w) & mask_below(bit & 28u));
            // set, and no bit of its block of four below it
            if ((((w >> (bit & 28u)) & 15u) & ((2u << (bit & 3u)) - 1u)) == (1u << (bit & 3u)) && at < slots)
                src = vals + (((size_t)t * SUBS + (pos >> 10)) * nw + q) * slots + at;
        }
        return src;
    };
    float v0[PEXP], v1[PEXP];
#pragma unroll
    for (int u = 0; u < PEXP; ++u) {
        v0[u] = v1[u] = 0.0f;
        if (i0[u] < n) v0[u] = ld1<NT_EXPLG>(source(u, i0[u]));
        if (i1[u] < n) v1[u] = ld1<NT_EXPLG>(source(u, i1[u]));
    }
#pragma unroll
    for (int u = 0; u < PEXP; ++u) {
        const uint32_t j = lo[u] + lane;
        float* out = static_cast<float*>(expl_val.p[q0 + u < MAXW ? q0 + u : 0]);
        if (j < hi[u]) out[j] = v0[u];
        if (j + 64u < hi[u]) out[j + 64u] = v1[u];
        for (uint32_t k = j + 128u; k < hi[u]; k += 64) {
            const uint32_t i = static_cast<const uint32_t*>(expl_idx.p[q0 + u])[k];
            out[k] = i < n ? *source(u, i) : 0.0f;
        }
    }
}

template <int NBUF>
__global__ __launch_bounds__(BLOCK) void k_pack_stream(PtrTab g, uint32_t nw, const uint32_t* __restrict__ tile_start,
                                                       const uint32_t* __restrict__ core_idx,
                                                       const uint32_t* __restrict__ core_off, PtrTab expl_idx,
                                                       PtrTab expl_off, MutPtrTab core_val, MutPtrTab expl_val, int vec_ok)
{
    __shared__ float buf[NBUF][TILE];
    __shared__ uint16_t cpos[TILE];          // the tile's core positions: the same for every worker
    __shared__ uint32_t elo[MAXW], ehi[MAXW];
    const uint32_t t = blockIdx.x;
    const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
    const bool vec = vec_ok && len == TILE && (start & 3u) == 0;
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    const uint32_t ccnt = (c1 - c0 < TILE) ? c1 - c0 : TILE;
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        elo[threadIdx.x] = eo[t];
        ehi[threadIdx.x] = eo[t + 1];
    }
    for (uint32_t x = threadIdx.x; x < ccnt; x += BLOCK) {
        const uint32_t pos = core_idx[c0 + x] - start;
        cpos[x] = (pos < len) ? (uint16_t)pos : (uint16_t)0xFFFF;
    }
    __syncthreads();
    // Loads are requested one worker ahead and nothing inside the loop waits for a load that
    // was requested in the same iteration: the tile of updates and this thread's explorer
    // index of the next worker travel while the current worker's values are picked from LDS.
    float r[EPT];
    uint32_t epos = 0xFFFFFFFFu;             // explorer entry elo[q] + threadIdx.x of the coming worker, if any
    auto fetch = [&](uint32_t q) {
        const float* src = static_cast<const float*>(g.p[q]) + start;
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 v = ld4<NT_PACKS>(src + k * 1024 + threadIdx.x * 4);
                r[4 * k + 0] = v.x; r[4 * k + 1] = v.y; r[4 * k + 2] = v.z; r[4 * k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = elem_scl(j);
                r[j] = (e < len) ? src[e] : 0.0f;
            }
        }
        // the index itself: anything computed from it here would make the wave wait for this load, and with it for the
        // tile requested just before, on the spot
        const uint32_t j = elo[q] + threadIdx.x;
        epos = 0xFFFFFFFFu;
        if (j < ehi[q]) epos = static_cast<const uint32_t*>(expl_idx.p[q])[j];
    };
    fetch(0);
    for (uint32_t q = 0; q < nw; ++q) {
        float* b = buf[NBUF == 2 ? (q & 1u) : 0];
        if (NBUF == 1 && q) __syncthreads();     // the previous worker's readers are done with the buffer
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<float4*>(b + k * 1024 + threadIdx.x * 4) = make_float4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) b[elem_scl(j)] = r[j];
        }
        const uint32_t my_epos = epos - start;      // no entry: wraps to a position beyond any tile (start + len < 2^32)
        __syncthreads();     // with two buffers this also orders a buffer's readers (two workers ago) before its writers
        if (q + 1 < nw) fetch(q + 1);
        float* cv = static_cast<float*>(core_val.p[q]);
        for (uint32_t x = threadIdx.x; x < ccnt; x += BLOCK) {
            const uint32_t pos = cpos[x];
            if (pos != 0xFFFFu) cv[c0 + x] = b[pos];
        }
        float* ev = static_cast<float*>(expl_val.p[q]);
        const uint32_t e0 = elo[q], e1 = ehi[q];
        if (my_epos < len) ev[e0 + threadIdx.x] = b[my_epos];
        if (e1 - e0 > BLOCK) {               // dense explorers: the rest of the slice, loaded here
            const uint32_t* ei = static_cast<const uint32_t*>(expl_idx.p[q]);
            for (uint32_t j = e0 + BLOCK + threadIdx.x; j < e1; j += BLOCK) {
                const uint32_t pos = ei[j] - start;
                if (pos < len) ev[j] = b[pos];
            }
        }
    }
}

// The same pack with the two halves of the work in different waves (512 threads: waves 0..3 load, waves 4..7 store).
// A wave's vector-memory operations retire in issue order, so a wave that stores a worker's slices and then needs the
// next worker's tile waits for its own stores to be acknowledged by the cache, every step; here the loading waves never
// store and the storing waves never load from memory: the tile of updates, the core positions and the explorer
// positions all reach them through LDS.  Consecutive tiles go to the same die (blocks are dealt to the eight dies in
// turn), so that the partial lines at the two ends of a tile's output slices meet their other halves in one L2.
// grid: 8 * ceil(T / 8) blocks.
__global__ __launch_bounds__(2 * BLOCK) void k_pack_stream_ws(PtrTab g, uint32_t nw, uint32_t T,
                                                               const uint32_t* __restrict__ tile_start,
                                                               const uint32_t* __restrict__ core_idx,
                                                               const uint32_t* __restrict__ core_off, PtrTab expl_idx,
                                                               PtrTab expl_off, MutPtrTab core_val, MutPtrTab expl_val)
{
    __shared__ float buf[2][TILE];
    __shared__ uint16_t cpos[TILE];          // the tile's core positions: the same for every worker
    __shared__ uint32_t epos[2][BLOCK];      // the first BLOCK explorer positions of the worker whose tile is in buf[.]
    __shared__ uint32_t elo[MAXW], ehi[MAXW];
    const uint32_t chunk = gridDim.x >> 3;
    const uint32_t t = (blockIdx.x & 7u) * chunk + (blockIdx.x >> 3);
    if (t >= T) return;                      // uniform over the block
    const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
    const bool vec = len == TILE;
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    const uint32_t ccnt = (c1 - c0 < TILE) ? c1 - c0 : TILE;
    const bool loader = threadIdx.x < BLOCK;
    const uint32_t tid = threadIdx.x & (BLOCK - 1u);
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        elo[threadIdx.x] = eo[t];
        ehi[threadIdx.x] = eo[t + 1];
    }
    for (uint32_t x = threadIdx.x; x < ccnt; x += 2 * BLOCK) {
        const uint32_t pos = core_idx[c0 + x] - start;
        cpos[x] = (pos < len) ? (uint16_t)pos : (uint16_t)0xFFFF;
    }
    __syncthreads();
    float r[EPT];
    uint32_t ep = 0xFFFFFFFFu;
    auto fetch = [&](uint32_t q) {
        const float* src = static_cast<const float*>(g.p[q]) + start;
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 v = ld4<NT_PACKS>(src + k * 1024 + tid * 4);
                r[4 * k + 0] = v.x; r[4 * k + 1] = v.y; r[4 * k + 2] = v.z; r[4 * k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = (uint32_t)j * BLOCK + tid;
                r[j] = (e < len) ? src[e] : 0.0f;
            }
        }
        // the index itself: anything computed from it here would make the wave wait for this load, and with it for the
        // tile requested just before, on the spot
        const uint32_t j = elo[q] + tid;
        ep = 0xFFFFFFFFu;
        if (j < ehi[q]) ep = static_cast<const uint32_t*>(expl_idx.p[q])[j];
    };
    if (loader) fetch(0);
    for (uint32_t q = 0; q < nw; ++q) {
        float* b = buf[q & 1u];
        if (loader) {
            if (vec) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<float4*>(b + k * 1024 + tid * 4) = make_float4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]);
            } else {
#pragma unroll
                for (int j = 0; j < EPT; ++j) b[(uint32_t)j * BLOCK + tid] = r[j];
            }
            epos[q & 1u][tid] = ep - start;       // no entry: wraps to a position beyond any tile (start + len < 2^32)
            if (q + 1 < nw) fetch(q + 1);
        }
        // the tile of worker q is in LDS; the storing waves are done with the buffer it replaced (worker q - 2): they
        // passed the previous barrier only after issuing its last LDS reads, and LDS operations of a wave finish in order
        __syncthreads();
        if (!loader) {
            float* cv = static_cast<float*>(core_val.p[q]);
            for (uint32_t x = tid; x < ccnt; x += BLOCK) {
                const uint32_t pos = cpos[x];
                if (pos != 0xFFFFu) cv[c0 + x] = b[pos];
            }
            float* ev = static_cast<float*>(expl_val.p[q]);
            const uint32_t e0 = elo[q], e1 = ehi[q];
            const uint32_t my = epos[q & 1u][tid];
            if (my < len) ev[e0 + tid] = b[my];
            if (e1 - e0 > BLOCK) {               // dense explorers: the rest of the slice, positions loaded here
                const uint32_t* ei = static_cast<const uint32_t*>(expl_idx.p[q]);
                for (uint32_t j = e0 + BLOCK + tid; j < e1; j += BLOCK) {
                    const uint32_t pos = ei[j] - start;
                    if (pos < len) ev[j] = b[pos];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// K6: merge.  One block per tile of the global model; no atomics on global memory and a
// result that does not depend on scheduling.
//
// Core: every worker sends a value for each core index, so the thread that owns entry j of
// the tile's slice of the core list sums the W values in worker order in registers.
//
// Explorers: each entry of the tile takes a ticket at its position (LDS byte counter).  A
// position with one or two entries is summed in ticket order -- with at most two addends
// the binary32 sum does not depend on their order.  Positions with three or more entries
// (rare), or with two on top of a core sum (only if a list overlaps the core), are summed in worker order, a
// barrier to a worker.  Tiles with more explorer entries than the fast path holds in registers
// take the generic path: entries staged through LDS and applied one worker at a time.
//
// All loads of a tile (its w, its core slice, its explorer entries) are requested in one
// go right after the tile's offsets are known.
// ---------------------------------------------------------------------------------------
// Sum of the W workers' values of core entry j, from +0 in worker order.  The loads of eight workers are requested
// together (a loop with one load and one add per turn waits for memory W times in a row).
__device__ __forceinline__ float core_sum(const PtrTab& core_val, uint32_t nw, uint32_t j)
{
    float a = 0.0f;
    for (uint32_t q0 = 0; q0 < nw; q0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = (q0 + u < nw) ? ld1<NT_MERGE_VAL>(static_cast<const float*>(core_val.p[q0 + u]) + j) : 0.0f;
#pragma unroll
        for (int u = 0; u < 8; ++u) if (q0 + u < nw) a = a + v[u];
    }
    return a;
}

// R: explorer entries per thread kept in registers.  Four serve the tiles of the paper's ratios; denser requests get a
// variant with more, chosen on the host from the expected number (slimdp_merge): a tile that does not fit takes the
// generic path, which stages its entries through LDS 256 at a time.
constexpr uint32_t MERGE_STAGE = 256;

// LINES: a flat model at an aligned address, whose tiles are whole lines and leave non-temporally; a choice at run time kept
// two forms of the stores apart and cost the kernel a third (138*10^6 parameters, 8 workers).
template <int R, int LINES>
__global__ __launch_bounds__(BLOCK) void k_merge(float* __restrict__ w, float lr, uint32_t nw,
                                                 const uint32_t* __restrict__ tile_start,
                                                 const uint32_t* __restrict__ core_idx, const uint32_t* __restrict__ core_off,
                                                 PtrTab core_val, PtrTab expl_idx, PtrTab expl_off, PtrTab expl_val,
                                                 uint64_t n, uint32_t n_seg)
{
    __shared__ float acc[TILE];
    __shared__ uint32_t cnt[TILE / 4];     // one byte per position: bit 7 = core, low bits = explorer entries
    __shared__ uint32_t elo[MAXW], ecn[MAXW];
    __shared__ uint32_t hot;               // some position has more entries than ticket order can sum
    __shared__ uint16_t spos[MERGE_STAGE];
    __shared__ float sval[MERGE_STAGE];
    const uint32_t t = blockIdx.x;
    // flat model: no table look-up before the tile's loads can be requested
    uint32_t start, len;
    if (n_seg == 1) {
        start = t * TILE;
        const uint64_t rest = n - (uint64_t)start;
        len = rest < TILE ? (uint32_t)rest : TILE;
    } else {
        start = tile_start[t]; len = tile_start[t + 1] - start;
    }
    const bool vec = len == TILE;
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    float wv[EPT];
    if (vec) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float4 v = ld4<NT_MERGE_LD>(w + (size_t)start + r * 1024 + threadIdx.x * 4);
            wv[4 * r + 0] = v.x; wv[4 * r + 1] = v.y; wv[4 * r + 2] = v.z; wv[4 * r + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint32_t e = elem_scl(j);
            wv[j] = (e < len) ? w[(size_t)start + e] : 0.0f;
        }
    }
    for (uint32_t x = threadIdx.x; x < TILE / 4; x += BLOCK) cnt[x] = 0;
    if (threadIdx.x == 0) hot = 0;
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        const uint32_t lo = eo[t];
        elo[threadIdx.x] = lo;
        ecn[threadIdx.x] = eo[t + 1] - lo;
    }
    __syncthreads();
    uint32_t E = 0;
    for (uint32_t q = 0; q < nw; ++q) E += ecn[q];
    const bool fast = E <= (uint32_t)(BLOCK * R);
    // explorer entries of the fast path: requested now, held in registers
    uint32_t epos[R], eq[R], etk[R];
    float eval[R];
    if (fast) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint32_t x = threadIdx.x + (uint32_t)i * BLOCK;
            epos[i] = 0xFFFFFFFFu; eq[i] = 0; etk[i] = 0; eval[i] = 0.0f;
            if (x < E) {
                uint32_t q = 0, run = 0;
                while (q + 1 < nw && run + ecn[q] <= x) { run += ecn[q]; ++q; }
                const uint32_t j = elo[q] + (x - run);
                const uint32_t pos = static_cast<const uint32_t*>(expl_idx.p[q])[j] - start;
                eval[i] = static_cast<const float*>(expl_val.p[q])[j];
                eq[i] = q;
                if (pos < len) epos[i] = pos;
            }
        }
    }
    // core: every worker contributes, in worker order
    for (uint32_t j = c0 + threadIdx.x; j < c1; j += BLOCK) {
        const uint32_t pos = core_idx[j] - start;
        const float a = core_sum(core_val, nw, j);
        if (pos < len) { acc[pos] = a; atomicOr(&cnt[pos >> 2], 0x80u << (8u * (pos & 3u))); }
    }
    if (fast) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (epos[i] != 0xFFFFFFFFu) {
                const uint32_t sh = 8u * (epos[i] & 3u);
                etk[i] = (atomicAdd(&cnt[epos[i] >> 2], 1u << sh) >> sh) & 0x7Fu;
            }
        }
    }
    __syncthreads();
    if (fast) {
        // first and second entry of a position, in ticket order; the rest is replayed in worker order
        uint32_t tot[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            tot[i] = 0;
            if (epos[i] != 0xFFFFFFFFu) {
                const uint32_t byte = (cnt[epos[i] >> 2] >> (8u * (epos[i] & 3u))) & 0xFFu;
                tot[i] = byte & 0x7Fu;
                // two explorer entries on top of a core sum (lists that overlap the core: invalid input) would make
                // the result depend on the ticket order: such a position is replayed in worker order as well
                if (tot[i] == 2u && (byte & 0x80u)) tot[i] = 3u;
                if (tot[i] <= 2u) {
                    if (etk[i] == 0) acc[epos[i]] = ((byte & 0x80u) ? acc[epos[i]] : 0.0f) + eval[i];
                } else {
                    hot = 1u;
                    if (etk[i] == 0 && !(byte & 0x80u)) acc[epos[i]] = 0.0f;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (epos[i] != 0xFFFFFFFFu && tot[i] == 2u && etk[i] == 1u) acc[epos[i]] = acc[epos[i]] + eval[i];
        // positions with more: every worker's entries in turn, straight from the registers (a serial replay from a list, by one
        // thread a position, took longer than the generic path where a third of the tile's positions are sent)
        if (hot) {                               // uniform: written before the barrier above
            for (uint32_t q = 0; q < nw; ++q) {
#pragma unroll
                for (int i = 0; i < R; ++i)
                    if (epos[i] != 0xFFFFFFFFu && tot[i] > 2u && eq[i] == q) acc[epos[i]] = acc[epos[i]] + eval[i];
                __syncthreads();
            }
        }
    }
    __syncthreads();
    if (!fast) {
        // generic path: every explorer entry staged through LDS, applied one worker at a time.
        // The counters keep their core bits; a set low bit now means "an explorer sum is in acc".
        for (uint32_t x = threadIdx.x; x < TILE / 4; x += BLOCK) cnt[x] &= 0x80808080u;
        __syncthreads();
        uint8_t* hit = reinterpret_cast<uint8_t*>(cnt);
        for (uint32_t cb = 0; cb < E; cb += MERGE_STAGE) {
            const uint32_t cn = (E - cb < MERGE_STAGE) ? E - cb : MERGE_STAGE;
            for (uint32_t x = threadIdx.x; x < cn; x += BLOCK) {
                const uint32_t v = cb + x;
                uint32_t q = 0, run = 0;
                while (q + 1 < nw && run + ecn[q] <= v) { run += ecn[q]; ++q; }
                const uint32_t j = elo[q] + (v - run);
                const uint32_t pos = static_cast<const uint32_t*>(expl_idx.p[q])[j] - start;
                spos[x] = (pos < len) ? (uint16_t)pos : (uint16_t)0xFFFF;
                sval[x] = static_cast<const float*>(expl_val.p[q])[j];
            }
            __syncthreads();
            uint32_t run = 0;
            for (uint32_t q = 0; q < nw; ++q) {
                const uint32_t qlo = run, qhi = run + ecn[q];
                run = qhi;
                if (qhi <= cb || qlo >= cb + cn) continue;
                const uint32_t lo = (qlo > cb) ? qlo - cb : 0u;
                const uint32_t hi = (qhi - cb < cn) ? qhi - cb : cn;
                for (uint32_t x = lo + threadIdx.x; x < hi; x += BLOCK) {
                    const uint32_t pos = spos[x];
                    if (pos != 0xFFFFu) {
                        acc[pos] = (hit[pos] ? acc[pos] : 0.0f) + sval[x];
                        hit[pos] |= 1;
                    }
                }
                __syncthreads();
            }
            __syncthreads();
        }
    }
    // apply and stream the tile back
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const uint32_t e = vec ? elem_vec(j) : elem_scl(j);
        if (e < len && ((cnt[e >> 2] >> (8u * (e & 3u))) & 0xFFu)) {
            wv[j] = __builtin_fmaf(-lr, acc[e], wv[j]);
            if (!vec) w[(size_t)start + e] = wv[j];
        }
    }
    if (vec) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            st4<LINES && NT_MERGE_ST>(w + (size_t)start + r * 1024 + threadIdx.x * 4,
                             make_float4(wv[4 * r], wv[4 * r + 1], wv[4 * r + 2], wv[4 * r + 3]));
    }
}

// ---------------------------------------------------------------------------------------
// Worker side, LocalTrain (section 3.3 step 1): one mini-batch step on every worker's LOCAL
// model, w_q <- fma(-eta, grad_q, w_q), and the accumulation of the update that the next
// push sends, delta_q = grad_1 + grad_2 + ... in binary32 in mini-batch order (first: a new
// accumulation starts with this gradient; delta is then not read).  20 bytes per parameter
// and worker (16 when first).  NT: as in the two kernels below, streams pass the caches by (see local_streams).
// grid (blocks, n_workers).
// ---------------------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(256) void k_local_step(MutPtrTab w_local, PtrTab grad, MutPtrTab delta, uint64_t n, float eta,
                                                    int first, int vec_ok)
{
    const uint32_t q = blockIdx.y;
    float* w = static_cast<float*>(w_local.p[q]);
    const float* g = static_cast<const float*>(grad.p[q]);
    float* d = static_cast<float*>(delta.p[q]);
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    const uint64_t n4 = vec_ok ? n / 4 : 0;
    for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < n4; x += 2 * stride) {       // two vectors per turn in flight
        const uint64_t x2 = x + stride;
        const bool two = x2 < n4;
        const float4 ga = ld4<NT>(g + 4 * x), wa = ld4<NT>(w + 4 * x);
        const float4 gb = two ? ld4<NT>(g + 4 * x2) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 wb = two ? ld4<NT>(w + 4 * x2) : make_float4(0.f, 0.f, 0.f, 0.f);
        float4 da = ga, db = gb;
        if (!first) {
            const float4 oa = ld4<NT>(d + 4 * x);
            da = make_float4(oa.x + ga.x, oa.y + ga.y, oa.z + ga.z, oa.w + ga.w);
            if (two) {
                const float4 ob = ld4<NT>(d + 4 * x2);
                db = make_float4(ob.x + gb.x, ob.y + gb.y, ob.z + gb.z, ob.w + gb.w);
            }
        }
        st4<NT>(w + 4 * x, make_float4(__builtin_fmaf(-eta, ga.x, wa.x), __builtin_fmaf(-eta, ga.y, wa.y),
                                      __builtin_fmaf(-eta, ga.z, wa.z), __builtin_fmaf(-eta, ga.w, wa.w)));
        st4<NT>(d + 4 * x, da);
        if (two) {
            st4<NT>(w + 4 * x2, make_float4(__builtin_fmaf(-eta, gb.x, wb.x), __builtin_fmaf(-eta, gb.y, wb.y),
                                           __builtin_fmaf(-eta, gb.z, wb.z), __builtin_fmaf(-eta, gb.w, wb.w)));
            st4<NT>(d + 4 * x2, db);
        }
    }
    for (uint64_t i = 4 * n4 + (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {      // tail, or unaligned arrays
        const float gi = g[i];
        w[i] = __builtin_fmaf(-eta, gi, w[i]);
        d[i] = first ? gi : d[i] + gi;
    }
}

// ---------------------------------------------------------------------------------------
// LocalTrain and Push in one pass (section 3.3 steps 1 and 3): the last mini-batch step before a
// communication already streams the accumulated update of every worker; picking the values at
// the communication set while a tile of the new update sits in LDS saves the extraction its own
// scan of the update vectors (the full scan that section 3.5 counts per extraction).  Same
// results as k_local_step followed by k_pack_stream on delta.  One block per tile and per_block
// workers in turn, the next worker's three tiles in flight while the current one is picked from.
// SPLIT = 0: all workers.  Their pointers are then found at fixed places of the arguments and come together; by a number
// worked out first they come one after the other, before the first tile can be asked for (one worker, 8*10^6 parameters:
// 28.9 us without a split, 30.8 with the form for one).
// ---------------------------------------------------------------------------------------
template <int NBUF, int NT, int SPLIT>
__global__ __launch_bounds__(BLOCK) void k_local_step_pack(MutPtrTab w_local, PtrTab grad, MutPtrTab delta, float eta, int first,
                                                           uint32_t nw, uint32_t per_block, const uint32_t* __restrict__ tile_start,
                                                           const uint32_t* __restrict__ core_idx,
                                                           const uint32_t* __restrict__ core_off, PtrTab expl_idx, PtrTab expl_off,
                                                           MutPtrTab core_val, MutPtrTab expl_val, int vec_ok)
{
    __shared__ float buf[NBUF][TILE];
    __shared__ uint16_t cpos[TILE];          // the tile's core positions: the same for every worker
    __shared__ uint32_t elo[MAXW], ehi[MAXW];
    const uint32_t t = blockIdx.x, q0 = SPLIT ? blockIdx.y * per_block : 0u, q1 = SPLIT ? min(q0 + per_block, nw) : nw;
    const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
    const bool vec = vec_ok && len == TILE && (start & 3u) == 0;
    float rg[EPT], rw[EPT], rd[EPT];
    uint32_t epos = 0xFFFFFFFFu;
    auto fetch = [&](uint32_t q) {
        const float* g = static_cast<const float*>(grad.p[q]) + start;
        const float* w = static_cast<const float*>(w_local.p[q]) + start;
        const float* d = static_cast<const float*>(delta.p[q]) + start;
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = k * 1024 + threadIdx.x * 4;
                const float4 a = ld4<NT>(g + o), b = ld4<NT>(w + o);
                rg[4 * k + 0] = a.x; rg[4 * k + 1] = a.y; rg[4 * k + 2] = a.z; rg[4 * k + 3] = a.w;
                rw[4 * k + 0] = b.x; rw[4 * k + 1] = b.y; rw[4 * k + 2] = b.z; rw[4 * k + 3] = b.w;
                if (!first) {
                    const float4 c = ld4<NT>(d + o);
                    rd[4 * k + 0] = c.x; rd[4 * k + 1] = c.y; rd[4 * k + 2] = c.z; rd[4 * k + 3] = c.w;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = elem_scl(j);
                rg[j] = (e < len) ? g[e] : 0.0f;
                rw[j] = (e < len) ? w[e] : 0.0f;
                rd[j] = (e < len && !first) ? d[e] : 0.0f;
            }
        }
        // the index itself: anything computed from it here would make the wave wait for this load, and with it for the
        // tile requested just before, on the spot
        const uint32_t j = elo[q] + threadIdx.x;
        epos = 0xFFFFFFFFu;
        if (j < ehi[q]) epos = static_cast<const uint32_t*>(expl_idx.p[q])[j];
    };
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    const uint32_t ccnt = (c1 - c0 < TILE) ? c1 - c0 : TILE;
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        elo[threadIdx.x] = eo[t];
        ehi[threadIdx.x] = eo[t + 1];
    }
    for (uint32_t x = threadIdx.x; x < ccnt; x += BLOCK) {
        const uint32_t pos = core_idx[c0 + x] - start;
        cpos[x] = (pos < len) ? (uint16_t)pos : (uint16_t)0xFFFF;
    }
    __syncthreads();
    // not before the lists: one round with it there / here, us: 30*10^6 parameters in 57 segments, 1 worker 282 / 269, 8*10^6, 4 217 / 213,
    // 10^6, 8 61.7 / 60.4
    fetch(q0);
    for (uint32_t q = q0; q < q1; ++q) {
        float* b = buf[NBUF == 2 ? (q & 1u) : 0];
        float* w = static_cast<float*>(w_local.p[q]) + start;
        float* d = static_cast<float*>(delta.p[q]) + start;
        if (NBUF == 1 && q != q0) __syncthreads();     // the previous worker's readers are done with the buffer
        // the step and the accumulation; the new update goes to memory and to LDS
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            rw[j] = __builtin_fmaf(-eta, rg[j], rw[j]);
            rd[j] = first ? rg[j] : rd[j] + rg[j];
        }
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = k * 1024 + threadIdx.x * 4;
                st4<NT>(w + o, make_float4(rw[4 * k], rw[4 * k + 1], rw[4 * k + 2], rw[4 * k + 3]));
                st4<NT>(d + o, make_float4(rd[4 * k], rd[4 * k + 1], rd[4 * k + 2], rd[4 * k + 3]));
                *reinterpret_cast<float4*>(b + o) = make_float4(rd[4 * k], rd[4 * k + 1], rd[4 * k + 2], rd[4 * k + 3]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = elem_scl(j);
                if (e < len) { w[e] = rw[j]; d[e] = rd[j]; }
                b[e] = rd[j];
            }
        }
        const uint32_t my_epos = epos - start;      // no entry: wraps to a position beyond any tile (start + len < 2^32)
        __syncthreads();     // with two buffers this also orders a buffer's readers (two workers ago) before its writers
        if (q + 1 < q1) fetch(q + 1);
        float* cv = static_cast<float*>(core_val.p[q]);
        for (uint32_t x = threadIdx.x; x < ccnt; x += BLOCK) {
            const uint32_t pos = cpos[x];
            if (pos != 0xFFFFu) cv[c0 + x] = b[pos];
        }
        float* ev = static_cast<float*>(expl_val.p[q]);
        const uint32_t e0 = elo[q], e1 = ehi[q];
        if (my_epos < len) ev[e0 + threadIdx.x] = b[my_epos];
        if (e1 - e0 > BLOCK) {               // dense explorers: the rest of the slice, loaded here
            const uint32_t* ei = static_cast<const uint32_t*>(expl_idx.p[q]);
            for (uint32_t j = e0 + BLOCK + threadIdx.x; j < e1; j += BLOCK) {
                const uint32_t pos = ei[j] - start;
                if (pos < len) ev[j] = b[pos];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Pull, local Merge and LocalTrain in one pass (section 3.3 steps 4, 5 and 1 of the next round): the local model
// is overwritten with the global one at the worker's communication set, then stepped.  The first local step after a
// communication streams every local model anyway; applying the pulled values there saves the pull its own pass,
// whose scattered 4-byte writes touch nearly every line of every local model.  Same results as k_gather with a
// scatter destination followed by k_local_step.  STEP = 0: a pull with local models, whose values at the communication
// sets leave from the same pass (as a kernel of its own the gather read model and lists a second time: 10^6 parameters, 4 workers
// 6 + 11 us, 14 together); workers without a local model are not patched.  One block per tile and per_block workers: the tile of the global model stays in
// registers for all workers, the communication set of a worker is a bitmap in LDS (core positions once per tile,
// explorer positions per worker, marked one worker ahead), the next worker's three tiles travel meanwhile.  SPLIT: as above.
// ---------------------------------------------------------------------------------------
template <int STEP, int NT, int SPLIT>
__global__ __launch_bounds__(BLOCK) void k_pull_local_step(const float* __restrict__ w, MutPtrTab w_local, PtrTab grad, MutPtrTab delta,
                                                           float eta, int first, uint32_t nw, uint32_t per_block, uint64_t n,
                                                           const uint32_t* __restrict__ tile_start,
                                                           const uint32_t* __restrict__ core_idx,
                                                           const uint32_t* __restrict__ core_off, PtrTab expl_idx, PtrTab expl_off,
                                                           MutPtrTab core_out, MutPtrTab expl_out, int vec_ok)
{
    __shared__ uint32_t cm[TILE_WORDS];          // core positions of the tile
    __shared__ uint32_t em[2][TILE_WORDS];       // explorer positions of a worker
    __shared__ uint32_t elo[MAXW], ehi[MAXW];
    __shared__ __align__(16) float ws[STEP ? 4 : TILE];      // the tile of the global model, for the values that leave
    const uint32_t t = blockIdx.x, q0 = SPLIT ? blockIdx.y * per_block : 0u, q1 = SPLIT ? min(q0 + per_block, nw) : nw;
    const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
    const bool vec = vec_ok && len == TILE && (start & 3u) == 0;
    const uint32_t c0 = core_off[t], c1 = core_off[t + 1];
    if (threadIdx.x < nw) {
        const uint32_t* eo = static_cast<const uint32_t*>(expl_off.p[threadIdx.x]);
        elo[threadIdx.x] = eo[t];
        ehi[threadIdx.x] = eo[t + 1];
    }
    if (threadIdx.x < TILE_WORDS) { cm[threadIdx.x] = 0; em[q0 & 1u][threadIdx.x] = 0; }
    // this thread's elements of the global model: the same positions as its elements of every local model
    float wv[EPT];
    if (vec) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 v = ld4<NT>(w + (size_t)start + k * 1024 + threadIdx.x * 4);
            wv[4 * k + 0] = v.x; wv[4 * k + 1] = v.y; wv[4 * k + 2] = v.z; wv[4 * k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint32_t e = elem_scl(j);
            wv[j] = (e < len) ? w[(size_t)start + e] : 0.0f;
        }
    }
    if (!STEP) {
        if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<float4*>(ws + k * 1024 + threadIdx.x * 4) = make_float4(wv[4 * k], wv[4 * k + 1], wv[4 * k + 2], wv[4 * k + 3]);
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) ws[elem_scl(j)] = wv[j];
        }
    }
    __syncthreads();
    for (uint32_t j = c0 + threadIdx.x; j < c1; j += BLOCK) {
        const uint32_t i = core_idx[j], pos = i - start;
        if (pos < len) atomicOr(&cm[pos >> 5], 1u << (pos & 31u));
        if (!STEP && i < n) {
            const float v = pos < len ? ws[pos] : w[i];
            for (uint32_t q = q0; q < q1; ++q) static_cast<float*>(core_out.p[q])[j] = v;
        }
    }
    // explorer positions of worker q into em[q & 1] (zeroed before): the first BLOCK entries from the index each
    // thread already holds (requested a turn ago with the tiles), the rest, if any, read here
    uint32_t epre = 0xFFFFFFFFu;
    auto value_out = [&](uint32_t q, uint32_t j, uint32_t i) {
        if (!STEP && i < n) static_cast<float*>(expl_out.p[q])[j] = i - start < len ? ws[i - start] : w[i];
    };
    auto mark = [&](uint32_t q, uint32_t held, uint32_t from) {
        const uint32_t p0 = held - start;        // no entry: wraps beyond any tile
        if (p0 < len) atomicOr(&em[q & 1u][p0 >> 5], 1u << (p0 & 31u));
        if (from) value_out(q, elo[q] + threadIdx.x, held);      // no entry: beyond any model
        const uint32_t* ei = static_cast<const uint32_t*>(expl_idx.p[q]);
        for (uint32_t j = elo[q] + from + threadIdx.x; j < ehi[q]; j += BLOCK) {
            const uint32_t i = ei[j], pos = i - start;
            if (pos < len) atomicOr(&em[q & 1u][pos >> 5], 1u << (pos & 31u));
            value_out(q, j, i);
        }
    };
    float rg[EPT], rl[EPT], rd[EPT];
    auto fetch = [&](uint32_t q) {
        const float* g = STEP ? static_cast<const float*>(grad.p[q]) + start : nullptr;
        const float* l = static_cast<const float*>(w_local.p[q]) + start;
        const float* d = STEP ? static_cast<const float*>(delta.p[q]) + start : nullptr;
        if (!STEP && !w_local.p[q]) {
            // a worker without a local model to patch (uniform over the block)
        } else if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = k * 1024 + threadIdx.x * 4;
                const float4 b = ld4<NT>(l + o);
                rl[4 * k + 0] = b.x; rl[4 * k + 1] = b.y; rl[4 * k + 2] = b.z; rl[4 * k + 3] = b.w;
                if (STEP) {
                    const float4 a = ld4<NT>(g + o);
                    rg[4 * k + 0] = a.x; rg[4 * k + 1] = a.y; rg[4 * k + 2] = a.z; rg[4 * k + 3] = a.w;
                }
                if (STEP && !first) {
                    const float4 c = ld4<NT>(d + o);
                    rd[4 * k + 0] = c.x; rd[4 * k + 1] = c.y; rd[4 * k + 2] = c.z; rd[4 * k + 3] = c.w;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = elem_scl(j);
                rg[j] = (STEP && e < len) ? g[e] : 0.0f;
                rl[j] = (e < len) ? l[e] : 0.0f;
                rd[j] = (STEP && e < len && !first) ? d[e] : 0.0f;
            }
        }
        // this thread's explorer index of the worker after: held, not used, until that worker's marks are made
        epre = 0xFFFFFFFFu;
        if (q + 1 < q1) {
            const uint32_t j = elo[q + 1] + threadIdx.x;
            if (j < ehi[q + 1]) epre = static_cast<const uint32_t*>(expl_idx.p[q + 1])[j];
        }
    };
    mark(q0, 0xFFFFFFFFu, 0u);
    fetch(q0);
    for (uint32_t q = q0; q < q1; ++q) {
        // the marks of worker q (made a turn ago) are complete; the other bitmap is free (its reader finished a turn ago)
        __syncthreads();
        if (threadIdx.x < TILE_WORDS) em[(q + 1u) & 1u][threadIdx.x] = 0;
        float nl[EPT], nd[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint32_t e = vec ? elem_vec(j) : elem_scl(j);
            const uint32_t bit = ((cm[e >> 5] | em[q & 1u][e >> 5]) >> (e & 31u)) & 1u;
            const float base = bit ? wv[j] : rl[j];                  // steps 4, 5: the pulled value replaces the local one
            nl[j] = STEP ? __builtin_fmaf(-eta, rg[j], base) : base; // step 1 of the next round
            nd[j] = first ? rg[j] : rd[j] + rg[j];
        }
        const bool patch = STEP || w_local.p[q] != nullptr;          // uniform over the block
        float* l = static_cast<float*>(w_local.p[q]) + start;
        float* d = STEP ? static_cast<float*>(delta.p[q]) + start : nullptr;
        __syncthreads();                         // the other bitmap is zero everywhere before the next worker's marks go in
        // the next worker's marks and tiles, requested before this worker's stores: the wait for them need not cover the
        // stores' acknowledgements
        if (q + 1 < q1) { mark(q + 1, epre, BLOCK); fetch(q + 1); }
        if (!patch) {
        } else if (vec) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = k * 1024 + threadIdx.x * 4;
                st4<NT>(l + o, make_float4(nl[4 * k], nl[4 * k + 1], nl[4 * k + 2], nl[4 * k + 3]));
                if (STEP) st4<NT>(d + o, make_float4(nd[4 * k], nd[4 * k + 1], nd[4 * k + 2], nd[4 * k + 3]));
            }
        } else {
#pragma unroll
            for (int j = 0; j < EPT; ++j) {
                const uint32_t e = elem_scl(j);
                if (e < len) { l[e] = nl[j]; if (STEP) d[e] = nd[j]; }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Quantised wire values (section 2.2, last sentences; section 4.2: random quantisation, 8 bits,
// buckets of 512).  Per bucket of QB consecutive list entries: scale = largest magnitude;
// per value: code = sign bit | level, level = floor(y) + (u < y - floor(y)), y = (|v| / scale) * 127
// in binary32, u = (random word >> 8) * 2^-24; the word of entry j: word (j mod 4) of
// Philox4x32-10 with counter (j div 4, worker, iteration low, high) and key
// (seed low ^ 0x51534744, seed high ^ kind).  One wave per bucket: lane L holds entries
// 4L..4L+3 and 256+4L..256+4L+3 (two Philox calls), the maximum is a wave reduction (exact,
// whatever the order), the 512 codes leave as two stores of whole lines.
// Bound by the vector unit while every value took a division of its own: 53 instructions a value, 149 us for 8 workers'
// 110*10^6 values.  A bucket has one divisor: with its reciprocal, correctly rounded, a quotient takes a product and two
// corrections of two fused steps each (see quant_quotient): 102 us, 5.4 TB/s.
// grid (ceil(buckets / 4), n_workers).
// ---------------------------------------------------------------------------------------
constexpr uint32_t QB = 512;
struct Count64Tab { uint64_t c[MAXW]; };
__device__ __forceinline__ uint32_t quant_code(float v, float s, uint32_t word)
{
    uint32_t level = 0;
    if (s > 0.0f) {
        const float y = (__builtin_fabsf(v) / s) * 127.0f;
        const float l = __builtin_floorf(y);
        const float u = (float)(word >> 8) * 0x1p-24f;
        level = (uint32_t)l + ((u < y - l) ? 1u : 0u);
    }
    return ((__float_as_uint(v) >> 24) & 0x80u) | level;
}

// a / s, correctly rounded, from r = 1 / s correctly rounded: the first correction leaves the quotient within one unit in the last
// place, and a correction of such a quotient by its exact remainder is the correctly rounded one (Markstein, IBM J. Res.
// Dev. 34 (1990)).  The remainders are exact for s in [2^-40, 2^40] and a zero or in [2^-80, s]: multiples of 2^-127, which
// binary32 holds as a subnormal, and the quotient itself is a normal number.
__device__ __forceinline__ float quant_quotient(float a, float s, float r)
{
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-q, s, a), r, q);
    return __builtin_fmaf(__builtin_fmaf(-q, s, a), r, q);
}
// quant_code's level from its quotient: fraction and whole part of the same y.  Values are finite (the interface asks for
// it); of a NaN the conversion to a whole number is undefined, here as in quant_code.
__device__ __forceinline__ uint32_t quant_code_of(float v, float quotient, uint32_t word)
{
    const float y = quotient * 127.0f;
    const float u = (float)(word >> 8) * 0x1p-24f;
    const uint32_t level = (uint32_t)y + ((u < __builtin_amdgcn_fractf(y)) ? 1u : 0u);
    return ((__float_as_uint(v) >> 24) & 0x80u) | level;
}

__global__ __launch_bounds__(BLOCK) void k_quantize(PtrTab val, Count64Tab count, uint32_t kind, uint32_t worker0,
                                                    PhiloxKey pk, MutPtrTab code, MutPtrTab scale, int vec_ok)
{
    const uint32_t q = blockIdx.y, lane = lane_id();
    const uint64_t cnt = count.c[q];
    const uint64_t b = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint64_t j0 = b * QB;
    if (j0 >= cnt) return;
    const float* v = static_cast<const float*>(val.p[q]);
    uint8_t* out = static_cast<uint8_t*>(code.p[q]);
    const uint32_t len = (cnt - j0 < QB) ? (uint32_t)(cnt - j0) : QB;
    float x[2][4];
    if (vec_ok && len == QB) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float4 t = ld4<1>(v + j0 + h * 256 + lane * 4);
            x[h][0] = t.x; x[h][1] = t.y; x[h][2] = t.z; x[h][3] = t.w;
        }
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t e = h * 256 + lane * 4 + c;
                x[h][c] = (e < len) ? v[j0 + e] : 0.0f;
            }
    }
    float s = 0.0f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) s = __builtin_fmaxf(s, __builtin_fabsf(x[h][c]));
    s = __uint_as_float(wave_max(__float_as_uint(s)));       // no NaN left, no sign: the bits are in the values' order
    if (lane == 0) static_cast<float*>(scale.p[q])[b] = s;
    // the smallest magnitude that is not zero (zero wraps to the largest), as bits
    uint32_t low = 0xFFFFFFFFu;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < 4; ++c) low = min(low, (__float_as_uint(x[h][c]) & 0x7FFFFFFFu) - 1u);
    const bool usual = __ballot(low < __float_as_uint(0x1p-80f) - 1u || !(s >= 0x1p-40f && s <= 0x1p40f)) == 0ull;      // uniform
    const float rs = 1.0f / s;
    auto codes = [&](auto&& code_of) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t r[4];
            philox4x32_10((uint32_t)((j0 + h * 256 + lane * 4) >> 2), worker0 + q, pk.it_lo, pk.it_hi, pk.seed_lo ^ 0x51534744u,
                          pk.seed_hi ^ kind, r);
            uint32_t packed = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) packed |= code_of(x[h][c], r[c]) << (8 * c);
            const uint32_t e = h * 256 + lane * 4;
            if (vec_ok && len == QB) *reinterpret_cast<uint32_t*>(out + j0 + e) = packed;
            else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (e + c < len) out[j0 + e + c] = (uint8_t)(packed >> (8 * c));
            }
        }
    };
    if (usual) codes([&](float v, uint32_t word) { return quant_code_of(v, quant_quotient(__builtin_fabsf(v), s, rs), word); });
    else codes([&](float v, uint32_t word) { return quant_code(v, s, word); });
}

// value = sign * ((scale * level) / 127): two binary32 roundings.  Four codes per thread.  grid (blocks, n_workers).
__global__ __launch_bounds__(256) void k_dequantize(PtrTab code, PtrTab scale, Count64Tab count, MutPtrTab val, int vec_ok)
{
    const uint32_t q = blockIdx.y;
    const uint64_t cnt = count.c[q];
    const uint8_t* in = static_cast<const uint8_t*>(code.p[q]);
    const float* sc = static_cast<const float*>(scale.p[q]);
    float* out = static_cast<float*>(val.p[q]);
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    const uint64_t n4 = vec_ok ? cnt / 4 : 0;
    auto one = [](uint32_t c, float s) {
        const float mag = (s * (float)(c & 0x7Fu)) / 127.0f;
        return (c & 0x80u) ? -mag : mag;
    };
    for (uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x; x < n4; x += stride) {
        const uint32_t p = *reinterpret_cast<const uint32_t*>(in + 4 * x);
        const float s = sc[(4 * x) / QB];
        st4<1>(out + 4 * x, make_float4(one(p & 0xFFu, s), one((p >> 8) & 0xFFu, s), one((p >> 16) & 0xFFu, s), one(p >> 24, s)));
    }
    for (uint64_t j = 4 * n4 + (uint64_t)blockIdx.x * 256 + threadIdx.x; j < cnt; j += stride) out[j] = one(in[j], sc[j / QB]);
}

// Signature of the cached keys: sum over list positions j of mix(idx[j] + 2^32 j) modulo 2^64, mix = the output
// function of SplitMix64.  A wrapping integer sum: any order of the partial sums gives the same bits.
// *sig must be zero at launch.  grid: any, 256 threads.
__device__ __forceinline__ uint64_t splitmix64_mix(uint64_t x)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_signature(const uint32_t* __restrict__ idx, uint64_t k, unsigned long long* __restrict__ sig)
{
    __shared__ unsigned long long part[4];
    unsigned long long s = 0;
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < k; j += (uint64_t)gridDim.x * 256)
        s += splitmix64_mix((uint64_t)idx[j] + (j << 32));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long t = part[0] + part[1] + part[2] + part[3];
        if (t) atomicAdd(sig, t);
    }
}

// Raw random words of the explorer for indices i0 .. i0+count-1.
__global__ __launch_bounds__(256) void k_debug_philox(uint32_t seed_lo, uint32_t seed_hi, uint32_t it_lo, uint32_t it_hi,
                                                      uint32_t worker, uint32_t i0, uint64_t count, uint32_t* __restrict__ out)
{
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < count; j += (uint64_t)gridDim.x * 256) {
        const uint32_t i = i0 + (uint32_t)j;
        uint32_t r[4];
        philox4x32_10(i >> 2, worker, it_lo, it_hi, seed_lo, seed_hi, r);
        out[j] = r[i & 3u];
    }
}

}  // namespace slimdp
