// Explorer selection (gfx950): per worker and segment the m parameters outside the core with the smallest
// (Philox word, index).  Included only by slimdp.hip, after slimdp_kernels.h.
//
// The draw (explore_subtile*, in the scoring pass or k_explore_keys) has sorted every word into a sure zone (bitmap) and
// a candidate zone of about twice the zone's slack, without looking at the core.  What remains takes three launches (and
// k_explore_init, the zones of every segment, where the sizes are not those of the request before):
//   k_explore_collect   per tile the sure parameters outside the core; the candidates outside the core go to the
//                       list of their (worker, segment)
//   k_explore_select    one block per (worker, segment): the demand left by the sure ones, a radix descent over the
//                       list held in registers, the chosen candidates set in the sure bitmap, the tile offsets
//   k_explore_emit      bitmap minus core -> ascending index lists; the exact rerun if a zone missed
// A segment's slack is 6 sqrt(m) + 32 on each side of m, so its list has at most 12 sqrt(n_s) + 64 entries and some spread:
// one block ranks it in the time of a launch or two (19 k of 138 M parameters; 1.7 k of 10^6), where levels, thresholds,
// marks, ties and scans as kernels of their own made sixteen launches of 2 to 8 us each.  A whole iteration of 10^6
// parameters went from 219 to 139 us, of 7*10^6 in 57 segments from 370 to 263 us, of 20*10^6 from 501 to 471 us.
#pragma once
#include "slimdp_kernels.h"

namespace slimdp {

// Writes the selection state of segments [seg0, seg0+count): where the sizes differ from those of the request before.  counts,
// rerun: cleared, if given (nbatch batches of n_seg counters each): after a call that left them in doubt; otherwise the last
// reader of either clears it, and a request of the sizes of the one before starts with its draw or its collection.
// As a launch of every request, and another of every announced draw, this took 2 to 6 us each.
__global__ __launch_bounds__(256) void k_explore_init(SegState* __restrict__ st, SegInitChunk chunk, uint32_t seg0, uint32_t count,
                                                      uint32_t nbatch, uint32_t* __restrict__ counts, uint32_t count_stride,
                                                      uint32_t* __restrict__ rerun)
{
    const uint32_t x = blockIdx.x * 256 + threadIdx.x;
    if (x == 0 && rerun) rerun[0] = 0;
    if (x < count) {
        const SegInit in = chunk.s[x];
        SegState s;
        s.need0 = in.need; s.out_base = in.out_base;
        s.bound_m1 = in.bound_m1; s.sure_m1 = in.sure_m1; s.has_gt = in.has_gt; s.bits = in.bits;
        s.pad[0] = s.pad[1] = 0;
        st[seg0 + x] = s;
    }
    if (counts && x < count * nbatch) counts[(size_t)(x / count) * count_stride + seg0 + x % count] = 0;
}

// Lists: entry (key, tile * TILE + offset inside the tile); batch b's segment s has its entries at
// list[b * stride + first[s]] .. , at most first[s + 1] - first[s] of them (more raise the rerun flag), counted in
// count[b * count_stride + s].  Every batch's counters have lines of their own (count_stride is a multiple of 32): atomics
// on one line take turns, whichever word they meet.  3 workers' counters of a flat model in one line kept
// k_explore_collect_wide at 99 us for 20*10^6 parameters (60 now), 8 workers' k_explore_collect at 75 for 138*10^6 (44 now).
struct ExploreLists { uint2* list; uint32_t* count; const uint32_t* first; uint64_t stride; uint32_t count_stride; };
constexpr uint32_t FLAG_RERUN = 1u;
// The rerun flag has two words, which requests use in turn: the emission of one clears the other's.
struct RerunFlag { uint32_t *now, *next; };

// Sure parameters outside the core of one tile, for batches b0 .. b0+BPW-1, by one wave.
template <int BPW>
__device__ __forceinline__ void count_sure(const uint32_t* __restrict__ core_bits, uint32_t n_words, const TileRef& tr, uint32_t t,
                                           uint32_t T, uint32_t b0, uint32_t nbatch, const uint32_t* __restrict__ sure_bits,
                                           uint32_t* __restrict__ cnt_sel)
{
    const uint32_t lane = lane_id();
    uint2 s2[BPW];
#pragma unroll
    for (int bb = 0; bb < BPW; ++bb) {
        s2[bb] = make_uint2(0u, 0u);
        if (b0 + bb < nbatch)
            s2[bb] = *reinterpret_cast<const uint2*>(sure_bits + ((size_t)(b0 + bb) * T + t) * TILE_WORDS + 2 * lane);
    }
    uint32_t kw[2];
    bitmap_window(core_bits, n_words, tr.start + lane * 64u, kw);
#pragma unroll
    for (int bb = 0; bb < BPW; ++bb) {
        if (b0 + bb >= nbatch) break;
        const uint32_t tot = wave_sum(__popc(s2[bb].x & ~kw[0]) + __popc(s2[bb].y & ~kw[1]));
        if (lane == 0) cnt_sel[(size_t)(b0 + bb) * T + t] = tot;
    }
}

// Narrow zones (draw with PAIRS = 1): two kinds of blocks in one launch.  The first sure_blocks count the sure
// parameters, one wave per tile and BPW batches (the core's bitmap is read once for them); the others gather the few
// candidates, one thread per (batch, sub-tile) so that a thread's chain of loads is count, pairs, core bits (a thread for
// a whole tile went through its candidates one after the other: 35 us at 10^6 parameters).  A block reserves its
// share of a list with one atomic (an atomic costs about 12 ns where thousands meet on one address).  A sub-tile with
// more pairs than its slot holds, or a full list, raises the rerun flag.
// grid: sure_blocks + nbatch * ceil(T / 64), sure_blocks = ceil(T / 4) * ceil(nbatch / BPW).
template <int BPW>
__global__ __launch_bounds__(BLOCK) void k_explore_collect(const uint32_t* __restrict__ core_bits, uint32_t n_words, uint64_t n,
                                                           const uint32_t* __restrict__ tile_start,
                                                           const uint32_t* __restrict__ tile_seg, uint32_t T, uint32_t n_seg,
                                                           uint32_t nbatch, uint32_t sure_blocks,
                                                           const uint32_t* __restrict__ sure_bits, uint32_t* __restrict__ cnt_sel,
                                                           const uint32_t* __restrict__ pairs, uint64_t pair_stride,
                                                           const uint32_t* __restrict__ cnt_cand, ExploreLists lists,
                                                           uint32_t* __restrict__ rerun)
{
    __shared__ uint32_t wtot[4], room;
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    if (blockIdx.x < sure_blocks) {
        const uint32_t quads = (T + 3u) / 4u;
        const uint32_t t = (blockIdx.x % quads) * 4u + wid, b0 = (blockIdx.x / quads) * BPW;
        if (t >= T) return;
        count_sure<BPW>(core_bits, n_words, tile_ref(t, n_seg, n, tile_start, tile_seg), t, T, b0, nbatch, sure_bits, cnt_sel);
        return;
    }
    const uint32_t per = (T + 63u) / 64u, gb = blockIdx.x - sure_blocks;
    const uint32_t b = gb / per, t0 = (gb % per) * 64u, x = t0 * SUBS + threadIdx.x, t = x / SUBS;      // b < nbatch
    uint32_t c = t < T ? cnt_cand[(size_t)b * T * SUBS + x] : 0u;
    if (c > PAIR_CAP) { atomicOr(rerun, FLAG_RERUN); c = 0; }
    // the first four pairs are held, more are read again
    const uint32_t* slot = pairs + (size_t)b * pair_stride + (size_t)x * PAIR_SLOT;
    uint4 p01 = make_uint4(0u, 0u, 0u, 0u), p23 = p01;
    if (c > 0) p01 = *reinterpret_cast<const uint4*>(slot);
    if (c > 2) p23 = *reinterpret_cast<const uint4*>(slot + 4);
    const uint32_t seg_lo = n_seg == 1 ? 0u : tile_seg[t0], seg_hi = n_seg == 1 ? 0u : tile_seg[min(t0 + 63u, T - 1u)];
    TileRef tr{0u, 0u, 0u};
    if (c > 0) tr = tile_ref(t, n_seg, n, tile_start, tile_seg);
    const uint32_t first_i = tr.start + (x % SUBS) * SUB;
    auto outside = [&](uint32_t e) { const uint32_t i = first_i + e; return (((core_bits[i >> 5] >> (i & 31u)) & 1u) ^ 1u) != 0u; };
    const uint32_t key[4] = {p01.x, p01.z, p23.x, p23.z}, ofs[4] = {p01.y, p01.w, p23.y, p23.w};
    uint32_t keep = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
        if (k < c && outside(ofs[k])) keep |= 1u << k;
    for (uint32_t k = 4; k < c; ++k)
        if (outside(slot[2 * k + 1])) keep |= 1u << k;
    const uint32_t mine = __popc(keep);
    // room in the lists: one reservation a block inside a segment, else one for each segment that a wave meets
    uint32_t at = NONE;
    auto reserve = [&](uint32_t seg, uint32_t total) {
        const uint32_t base = atomicAdd(&lists.count[(size_t)b * lists.count_stride + seg], total);
        const uint32_t cap = lists.first[seg + 1] - lists.first[seg];
        if (base + total <= cap && base + total >= base) return base;
        atomicOr(rerun, FLAG_RERUN);
        return NONE;
    };
    if (seg_lo == seg_hi) {
        uint32_t total;
        const uint32_t excl = block_excl_scan<4>(mine, wtot, total);
        if (threadIdx.x == 0) room = total ? reserve(seg_lo, total) : NONE;
        __syncthreads();
        if (mine && room != NONE) at = room + excl;
    } else {
        unsigned long long todo = __ballot(mine != 0u);
        while (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const uint32_t seg = __shfl(tr.seg, leader, 64);
            const bool in = mine != 0u && tr.seg == seg;
            const uint32_t v = in ? mine : 0u, incl = wave_incl_scan(v), total = last_lane(incl);
            uint32_t base = NONE;
            if ((int)lane == leader) base = reserve(seg, total);
            base = __shfl(base, leader, 64);
            if (in && base != NONE) at = base + incl - v;
            todo &= ~__ballot(in);
        }
    }
    if (at == NONE) return;
    uint2* out = lists.list + (size_t)b * lists.stride + lists.first[tr.seg] + at;
    const uint32_t pos0 = t * TILE + (x % SUBS) * SUB;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
        if ((keep >> k) & 1u) *out++ = make_uint2(key[k], pos0 + ofs[k]);
    for (uint32_t k = 4; k < c; ++k)
        if ((keep >> k) & 1u) *out++ = make_uint2(slot[2 * k], pos0 + slot[2 * k + 1]);
}

// Zones with many candidates in a sub-tile (draw with PAIRS = 0: small segments, whose slack is a large share of them):
// candidate bitmap and keys compacted per sub-tile.  One wave per tile; a wave collects the entries of its run of tiles
// in LDS and hands them over with one atomic when the segment changes or the buffer is full.  grid (blocks, n_workers).
constexpr int WIDE_KPL = 8;                     // keys per lane requested ahead: 128 per sub-tile
constexpr uint32_t WIDE_STAGE = 512;
__global__ __launch_bounds__(BLOCK) void k_explore_collect_wide(const uint32_t* __restrict__ core_bits, uint32_t n_words, uint64_t n,
                                                                const uint32_t* __restrict__ tile_start,
                                                                const uint32_t* __restrict__ tile_seg, uint32_t T, uint32_t n_seg,
                                                                const uint32_t* __restrict__ sure_bits, uint32_t* __restrict__ cnt_sel,
                                                                const uint32_t* __restrict__ cand_bits,
                                                                const uint32_t* __restrict__ cand_keys, uint64_t keys_stride,
                                                                ExploreLists lists, uint32_t* __restrict__ rerun)
{
    __shared__ uint32_t kb[4][SUBS * 16 * WIDE_KPL];
    __shared__ uint2 stage[4][WIDE_STAGE];
    const uint32_t b = blockIdx.y, lane = lane_id(), wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t wv = blockIdx.x * 4u + wid, waves = gridDim.x * 4u;
    const uint32_t t0 = (uint32_t)((uint64_t)T * wv / waves), t1 = (uint32_t)((uint64_t)T * (wv + 1u) / waves);
    uint32_t* kbw = kb[wid];
    uint2* sw = stage[wid];
    uint32_t fill = 0, held = 0;                 // entries staged, and their segment (uniform over the wave)
    // room for cnt entries in the list of segment seg; NULL: the list is full
    auto reserve = [&](uint32_t seg, uint32_t cnt) -> uint2* {
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&lists.count[(size_t)b * lists.count_stride + seg], cnt);
        base = __shfl(base, 0, 64);
        const uint32_t first = lists.first[seg], cap = lists.first[seg + 1] - first;
        if (base + cnt > cap || base + cnt < base) {
            if (lane == 0) atomicOr(rerun, FLAG_RERUN);
            return nullptr;
        }
        return lists.list + (size_t)b * lists.stride + first + base;
    };
    auto flush = [&]() {
        if (fill == 0) return;
        uint2* out = reserve(held, fill);
        wave_sync();
        if (out)
            for (uint32_t x = lane; x < fill; x += 64) out[x] = sw[x];
        wave_sync();
        fill = 0;
    };
    for (uint32_t t = t0; t < t1; ++t) {
        const TileRef tr = tile_ref(t, n_seg, n, tile_start, tile_seg);
        const size_t bt = (size_t)b * T + t;
        // everything this tile needs is requested here, before any of it is used
        const uint2 s2 = *reinterpret_cast<const uint2*>(sure_bits + bt * TILE_WORDS + 2 * lane);
        const uint2 c2 = *reinterpret_cast<const uint2*>(cand_bits + bt * TILE_WORDS + 2 * lane);
        const uint32_t* keys = cand_keys + (size_t)b * keys_stride + tr.start;
        uint32_t kv[WIDE_KPL];
        load_sublists<WIDE_KPL>(keys, lane, kv);
        uint32_t kw[2];
        bitmap_window(core_bits, n_words, tr.start + lane * 64u, kw);
        const uint32_t sure = wave_sum(__popc(s2.x & ~kw[0]) + __popc(s2.y & ~kw[1]));
        if (lane == 0) cnt_sel[bt] = sure;
        const uint32_t cw[2] = {c2.x, c2.y};
        const uint32_t newc = __popc(cw[0] & ~kw[0]) + __popc(cw[1] & ~kw[1]);
        const uint32_t incl = wave_incl_scan(newc), total = last_lane(incl);
        if (total == 0) continue;
        const bool direct = total > WIDE_STAGE;
        if (fill && (held != tr.seg || direct || fill + total > WIDE_STAGE)) flush();
        uint2* out = direct ? reserve(tr.seg, total) : nullptr;
        wave_sync();
#pragma unroll
        for (int i = 0; i < WIDE_KPL; ++i) kbw[(lane >> 4) * (16 * WIDE_KPL) + (lane & 15u) + 16 * i] = kv[i];
        wave_sync();
        const uint32_t pos = sublist_pos(lane, __popc(cw[0]) + __popc(cw[1]));      // place of the lane's first candidate
        const uint32_t sub = pos >> 10;
        uint32_t j = pos & (SUB - 1u), o = incl - newc;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t m = cw[h];
            while (m) {
                const uint32_t p = __ffs(m) - 1;
                m &= m - 1;
                const uint32_t jj = j++;
                if ((kw[h] >> p) & 1u) continue;
                const uint32_t key = (jj < 16u * WIDE_KPL) ? kbw[sub * (16 * WIDE_KPL) + jj] : keys[sub * SUB + jj];
                const uint2 e = make_uint2(key, t * TILE + lane * 64u + (uint32_t)h * 32u + p);
                if (!direct) sw[fill + o] = e;
                else if (out) out[o] = e;
                ++o;
            }
        }
        if (!direct) { fill += total; held = tr.seg; }
    }
    flush();
}

// ---------------------------------------------------------------------------------------
// One block per (segment, worker).  The sure parameters outside the core come off the demand; the rest is taken from the
// list: a radix descent, 12 bits a level from the top of the zone's width, that ends as soon as a whole bin is
// wanted, ties at the threshold key going to the lowest positions.  The list's first KEEP * NT entries stay in registers
// from the first level to the last, longer ones are read again.  A chosen candidate is set in the sure bitmap and added to its
// tile's count; the prefix of the counts gives the tile offsets (every wave owns a run of tiles, whose sums
// are known beforehand).  Bound by latency: a chain of some ten trips to the L2 and as many block barriers, and by the
// atomics that mark the chosen, two misses each, from one compute unit: 11 us at 10^6 parameters, 54 us for the 20,400
// entries of 20*10^6 at 17 %, 53 us for 19,000 entries in 33,779 tiles.  More blocks to a list, each marking a share, take
// 43 us for the 20,400, but are slower on short lists (14 -> 17 us for 228 of them) and beside a kernel that fills the chip.
// A demand that the zones cannot meet raises the rerun flag.  grid (n_seg, n_workers), NT threads.
// ---------------------------------------------------------------------------------------
constexpr uint32_t TIE_CAP = 1024;
constexpr int KEEP = 8;
template <int NT>
__global__ __launch_bounds__(NT) void k_explore_select(const SegState* __restrict__ states, const uint32_t* __restrict__ seg_first_tile,
                                                       uint32_t T, uint32_t n_seg, ExploreLists lists, uint32_t* __restrict__ cnt_sel,
                                                       uint32_t* __restrict__ sure_bits, MutPtrTab out_off, uint32_t* __restrict__ rerun)
{
    constexpr int NWV = NT / 64, NBIN = 4096, PER = NBIN / NT;
    __shared__ uint32_t hist[NBIN];
    __shared__ uint32_t wsum[NWV], wtot[NWV], sh[4], ntie;
    __shared__ uint32_t tpos[TIE_CAP];
    const uint32_t seg = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
    const SegState* st = states + seg;
    const uint32_t f0 = n_seg == 1 ? 0u : seg_first_tile[seg], f1 = n_seg == 1 ? T : seg_first_tile[seg + 1];
    const uint32_t cap = lists.first[seg + 1] - lists.first[seg];
    uint32_t* counter = lists.count + (size_t)b * lists.count_stride + seg;
    const uint32_t cnt = *counter;
    const uint2* list = lists.list + (size_t)b * lists.stride + lists.first[seg];
    const uint32_t need0 = st->need0, base = st->out_base, bits = st->bits;
    if (cnt > cap) {                                         // the rerun flag is up
        __syncthreads();
        if (tid == 0) *counter = 0;
        return;
    }
    uint32_t key[KEEP], pos[KEEP];
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const uint32_t x = tid + (uint32_t)i * NT;
        key[i] = 0; pos[i] = NONE;
        if (x < cnt) { const uint2 e = list[x]; key[i] = e.x; pos[i] = e.y; }
    }
    // every wave owns tiles [w0, w1) of the segment
    uint32_t* cs = cnt_sel + (size_t)b * T + f0;
    const uint32_t nt = f1 - f0, per = (nt + NWV - 1u) / NWV;
    const uint32_t w0 = min(wid * per, nt), w1 = min(w0 + per, nt);
    {
        uint32_t sum = 0;
#pragma unroll 8
        for (uint32_t x = w0 + lane; x < w1; x += 64) sum += cs[x];
        sum = wave_sum(sum);
        if (lane == 0) wsum[wid] = sum;
    }
    if (tid == 0) ntie = 0;
    __syncthreads();
    if (tid == 0) *counter = 0;                              // read by every thread; clear for the next request
    uint32_t nsure = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) nsure += wsum[w];
    __syncthreads();                                         // the marks below add to wsum
    if (nsure > need0 || need0 - nsure > cnt) {              // a zone missed: the request again, exactly
        if (tid == 0) atomicOr(rerun, FLAG_RERUN);
        return;
    }
    // keys >> shift above `prefix` are taken, those equal to it are `equal` many, of which `need` are wanted
    uint32_t need = need0 - nsure, shift = bits, prefix = 0, equal = cnt;
    while (need != 0 && need != equal && shift != 0) {
        const uint32_t nb = min(12u, shift), up = shift;
        shift -= nb;
        for (uint32_t x = tid; x < NBIN; x += NT) hist[x] = 0;
        __syncthreads();
        const uint32_t mask = (1u << nb) - 1u;
#pragma unroll
        for (int i = 0; i < KEEP; ++i)
            if (pos[i] != NONE && (uint32_t)((uint64_t)key[i] >> up) == prefix) atomicAdd(&hist[(key[i] >> shift) & mask], 1u);
        for (uint32_t x = tid + KEEP * NT; x < cnt; x += NT) {
            const uint32_t k = list[x].x;
            if ((uint32_t)((uint64_t)k >> up) == prefix) atomicAdd(&hist[(k >> shift) & mask], 1u);
        }
        __syncthreads();
        uint32_t c[PER], sum = 0;
        const uint32_t low = NBIN - (tid + 1u) * PER;        // this thread's bins; thread 0 has the largest
#pragma unroll
        for (int e = 0; e < PER; ++e) { c[e] = hist[low + e]; sum += c[e]; }
        uint32_t total;
        const uint32_t excl = block_excl_scan<NWV>(sum, wtot, total);
        if (excl < need && need <= excl + sum) {
            uint32_t run = excl;
#pragma unroll
            for (int e = PER - 1; e >= 0; --e) {
                if (run < need && need <= run + c[e]) { sh[0] = low + (uint32_t)e; sh[1] = need - run; sh[2] = c[e]; }
                run += c[e];
            }
        }
        __syncthreads();
        prefix = (prefix << nb) | sh[0]; need = sh[1]; equal = sh[2];
        __syncthreads();
    }
    const bool all = need == equal;                          // the whole last bin is wanted
    const uint32_t quota = need;
    auto take = [&](uint32_t p) {
        const uint32_t t = p / TILE, o = p % TILE;
        atomicOr(&sure_bits[((size_t)b * T + t) * TILE_WORDS + (o >> 5)], 1u << (o & 31u));
        atomicAdd(&cs[t - f0], 1u);
        atomicAdd(&wsum[(t - f0) / per], 1u);
    };
    auto decide = [&](uint32_t k, uint32_t p) {
        const uint32_t d = (uint32_t)((uint64_t)k >> shift);
        if (d > prefix || (d == prefix && all)) take(p);
        else if (d == prefix && quota != 0) {                // shift is 0 here: equal keys, not all of them wanted
            const uint32_t slot = atomicAdd(&ntie, 1u);
            if (slot < TIE_CAP) tpos[slot] = p;
        }
    };
    if (need0 != nsure) {
#pragma unroll
        for (int i = 0; i < KEEP; ++i)
            if (pos[i] != NONE) decide(key[i], pos[i]);
        for (uint32_t x = tid + KEEP * NT; x < cnt; x += NT) { const uint2 e = list[x]; decide(e.x, e.y); }
        __syncthreads();
        const uint32_t nt_all = ntie;
        if (nt_all > TIE_CAP) {
            if (tid == 0) atomicOr(rerun, FLAG_RERUN);
            return;
        }
        for (uint32_t q = tid; q < nt_all; q += NT) {
            const uint32_t p = tpos[q];
            uint32_t rank = 0;
            for (uint32_t r = 0; r < nt_all; ++r) rank += tpos[r] < p ? 1u : 0u;
            if (rank < quota) take(p);
        }
    }
    __syncthreads();
    // Tile offsets: the counts were added to by other waves of this block, hence the atomic loads.  Consecutive lanes take
    // consecutive tiles; eight tiles to a lane made every load and store touch sixteen lines: 43 us for 33,779 tiles.
    uint32_t* off = static_cast<uint32_t*>(out_off.p[b]) + f0;
    uint32_t run = base;
    for (uint32_t w = 0; w < wid; ++w) run += wsum[w];
    for (uint32_t x0 = w0; x0 < w1; x0 += 512) {
        uint32_t v[8];
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e) {
            const uint32_t x = x0 + e * 64u + lane;
            v[e] = x < w1 ? __hip_atomic_load(&cs[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        }
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e) {
            if (x0 + e * 64u >= w1) break;                   // uniform: a scan costs a short segment a microsecond
            const uint32_t x = x0 + e * 64u + lane, incl = wave_incl_scan(v[e]);
            if (x < w1) off[x] = run + incl - v[e];
            run += last_lane(incl);
        }
    }
    if (f1 == T && tid == 0) off[nt] = base + need0;
}

// =======================================================================================
// Explorer, exact rerun.  When the zones of a draw missed (the rerun flag is up; once in about
// 10^9 draws, or forced by a test switch) this routine redoes the whole request from the
// definition, slowly and with no assumption: per worker one block walks every segment,
// finds the need-th smallest Philox word among the parameters outside the core by a
// three-pass radix descent over ALL of them (11 + 11 + 10 bits, words recomputed in every
// pass), then emits tile by tile in index order, ties at the threshold word going to the
// lowest indices.  By a block of NT threads; h: EXACT_NBIN words of LDS.
// =======================================================================================
__device__ __forceinline__ uint32_t explore_word(uint32_t i, uint32_t worker, PhiloxKey pk)
{
    uint32_t r[4];
    philox4x32_10(i >> 2, worker, pk.it_lo, pk.it_hi, pk.seed_lo, pk.seed_hi, r);
    const uint32_t c = i & 3u;
    return c == 0 ? r[0] : c == 1 ? r[1] : c == 2 ? r[2] : r[3];
}

constexpr uint32_t EXACT_NBIN = 2048;
template <int NT>
__device__ __forceinline__ void explore_exact(uint32_t* h, const uint32_t* __restrict__ core_bits, const uint32_t* __restrict__ tile_start,
                              const uint32_t* __restrict__ seg_first_tile, uint32_t T, uint32_t n_seg,
                              const SegState* __restrict__ states, uint32_t worker, PhiloxKey pk, uint32_t* __restrict__ out,
                              uint32_t* __restrict__ off, uint32_t expected, uint32_t* __restrict__ flags)
{
    constexpr uint32_t PER = EXACT_NBIN / NT, EACH = TILE / NT;      // bins, and parameters of a tile, per thread
    constexpr int NWV = NT / 64;
    static_assert(EACH <= 32, "a thread's parameters of a tile are flags of one word");
    __shared__ uint32_t wtot[NWV];
    __shared__ uint32_t sh[4];
    const uint32_t tid = threadIdx.x;
    uint32_t run = 0;                                // indices emitted so far (uniform)
    for (uint32_t seg = 0; seg < n_seg; ++seg) {
        const uint32_t f0 = seg_first_tile[seg], f1 = seg_first_tile[seg + 1];
        uint32_t need = states[seg].need0;
        // ---- the need-th smallest word: descent over bits 31..21, 20..10, 9..0
        uint32_t prefix = 0, short_of = 0;
        const uint32_t shifts[3] = {21u, 10u, 0u}, nbits[3] = {11u, 11u, 10u};
        for (int p = 0; p < 3 && need != 0 && !short_of; ++p) {
            for (uint32_t x = tid; x < EXACT_NBIN; x += NT) h[x] = 0;
            __syncthreads();
            const uint32_t hi_shift = shifts[p] + nbits[p];        // bits above this pass's digit
            for (uint32_t t = f0; t < f1; ++t) {
                const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
                for (uint32_t e = tid; e < len; e += NT) {
                    const uint32_t i = start + e;
                    if ((core_bits[i >> 5] >> (i & 31u)) & 1u) continue;
                    const uint32_t r = explore_word(i, worker, pk);
                    if (hi_shift < 32u && (r >> hi_shift) != prefix) continue;
                    atomicAdd(&h[(r >> shifts[p]) & ((1u << nbits[p]) - 1u)], 1u);
                }
            }
            __syncthreads();
            // the bin that holds the need-th smallest: consecutive bins per thread, ascending
            uint32_t sum = 0;
#pragma unroll
            for (uint32_t e = 0; e < PER; ++e) sum += h[PER * tid + e];
            uint32_t total;
            const uint32_t excl = block_excl_scan<NWV>(sum, wtot, total);
            if (tid == 0) sh[2] = (total < need) ? 1u : 0u;
            if (excl < need && need <= excl + sum) {
                uint32_t before = excl, bin = PER * tid;
                while (need > before + h[bin]) before += h[bin++];
                sh[0] = bin; sh[1] = need - before;
            }
            __syncthreads();
            if (sh[2]) { short_of = 1; if (tid == 0) atomicOr(&flags[1], 2u); }     // fewer eligible parameters than requested
            else { prefix = (prefix << nbits[p]) | sh[0]; need = sh[1]; }
            __syncthreads();
        }
        // words below tau are taken, of the words equal to tau the first `need` in index order
        const uint32_t tau = short_of ? 0xFFFFFFFFu : prefix;
        const uint32_t take_all = short_of;
        const uint32_t want = states[seg].need0;
        uint32_t ties_seen = 0;                      // uniform
        // ---- ordered emission, tile by tile (consecutive parameters per thread)
        for (uint32_t t = f0; t < f1; ++t) {
            const uint32_t start = tile_start[t], len = tile_start[t + 1] - start;
            uint32_t sel = 0, tie = 0;
            if (want != 0) {
#pragma unroll 1
                for (uint32_t c = 0; c < EACH; ++c) {
                    const uint32_t e = EACH * tid + c;
                    if (e >= len) continue;
                    const uint32_t i = start + e;
                    if ((core_bits[i >> 5] >> (i & 31u)) & 1u) continue;
                    const uint32_t r = explore_word(i, worker, pk);
                    if (take_all || r < tau) sel |= 1u << c;
                    else if (r == tau) tie |= 1u << c;
                }
            }
            uint32_t tie_total;
            const uint32_t tie_excl = block_excl_scan<NWV>(__popc(tie), wtot, tie_total);
            uint32_t rank = ties_seen + tie_excl;
#pragma unroll 1
            for (uint32_t c = 0; c < EACH; ++c)
                if ((tie >> c) & 1u) { if (rank < need) sel |= 1u << c; ++rank; }
            ties_seen += tie_total;
            uint32_t sel_total;
            uint32_t o = run + block_excl_scan<NWV>(__popc(sel), wtot, sel_total);
            if (tid == 0) off[t] = run;
#pragma unroll 1
            for (uint32_t c = 0; c < EACH; ++c)
                if ((sel >> c) & 1u) { if (o < expected) out[o] = start + EACH * tid + c; ++o; }
            run += sel_total;
        }
    }
    if (tid == 0) {
        off[T] = run;
        if (run != expected) atomicOr(&flags[1], 1u);
    }
}

// Ordered emission from the sure bitmap (chosen candidates included) minus the core.  One wave per tile and BPW batches.
// With the rerun flag up the first BPW blocks of a batch group redo the request instead, one batch each (k_explore_select and
// everything before it is void then); at most 64 registers, eight waves to a SIMD.
// NT = 256, for a request on the side stream: beside a kernel of small blocks that fills the chip a block of sixteen waves
// waits until so many are free at once on one unit (beside k_merge 330 to 600 us for 138*10^6 parameters and 8 workers,
// 59 alone; a launch of sixteen-wave blocks that read the flag and end, as the rerun was there, 4 to 275 us).
// grid (max(BPW, ceil(T / waves of a block)), ceil(nbatch / BPW)).
template <int BPW, int NT>
__global__ __launch_bounds__(NT, 8) void k_explore_emit(const uint32_t* __restrict__ core_bits, uint32_t n_words, uint64_t n,
                                                       const uint32_t* __restrict__ tile_start,
                                                       const uint32_t* __restrict__ tile_seg,
                                                       const uint32_t* __restrict__ seg_first_tile, uint32_t T, uint32_t n_seg,
                                                       uint32_t nbatch, const SegState* __restrict__ states, uint32_t worker0,
                                                       PhiloxKey pk, const uint32_t* __restrict__ sure_bits, MutPtrTab out_off,
                                                       MutPtrTab out_idx, uint32_t expected, RerunFlag rerun, uint32_t* __restrict__ flags)
{
    constexpr uint32_t WAVES = NT / 64;
    __shared__ __align__(8) uint16_t stage[WAVES][EMIT_STAGE];
    static_assert(sizeof stage >= EXACT_NBIN * sizeof(uint32_t), "the rerun counts in the stage");
    const uint32_t b0 = blockIdx.y * BPW;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *rerun.next = 0;
    if (*rerun.now != 0) {                       // nobody raises the flag while this kernel runs
        const uint32_t b = b0 + blockIdx.x;
        if (blockIdx.x < (uint32_t)BPW && b < nbatch)
            explore_exact<NT>(reinterpret_cast<uint32_t*>(stage), core_bits, tile_start, seg_first_tile, T, n_seg, states, worker0 + b, pk,
                              static_cast<uint32_t*>(out_idx.p[b]), static_cast<uint32_t*>(out_off.p[b]), expected, flags);
        return;
    }
    const uint32_t t = blockIdx.x * WAVES + (threadIdx.x >> 6), lane = lane_id();
    if (t >= T) return;
    const TileRef tr = tile_ref(t, n_seg, n, tile_start, tile_seg);
    uint2 s2[BPW];
    uint32_t off_t[BPW];
#pragma unroll
    for (int bb = 0; bb < BPW; ++bb) {
        s2[bb] = make_uint2(0u, 0u); off_t[bb] = 0;
        if (b0 + bb < nbatch) {
            s2[bb] = *reinterpret_cast<const uint2*>(sure_bits + ((size_t)(b0 + bb) * T + t) * TILE_WORDS + 2 * lane);
            off_t[bb] = static_cast<const uint32_t*>(out_off.p[b0 + bb])[t];
        }
    }
    uint32_t kw[2];
    bitmap_window(core_bits, n_words, tr.start + lane * 64u, kw);
#pragma unroll
    for (int bb = 0; bb < BPW; ++bb) {
        const uint32_t b = b0 + bb;
        if (b >= nbatch) break;
        const uint32_t fm0 = s2[bb].x & ~kw[0], fm1 = s2[bb].y & ~kw[1];
        const uint32_t ocnt = __popc(fm0) + __popc(fm1);
        const uint32_t incl = wave_incl_scan(ocnt);
        uint32_t* out = static_cast<uint32_t*>(out_idx.p[b]);
        if (t == T - 1 && lane == 63 && off_t[bb] + incl != expected) atomicOr(&flags[1], 1u);
        emit_indices(fm0, fm1, incl, tr.start, off_t[bb], expected, stage[threadIdx.x >> 6], out);
    }
}

}  // namespace slimdp
