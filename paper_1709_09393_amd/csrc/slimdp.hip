// libslimdp host side: the C ABI of include/slimdp.h.  Argument checks, workspace carving
// and kernel launches only; every step of the path runs in the kernels of slimdp_kernels.h,
// slimdp_core.h and slimdp_explore.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "slimdp.h"
#include "slimdp_kernels.h"
#include "slimdp_core.h"
#include "slimdp_explore.h"

using namespace slimdp;

namespace {

thread_local std::string g_create_error;

struct Tiling {
    std::vector<uint32_t> tile_start;      // T+1
    std::vector<uint32_t> tile_seg;        // T
    std::vector<uint32_t> seg_first_tile;  // n_seg+1
    bool word_aligned = true;              // every tile starts on a bitmap word
    bool quad_aligned = true;              // every tile starts on a Philox block (index divisible by 4)
    bool mostly_quads = true;              // ... at least every other one does
};

bool valid_shape(uint64_t n, uint32_t n_seg, const uint64_t* seg_off)
{
    if (n == 0 || n > SLIMDP_MAX_N || n_seg == 0 || n_seg > SLIMDP_MAX_SEGMENTS || !seg_off) return false;
    if (seg_off[0] != 0 || seg_off[n_seg] != n) return false;
    for (uint32_t s = 0; s < n_seg; ++s)
        if (seg_off[s + 1] <= seg_off[s]) return false;
    return true;
}

Tiling make_tiling(uint64_t n, uint32_t n_seg, const uint64_t* seg_off)
{
    Tiling tl;
    tl.seg_first_tile.resize(n_seg + 1);
    uint64_t quads = 0;
    for (uint32_t s = 0; s < n_seg; ++s) {
        tl.seg_first_tile[s] = (uint32_t)tl.tile_seg.size();
        for (uint64_t a = seg_off[s]; a < seg_off[s + 1]; a += TILE) {
            tl.tile_start.push_back((uint32_t)a);
            tl.tile_seg.push_back(s);
            if (a & 31u) tl.word_aligned = false;
            if (a & 3u) tl.quad_aligned = false; else ++quads;
        }
    }
    tl.seg_first_tile[n_seg] = (uint32_t)tl.tile_seg.size();
    tl.mostly_quads = 2 * quads >= tl.tile_seg.size();
    tl.tile_start.push_back((uint32_t)n);   // n <= 2^31
    return tl;
}

uint64_t count_tiles(uint64_t n, uint32_t n_seg, const uint64_t* seg_off)
{
    (void)n;
    uint64_t T = 0;
    for (uint32_t s = 0; s < n_seg; ++s) T += (seg_off[s + 1] - seg_off[s] + TILE - 1) / TILE;
    return T;
}

// Where each segment's list of explorer candidates begins.  The zones of a request for m of n_s parameters hold
// 2 (6 sqrt(m) + 32) words outside the core on average (explorer_init); the room is for the largest m and eight
// standard deviations more.
std::vector<uint32_t> list_starts(uint32_t n_seg, const uint64_t* seg_off)
{
    std::vector<uint32_t> first(n_seg + 1, 0u);
    for (uint32_t s = 0; s < n_seg; ++s) {
        const uint64_t ns = seg_off[s + 1] - seg_off[s];
        const double mean = 2.0 * (6.0 * std::sqrt((double)ns) + 32.0);
        const uint64_t cap = (uint64_t)std::ceil(mean + 8.0 * std::sqrt(mean)) + 64;
        first[s + 1] = first[s] + (uint32_t)(cap < ns ? cap : ns);          // the sum is at most n
    }
    return first;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// One linear pass hands out the workspace; run once with base == nullptr to size it.
struct Carver {
    char* base;
    size_t pos = 0;
    explicit Carver(char* b) : base(b) {}
    template <class Tp> Tp* take(size_t count)
    {
        pos = align_up(pos, 256);
        Tp* p = base ? reinterpret_cast<Tp*>(base + pos) : nullptr;
        pos += count * sizeof(Tp);
        return p;
    }
};

}  // namespace

struct slimdp_ctx {
    uint64_t n = 0;
    uint32_t maxW = 0, n_seg = 0, T = 0;
    uint64_t seed = 0;
    hipStream_t stream = nullptr;
    // an announced explorer draw can run beside the caller's stream: pure integer work that fills the
    // arithmetic units the memory-bound kernels leave idle
    hipStream_t side = nullptr;
    hipEvent_t ev_consumed = nullptr;      // main stream: everything enqueued before a side-stream draw (readers of its buffers)
    hipEvent_t ev_drawn = nullptr;         // side stream: the announced draw is complete
    bool side_pending = false;             // a side draw was launched and the main stream has not waited for it yet
    bool draw_fresh = false;               // ... and no call that takes lists has been enqueued since
    // asynchronous slimdp_sample_explore requests (option "explore_async") that the main stream has not waited for yet:
    // their completion events on the side stream and the address ranges they write
    static constexpr int N_PENDING = 4;
    struct PendingExplore {
        hipEvent_t ev = nullptr;
        bool live = false;
        uint64_t seq = 0;
        uint32_t nw = 0;
        uintptr_t idx[MAXW] = {}, off[MAXW] = {};
        uint64_t idx_bytes = 0, off_bytes = 0;
    } pend[N_PENDING];
    uint64_t pend_seq = 0;
    uint64_t asked_epoch = ~0ull;          // the core epoch at the last explorer request
    int64_t opt_explore_async = 0;         // 1: requests on the side stream where that pays (stays_on_main), 2: test, all of them
    int device = 0, cus = 256;
    std::vector<uint64_t> seg_off;
    Tiling tl;
    char* ws = nullptr;
    size_t ws_bytes = 0;
    uint64_t keys_stride = 0;
    // device tables
    uint32_t *d_tile_start = nullptr, *d_tile_seg = nullptr, *d_seg_first_tile = nullptr, *d_flags = nullptr;
    // core selection
    CoreState* c_state = nullptr;
    CorePlan* c_plan = nullptr;            // core sizes per segment (segmented models)
    std::vector<uint64_t> c_plan_k;        // the sizes c_plan holds
    uint32_t *c_hist = nullptr, *c_gt_bits = nullptr, *c_cand_bits = nullptr, *c_cand_keys = nullptr;
    uint2 *c_tile_pre = nullptr, *c_group_tail = nullptr;
    uint32_t *c_pred = nullptr, *c_used = nullptr;   // predicted level-0 threshold bin per segment; the bin the scoring pass sorted against
    bool cls_by_score = false;                       // the last scoring pass classified whole tiles against c_pred
    bool hist_clean = true;                          // c_hist is zero once everything enqueued has run (a selection leaves it so)
    bool recorded = false;                           // a call of this context went into a graph: see device_state_known
    uint32_t *c_cnt_gt = nullptr, *c_cnt_cand = nullptr;
    // explorer selection (batch = worker)
    SegState* e_state = nullptr;           // per segment, the same for every worker
    SegState* e_draw_state = nullptr;      // zone bounds of the announced draw (side stream)
    std::vector<SegInit> e_state_holds, e_draw_holds;      // what they hold; empty: not known
    bool lists_clean = false;              // the lists' counters and the coming request's rerun flag are zero
    uint32_t rerun_turn = 0;               // which of the two rerun flags that is
    // sizes and zones of the last requests, kept while the sizes stay the same
    struct Plan {
        bool valid = false;
        std::vector<uint64_t> k_seg, m_seg;
        uint32_t n_workers = 0;
        int64_t force = 0, tail = 0;
        std::vector<SegInit> init;
        uint64_t M = 0;
        bool narrow = false, pairs = false;
    } plan;
    uint32_t *e_sure_bits = nullptr, *e_cand_bits = nullptr;
    uint32_t* e_pair_keys = nullptr;       // narrow zones: per sub-tile a slot of (key, offset) pairs
    uint64_t pair_stride = 0;              // words per worker of the pair slots
    uint32_t* e_cand_keys = nullptr;       // wide zones: candidate keys compacted per sub-tile over the whole index range;
                                           // its own allocation, made by the first request that needs it
    uint32_t *e_cnt_cand = nullptr, *e_cnt_sel = nullptr;
    uint2* e_list = nullptr;               // candidates outside the core, per (worker, segment): see ExploreLists
    uint32_t *e_list_count = nullptr, *d_list_first = nullptr;
    std::vector<uint32_t> list_first;      // n_seg+1
    // host state
    uint64_t epoch = 0;
    bool hist_pending = false;
    const float* hist_score = nullptr;
    int64_t opt_force_fallback = 0;
    int64_t opt_per_tile_tail = 0;
    int64_t opt_strided = 1;               // flat model: persistent blocks take every P-th tile
    int64_t opt_side_blocks = 2;           // blocks per compute unit of a side-stream draw
    int64_t opt_hint_mode = 0;             // 0: the announced draw rides inside slimdp_score; 1: side stream
    // speculative packing: its own allocation, made when the option is switched on
    struct Spec {
        bool on = false;
        char* mem = nullptr;
        uint32_t* lo[2] = {nullptr, nullptr};   // capture bound per segment: [cur] read by the scoring pass, the other written by the selection
        uint32_t* fail = nullptr;               // per segment: the selection's threshold fell below the capture bound
        uint2* bits = nullptr;
        float* vals = nullptr;
        float* evals = nullptr;                 // explorer capture, where there is room for one (see expl_capture_words)
        char* evals_mem = nullptr;              // ... of its own, for option "explore_keep" = 2 where the sizes ask for none
        int cur = 0;
        bool next_written = false;              // a selection has refreshed lo[cur ^ 1] since the last capture
        bool bound_valid = false;               // lo[cur] comes from a selection (else: nothing, or a sampled estimate)
        uint32_t* sample = nullptr;             // keys of the sampled significances (flat model)
        // the capture made by the last slimdp_score, and the selection that used that score
        bool captured = false;
        const float* score = nullptr;
        const float* g[MAXW] = {};
        uint32_t W = 0;
        uint64_t core_epoch = 0;                // 0: no selection on the captured score yet
        // explorer values kept beside it: slots a sub-tile and worker (0: none), for how many workers; void once another draw
        // has gone to the bitmap that tells which they are
        uint32_t expl_slots = 0;
    } spec;
    int64_t opt_pack_nbuf = 2;
    int64_t opt_pack_kernel = 1;           // general pack: 1 = loading and storing waves apart, 0 = one set of waves
    int64_t opt_pull_kernel = 1;           // local overwrite of a pull: 1 = a pass that streams the local models, 0 = scattered writes
    int64_t opt_build_blocks = 4;          // blocks per compute unit of the core candidate pass
    int64_t opt_pack_core_blocks = 0;      // blocks per compute unit of the pack from the capture (0: one per 1024 list entries)
    int64_t opt_core_predict = 1;          // the flat scoring kernel sorts whole tiles against the predicted threshold bin (0: never; 2: test, a wrong bin)
    int64_t opt_explore_keep = 1;          // the scoring pass keeps the explorers' values beside the core's: 1 by size, 2 whenever it can, 0 never
    int64_t opt_score_pipeline = 1;        // flat aligned models: the scoring kernel with two rounds of loads in flight
    int64_t opt_expected_core = -1;        // core size the next selection will ask for (flat model), if the caller says
    int64_t opt_estimate_bias = 0;         // test switch: added to a sampled capture bound
    uint64_t last_K = 0;                   // core size of the last selection
    bool have_last_K = false;
    // explorer draw announced by slimdp_explore_hint (hint) / already drawn inside slimdp_score (pre)
    struct Draw {
        bool valid = false;
        uint64_t iteration = 0;
        uint32_t worker0 = 0, n_workers = 0;
        std::vector<uint64_t> k_seg, m_seg;
        bool pairs = false;          // drawn in the format of narrow zones (pairs)
        bool same(uint64_t it, uint32_t w0, uint32_t nw, const uint64_t* k, const uint64_t* m, uint32_t n_seg) const
        {
            if (!valid || it != iteration || w0 != worker0 || nw != n_workers) return false;
            for (uint32_t s = 0; s < n_seg; ++s)
                if (k[s] != k_seg[s] || m[s] != m_seg[s]) return false;
            return true;
        }
    } hint, pre;
    std::string err;
};

namespace {

// every number of tiles that the interface serves fits the groups' table
static_assert(core_groups((uint32_t)(SLIMDP_MAX_N / TILE + SLIMDP_MAX_SEGMENTS), 1u) <= CORE_GROUPS, "groups of tiles");

// Tables and the buffers of the core selection (all that a selection without explorers needs).  The histogram comes
// first: in the static scratch array it is found at the same place whatever the size of the call before.
void carve_core(slimdp_ctx* c, Carver& cv)
{
    const size_t T = c->T, S = c->n_seg;
    c->c_hist = cv.take<uint32_t>(S * H_STRIDE);
    c->d_tile_start = cv.take<uint32_t>(T + 1);
    c->d_tile_seg = cv.take<uint32_t>(T);
    c->d_seg_first_tile = cv.take<uint32_t>(S + 1);
    c->d_list_first = cv.take<uint32_t>(S + 1);
    c->c_pred = cv.take<uint32_t>(S);
    c->d_flags = cv.take<uint32_t>(64);          // the tables above and the flags are uploaded in one copy: see slimdp_create
    c->c_state = cv.take<CoreState>(S);
    c->c_plan = cv.take<CorePlan>(S);
    c->c_gt_bits = cv.take<uint32_t>(T * TILE_WORDS);
    c->c_cand_bits = cv.take<uint32_t>(T * TILE_WORDS);
    c->c_cand_keys = cv.take<uint32_t>(c->keys_stride);
    c->c_cnt_gt = cv.take<uint32_t>(T * SUBS);
    c->c_cnt_cand = cv.take<uint32_t>(T * SUBS);
    c->c_tile_pre = cv.take<uint2>(T);
    c->c_group_tail = cv.take<uint2>(CORE_GROUPS);
    c->c_used = cv.take<uint32_t>(S);
}

void carve(slimdp_ctx* c, Carver& cv)
{
    const size_t T = c->T, S = c->n_seg, B = c->maxW;
    carve_core(c, cv);
    c->e_state = cv.take<SegState>(S);
    c->e_draw_state = cv.take<SegState>(S);
    c->e_sure_bits = cv.take<uint32_t>(B * T * TILE_WORDS);
    c->e_cand_bits = cv.take<uint32_t>(B * T * TILE_WORDS);
    c->e_list_count = cv.take<uint32_t>(B * align_up(S, 32));
    c->e_list = cv.take<uint2>(B * (size_t)c->list_first[S]);
    c->e_pair_keys = cv.take<uint32_t>(B * c->pair_stride);
    c->e_cnt_cand = cv.take<uint32_t>(B * T * SUBS);
    c->e_cnt_sel = cv.take<uint32_t>(B * T);
}

int fail(slimdp_ctx* c, int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf; else g_create_error = buf;
    return code;
}

int hip_fail(slimdp_ctx* c, hipError_t e, const char* what)
{
    return fail(c, SLIMDP_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define SLIMDP_HIP(c, call)                                        \
    do {                                                           \
        hipError_t e__ = (call);                                   \
        if (e__ != hipSuccess) return hip_fail((c), e__, #call);   \
    } while (0)

#define SLIMDP_LAUNCHED(c, name)                                   \
    do {                                                           \
        hipError_t e__ = hipGetLastError();                        \
        if (e__ != hipSuccess) return hip_fail((c), e__, name);    \
    } while (0)

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

uint32_t fill_grid(uint64_t count) { uint64_t g = (count + 255) / 256; return (uint32_t)(g < 1 ? 1 : (g > 4096 ? 4096 : g)); }

int fill(slimdp_ctx* c, uint32_t* p, uint64_t count, uint32_t v)
{
    if (count == 0) return SLIMDP_OK;
    hipLaunchKernelGGL(k_fill_u32, dim3(fill_grid(count)), dim3(256), 0, c->stream, p, count, v);
    SLIMDP_LAUNCHED(c, "k_fill_u32");
    return SLIMDP_OK;
}

RerunFlag rerun_flag(const slimdp_ctx* c) { return RerunFlag{c->d_flags + 2 * c->rerun_turn, c->d_flags + 2 * (c->rerun_turn ^ 1u)}; }

// Brings st to init, unless it holds that already; clear: the list counters and the rerun flag as well.  Only where the host knows
// what the device holds (known) is anything left out.
int init_states(slimdp_ctx* c, SegState* st, std::vector<SegInit>& holds, const std::vector<SegInit>& init, bool known, bool clear, uint32_t nbatch,
                hipStream_t stream)
{
    const bool same = known && holds.size() == init.size() && memcmp(holds.data(), init.data(), init.size() * sizeof(SegInit)) == 0;
    if (same && !clear) return SLIMDP_OK;
    holds.clear();
    for (uint32_t s0 = 0; s0 < c->n_seg; s0 += INIT_CHUNK) {
        SegInitChunk chunk;
        const uint32_t cnt = (c->n_seg - s0 < (uint32_t)INIT_CHUNK) ? c->n_seg - s0 : (uint32_t)INIT_CHUNK;
        memset(&chunk, 0, sizeof chunk);
        for (uint32_t j = 0; j < cnt; ++j) chunk.s[j] = init[s0 + j];
        const uint32_t threads = cnt * (clear ? nbatch : 1u);
        hipLaunchKernelGGL(k_explore_init, dim3((threads + 255) / 256), dim3(256), 0, stream, st, chunk, s0, cnt, nbatch,
                           clear ? c->e_list_count : nullptr, (uint32_t)align_up(c->n_seg, 32),
                           clear && s0 == 0 ? rerun_flag(c).now : nullptr);
        SLIMDP_LAUNCHED(c, "k_explore_init");
    }
    if (known) holds = init;
    return SLIMDP_OK;
}

uint32_t persistent_blocks(const slimdp_ctx* c, uint32_t per_cu, uint32_t nbatch)
{
    uint64_t p = (uint64_t)c->cus * per_cu / (nbatch ? nbatch : 1);
    if (p < 32) p = 32;
    if (p > c->T) p = c->T;
    return (uint32_t)p;
}

// How many workers a wave of the stand-alone draw takes in turn: as many as share the lanes' part of the random words, while
// the tiles alone make per_cu blocks for every compute unit.
uint32_t draw_group(const slimdp_ctx* c, uint32_t per_cu, uint32_t n_workers)
{
    uint32_t g = n_workers;
    while (g > 1 && (uint64_t)c->T * ((n_workers + g - 1) / g) < (uint64_t)c->cus * per_cu) g = (g + 1) / 2;
    return g;
}

// Whether a scoring pass of W workers keeps the explorers' update values, if it is left to the sizes.  A gather of 2 % of the
// parameters reads 44 % of the updates' lines, which costs little only while they come from the caches (256 MB), and one worker's
// too little for the scoring pass to earn it.  Whole iteration with and without, us: 138*10^6 parameters, 8 workers 2,140 / 2,320
// (5 %: 2,475 / 2,827), 16*10^6 and 8 339 / 355, 8*10^6 and 8 232 / 237, 32*10^6 and 2 316 / 322, but 8*10^6 and 4 185 / 184, 10^6 and
// 4 (scoring and pack alone) 31 / 24, 64*10^6 and 1 481 / 475.
bool expl_worth_keeping(uint64_t n, uint32_t W) { return W >= 2 && n * W * 4u >= (256ull << 20); }

// Room of the explorer capture, in words: the pipelined scoring kernel's, which serves flat models below 2^30 parameters and
// captures for 1, 2, 4, 8 or 16 workers.  Only where some number of workers that the context serves is worth keeping, or for all (forced).
size_t expl_capture_words(uint64_t n, uint64_t T, uint32_t max_workers, uint32_t n_seg, bool forced)
{
    if (n_seg != 1 || n >= (1ull << 30)) return 0;
    uint32_t most = 1;
    while (most < 16 && 2 * most <= max_workers) most *= 2;
    return forced || expl_worth_keeping(n, most) ? (size_t)T * SUBS * most * EXPL_SLOTS_MAX : 0;
}

// Slots for the explorer values of a sub-tile, from the share of the words in the sure zone: of its 256 blocks of four those
// with a sure parameter.  What does not fit is gathered: up to 0.23 % with the few (2.3 % of the words sure), up to 5.2 % with the
// larger number (5.1 %); above that nothing is kept.
uint32_t expl_slots(const SegInit& in)
{
    if (!in.has_gt) return 0;
    const double p = ((double)in.sure_m1 + 1.0) / 4294967296.0, full = 1.0 - std::pow(1.0 - p, 4.0);
    if (256.0 * full + 2.0 * std::sqrt(256.0 * full * (1.0 - full)) <= (double)EXPL_SLOTS_FEW) return EXPL_SLOTS_FEW;
    return 256.0 * full <= (double)EXPL_SLOTS_MAX ? EXPL_SLOTS_MAX : 0u;
}

// Whether the local models, gradients and updates (three arrays a worker) pass the caches by: they do not where the next pass
// finds a good part of them in the 256 MB of the last level.  One round of a worker's side in separate calls, non-temporal / not, us:
// 10^6 parameters, 4 workers (48 MB) 54 / 48; 3*10^6, 8 (288 MB) 212 / 191; 8*10^6, 4 (384 MB) 287 / 271; but 5*10^6, 8 (480 MB)
// 341 / 352 and 16*10^6, 8 1,090 / 1,239.
constexpr uint64_t STREAMS_HELD = 400000000u;
bool local_streams(const slimdp_ctx* c, uint32_t n_workers, uint64_t held = STREAMS_HELD) { return c->n * n_workers * 12u > held; }
// The two fused passes follow each other with little in between: where both leave their arrays in the caches, they evict each other's
// before the line above.  Step with extraction and pull with step, one round, both non-temporal / neither / the first only: 8*10^6
// parameters, 2 workers (192 MB) 131 / 129 / 126; 12*10^6, 2 (288 MB) 182 / 179 / 175; 7*10^6, 4 (336 MB) 200 / 198 / 189; 8*10^6, 4 (384 MB)
// 230 / 250 / 218; 16*10^6, 2 243 / 272 / 236.  One worker's are better off non-temporal at any size: 3*10^6 32.5 / 35.4 / 32.8, 5*10^6 50.7 /
// 53.7 / 51.6, 30*10^6 264 / 294 / 264.
// Where most tiles go by single floats (layered models whose tiles do not begin on multiples of four), both are better off
// non-temporal from 150 MB on: 57 segments, both / as above, 8*10^6, 2 124 / 131; 16*10^6, 2 236 / 254; 4*10^6, 4 120 / 128; 8*10^6, 4 227 / 242;
// 4*10^6, 8 223 / 230; but 6*10^6, 2 (144 MB) 93 / 89.
constexpr uint64_t FUSED_PACK_HELD = 300000000u, FUSED_FLOATS_HELD = 150000000u;
bool fused_streams(const slimdp_ctx* c, uint32_t n_workers, uint64_t held)
{
    return n_workers == 1 || local_streams(c, n_workers, c->tl.mostly_quads ? held : FUSED_FLOATS_HELD);
}

// How many workers a block of the passes over tiles takes in turn: all of them, so that what they share is read once, unless
// that leaves compute units without a block (one round of 10^6 parameters and 4 workers in 245 tiles: 50.7 us with all four,
// 48.0 with two a block, 51.2 with one; 2*10^6: 74.6 with four, 83.3 with one).
uint32_t workers_per_block(const slimdp_ctx* c, uint32_t n_workers)
{
    uint32_t per = n_workers;
    while (per > 1 && (uint64_t)c->T * ((n_workers + per - 1) / per) < (uint32_t)c->cus) per = (per + 1) / 2;
    return per;
}

template <class P> bool table_ok(P const* tab, uint32_t nw, bool allow_null_entries = false)
{
    if (!tab) return false;
    if (!allow_null_entries)
        for (uint32_t q = 0; q < nw; ++q)
            if (!tab[q]) return false;
    return true;
}

template <class Tab, class P> Tab make_tab(P const* tab, uint32_t nw)
{
    Tab t;
    for (int q = 0; q < MAXW; ++q) t.p[q] = nullptr;
    if (tab)
        for (uint32_t q = 0; q < nw; ++q) t.p[q] = (decltype(t.p[0]))tab[q];
    return t;
}

// Whether the device holds what the host's notes say it holds once everything enqueued has run (clear histograms, the
// segments' core sizes).  A call recorded into a graph runs later, any number of times or never: it must set what it needs
// by itself, and from then on a replay may have left other contents than the eager calls did.  Every call that goes by
// such a note, or leaves one, asks here before it looks at the note: one that did not ask would go unnoticed when recorded.
bool device_state_known(slimdp_ctx* c)
{
    if (c->stream && !c->recorded) {         // the default stream cannot be recorded
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(c->stream, &st) != hipSuccess || st != hipStreamCaptureStatusNone) c->recorded = true;
    }
    return !c->recorded;
}

// Whether an explorer request runs on the context's own stream although the options would have it on the side stream: an event
// and a wait across streams, there and back, leave the device idle for some 20 us, and beside other work the request's chain is
// slower.  Measured whole iterations, own stream / side stream, us:
//   to be drawn first, after a reselection: the lists are wanted at once.  By tiles times workers
//                       10^6 parameters, 4 workers (980) 46 / 91; 2*10^6, 8 (3,900) 106 / 128; 20*10^6, 1 (4,900) 204 / 216; 30*10^6, 1 (7,300)
//                       261 / 274; 8*10^6, 4 (7,800) 162 / 179; 8*10^6, 8 (15,600) 158 / 143; 138*10^6, 8 1,820 / 1,480
//   to be drawn first, for the same core as the request before: one iteration ahead, beside a pack and a merge that take the
//   longer the larger the model is even of one worker.  By tiles times (workers + 4), on two machines
//                       5*10^6, 1 (6,100) 43 / 56 to 65; 4*10^6, 4 (7,800) 64 / 65 to 74; 2*10^6, 16 (9,800) 92 / 93 to 103; 4*10^6, 8 (11,700) 90 / 77
//                       to 83; 8*10^6, 2 (11,700) 72 / 59 to 70; 12*10^6, 1 (14,600) 72 / 67; 20*10^6, 1 105 / 88; 30*10^6, 1 145 / 122; 8*10^6, 4 98 / 77;
//                       7*10^6 in 57 segments, 4 113 / 96; 30*10^6 in 57 segments, 1 199 / 185
//   drawn by the scoring pass of a reselecting iteration
//                       8*10^6, 8 (15,600) 207 / 226; 16*10^6, 8 (31,000) 330 / 335; 64*10^6, 4 (62,500) 658 / 644; 138*10^6, 8 2,150 / 2,115;
//                       but 138*10^6, 2 (67,500) 1,016 / 1,133: one or two workers' pack is too short to hide it
// The lines of "drawn" are also right for a draw that the side stream has made beside a pack and a merge since.  A request that
// follows its announcement at once stays behind the draw on the side stream, for the next calls to run beside both: on its own
// stream the context would wait for the draw, and pack and merge for the request's chain.  Cached core keys, request one iteration
// ahead, own / side: 8*10^6, 8 176 / 128; 10^7 in 57 segments, 4 186 / 135; 64*10^6, 2 385 / 300; 138*10^6, 1 561 / 464; 2 742 / 593.
// Announced before pack and merge, requested after them: 8*10^6, 8 137 / 150; 64*10^6, 2 327 / 341; 138*10^6, 1 505 / 520; 2 642 / 656.
bool stays_on_main(const slimdp_ctx* c, uint32_t n_workers, bool drawn)
{
    if (c->opt_explore_async == 2 || (c->side_pending && c->draw_fresh)) return false;
    const uint64_t work = (uint64_t)c->T * n_workers;
    if (drawn) return work <= 32000 || n_workers <= 2;
    return work <= 8500 && (c->asked_epoch != c->epoch || work + 4ull * c->T <= 10700);
}

// Whether an announced draw is left to its request, although it could begin on the side stream now.  Cached core keys, announced and
// requested one iteration ahead, draw with the request / ahead, us, by tiles times (workers + 4): 12*10^6, 1 worker (14,600) 66 / 82;
// 8*10^6, 4 (15,600) 77 / 90; 16*10^6, 2 (23,400) 90 / 90; 20*10^6, 1 (24,400) 88 / 90; 30*10^6, 1 (36,600) 122 / 117; in 57 segments 185 / 162.
bool draw_waits(const slimdp_ctx* c, uint32_t n_workers)
{
    const uint64_t work = (uint64_t)c->T * n_workers;
    return c->opt_explore_async != 2 && work <= 8500 && work + 4ull * c->T <= 24000;
}

// The context's stream waits for whatever the side stream still has in flight (an announced draw, asynchronous
// explorer requests) before it touches what that work reads or writes.
int wait_for_side(slimdp_ctx* c)
{
    int last = -1;
    for (int j = 0; j < slimdp_ctx::N_PENDING; ++j)
        if (c->pend[j].live && (last < 0 || c->pend[j].seq > c->pend[last].seq)) last = j;
    if (last >= 0) {                     // the side stream runs in order: the newest request's event covers all
        SLIMDP_HIP(c, hipStreamWaitEvent(c->stream, c->pend[last].ev, 0));
        for (int j = 0; j < slimdp_ctx::N_PENDING; ++j) c->pend[j].live = false;
        c->side_pending = false;         // a draw that preceded it on the same stream is done as well
    }
    if (c->side_pending) {
        SLIMDP_HIP(c, hipStreamWaitEvent(c->stream, c->ev_drawn, 0));
        c->side_pending = false;
    }
    return SLIMDP_OK;
}

// A call that reads explorer lists waits for the asynchronous requests that write any of them (address ranges
// compared, so views into the same allocation count), and with them for every older request; requests whose
// arrays it does not touch keep running beside it.
int wait_for_lists(slimdp_ctx* c, uint32_t nw, const uint32_t* const* expl_idx, const uint32_t* const* expl_off,
                   const uint64_t* m_w)
{
    int hit = -1;
    c->draw_fresh = false;
    for (int j = 0; j < slimdp_ctx::N_PENDING; ++j) {
        const slimdp_ctx::PendingExplore& p = c->pend[j];
        if (!p.live) continue;
        bool touches = false;
        for (uint32_t a = 0; a < nw && !touches; ++a)
            for (uint32_t b = 0; b < p.nw && !touches; ++b) {
                const uintptr_t i0 = reinterpret_cast<uintptr_t>(expl_idx ? expl_idx[a] : nullptr);
                const uintptr_t o0 = reinterpret_cast<uintptr_t>(expl_off ? expl_off[a] : nullptr);
                // exactly: an array that begins where another ends is no part of it
                if (i0 && i0 < p.idx[b] + p.idx_bytes && p.idx[b] < i0 + std::max<uint64_t>(m_w ? m_w[a] * 4 : 0, 4)) touches = true;
                if (o0 && o0 < p.off[b] + p.off_bytes && p.off[b] < o0 + p.off_bytes) touches = true;
            }
        if (touches && (hit < 0 || p.seq > c->pend[hit].seq)) hit = j;
    }
    if (hit < 0) return SLIMDP_OK;
    SLIMDP_HIP(c, hipStreamWaitEvent(c->stream, c->pend[hit].ev, 0));
    const uint64_t upto = c->pend[hit].seq;
    for (int j = 0; j < slimdp_ctx::N_PENDING; ++j)
        if (c->pend[j].live && c->pend[j].seq <= upto) c->pend[j].live = false;
    return SLIMDP_OK;
}

int check_epoch(slimdp_ctx* c, uint64_t core_epoch)
{
    if (c->epoch == 0 || core_epoch != c->epoch)
        return fail(c, SLIMDP_ERR_STALE_CORE, "core_epoch %llu is not the context's current core epoch %llu",
                    (unsigned long long)core_epoch, (unsigned long long)c->epoch);
    return SLIMDP_OK;
}

// Explorer requests whose zones are not narrow compact their candidate keys over the whole index range: that buffer
// (4 bytes per parameter and worker) is allocated by the first such request and kept.
int ensure_wide_keys(slimdp_ctx* c)
{
    if (c->e_cand_keys) return SLIMDP_OK;
    const size_t bytes = (size_t)c->maxW * c->keys_stride * sizeof(uint32_t);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&c->e_cand_keys), bytes);
    if (e != hipSuccess) {
        c->e_cand_keys = nullptr;
        return fail(c, SLIMDP_ERR_WORKSPACE, "explorer with wide zones: hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
    }
    return SLIMDP_OK;
}

// The explorer capture that option "explore_keep" = 2 asks for beside "speculative_pack", where the sizes alone ask for none.
int ensure_expl_capture(slimdp_ctx* c)
{
    if (!c->spec.mem || c->spec.evals) return SLIMDP_OK;
    const size_t bytes = expl_capture_words(c->n, c->T, c->maxW, c->n_seg, true) * sizeof(float);
    if (bytes == 0) return SLIMDP_OK;
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&c->spec.evals_mem), bytes);
    if (e != hipSuccess) {
        c->spec.evals_mem = nullptr;
        return fail(c, SLIMDP_ERR_WORKSPACE, "slimdp_set_option(explore_keep): hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(e));
    }
    c->spec.evals = reinterpret_cast<float*>(c->spec.evals_mem);
    return SLIMDP_OK;
}

// Probability that one sub-tile holds more than PAIR_CAP candidates of one draw when lambda are expected (the draw
// marks each of its up to 1024 words independently: Poisson tail, summed directly so that tiny values keep their digits).
double pair_overflow_prob(double lambda)
{
    if (lambda <= 0.0) return 0.0;
    const int j0 = (int)PAIR_CAP + 1;
    double term = std::exp(-lambda + j0 * std::log(lambda) - std::lgamma((double)j0 + 1.0)), sum = 0.0;
    for (int j = j0; j < j0 + 4096; ++j) {
        sum += term;
        term *= lambda / (double)(j + 1);
        if (term < 1e-18 * sum && (double)j > lambda) break;
    }
    return sum < 1.0 ? sum : 1.0;
}

// Per-segment start of the explorer's radix descent.  The m-th smallest Philox word of the
// avail = n_s - k_s parameters outside the core lies, with overwhelming probability, between
// the words that m - 6 sqrt(m) - 32 and m + 6 sqrt(m) + 32 of them are expected to stay below:
// words up to the first are taken without ranking (sure zone), only the words between the two
// become candidates.  The exact rerun with every word a candidate catches a miss on either
// side.  Returns an error code for impossible requests; *narrow is set when every segment
// got a narrow candidate zone; *short_list when no sub-tile is likely to see more candidates
// than its pair slot holds (small segments have relatively wide zones: twelve standard
// deviations of a small m are a large share of it).
int explorer_init(slimdp_ctx* ctx, const char* who, const uint64_t* k_seg, const uint64_t* m_seg, uint32_t n_workers,
                  std::vector<SegInit>& init, uint64_t* M_out, bool* narrow, bool* short_list)
{
    uint64_t M = 0;
    bool all_narrow = true;
    double overflows = 0.0;        // expected number of sub-tiles of the request with more candidates than a pair slot holds
    init.resize(ctx->n_seg);
    for (uint32_t s = 0; s < ctx->n_seg; ++s) {
        const uint64_t ns = ctx->seg_off[s + 1] - ctx->seg_off[s];
        if (k_seg[s] > ns || m_seg[s] > ns - k_seg[s])
            return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "%s: segment %u: m=%llu exceeds the %llu parameters outside the core",
                        who, s, (unsigned long long)m_seg[s], (unsigned long long)(k_seg[s] > ns ? 0 : ns - k_seg[s]));
        const uint64_t m = m_seg[s];
        SegInit in{(uint32_t)m, (uint32_t)M, 0u, 0u, 0u, 0u};
        M += m;
        if (m > 0) {
            const double avail = (double)(ns - k_seg[s]);
            const double slack = 6.0 * std::sqrt((double)m) + 32.0;
            double hi = ((double)m + slack) / avail, lo = ((double)m - slack) / avail;
            if (ctx->opt_force_fallback == 1) { hi = 0.25 * (double)m / avail; lo = 0.5 * hi; }     // too few candidates
            if (ctx->opt_force_fallback == 2) { hi = 2.0 * (double)m / avail; lo = 0.75 * hi; }     // sure zone too large
            uint64_t width = 1ull << 32;                     // number of distinct candidate words
            overflows += pair_overflow_prob((hi - (lo > 0.0 ? lo : 0.0)) * (double)SUB) * ((double)ns / SUB + 2.0) * n_workers;
            if (hi >= 0.95) all_narrow = false;
            uint64_t B1 = hi < 1.0 ? (uint64_t)std::ceil(hi * 4294967296.0) : 1ull << 32;
            if (B1 < 1) B1 = 1;
            if (B1 > (1ull << 32)) B1 = 1ull << 32;
            in.bound_m1 = (uint32_t)(B1 - 1);
            width = B1;
            const uint64_t B0 = lo > 0.0 ? (uint64_t)std::floor(lo * 4294967296.0) : 0;
            if (B0 >= 1 && B0 < B1) {                        // words 0 .. B0-1 are sure, B0 .. B1-1 candidates
                in.sure_m1 = (uint32_t)(B0 - 1);
                in.has_gt = 1;
                width = B1 - B0;
            }
            while (((width - 1) >> in.bits) != 0) ++in.bits;
        }
        init[s] = in;
    }
    *M_out = M;
    *narrow = all_narrow;
    // an overflowing slot costs the exact rerun (a thousand times the whole request): taken only if that is unlikely
    *short_list = all_narrow && !ctx->opt_per_tile_tail && overflows <= 1e-5;
    return SLIMDP_OK;
}

// The same, kept while the sizes stay what they were (the announcement, the scoring pass and the request of every iteration
// ask for it: 0.2 us a segment each).
int explorer_plan(slimdp_ctx* ctx, const char* who, const uint64_t* k_seg, const uint64_t* m_seg, uint32_t n_workers)
{
    slimdp_ctx::Plan& p = ctx->plan;
    const uint32_t S = ctx->n_seg;
    if (p.valid && p.n_workers == n_workers && p.force == ctx->opt_force_fallback && p.tail == ctx->opt_per_tile_tail &&
        std::equal(k_seg, k_seg + S, p.k_seg.begin()) && std::equal(m_seg, m_seg + S, p.m_seg.begin()))
        return SLIMDP_OK;
    p.valid = false;
    const int rc = explorer_init(ctx, who, k_seg, m_seg, n_workers, p.init, &p.M, &p.narrow, &p.pairs);
    if (rc) return rc;
    p.k_seg.assign(k_seg, k_seg + S); p.m_seg.assign(m_seg, m_seg + S);
    p.n_workers = n_workers; p.force = ctx->opt_force_fallback; p.tail = ctx->opt_per_tile_tail;
    p.valid = true;
    return SLIMDP_OK;
}

}  // namespace

extern "C" {

uint64_t slimdp_num_tiles(uint64_t n, uint32_t n_seg, const uint64_t* seg_off)
{
    if (!valid_shape(n, n_seg, seg_off)) return 0;
    return count_tiles(n, n_seg, seg_off);
}

uint64_t slimdp_workspace_bytes(uint64_t n, uint32_t max_workers, uint32_t n_seg, const uint64_t* seg_off)
{
    if (!valid_shape(n, n_seg, seg_off) || max_workers == 0 || max_workers > SLIMDP_MAX_WORKERS) return 0;
    slimdp_ctx tmp;
    tmp.n = n; tmp.maxW = max_workers; tmp.n_seg = n_seg;
    tmp.T = (uint32_t)count_tiles(n, n_seg, seg_off);
    tmp.keys_stride = align_up(n, TILE) + TILE;
    tmp.pair_stride = (uint64_t)tmp.T * SUBS * PAIR_SLOT;
    tmp.list_first = list_starts(n_seg, seg_off);
    Carver cv(nullptr);
    carve(&tmp, cv);
    return align_up(cv.pos, 256);
}

uint64_t slimdp_capture_bytes(uint64_t n, uint32_t max_workers, uint32_t n_seg, const uint64_t* seg_off)
{
    if (!valid_shape(n, n_seg, seg_off) || max_workers == 0 || max_workers > SLIMDP_MAX_WORKERS) return 0;
    const uint64_t T = count_tiles(n, n_seg, seg_off);
    Carver cv(nullptr);
    cv.take<uint32_t>(n_seg); cv.take<uint32_t>(n_seg); cv.take<uint32_t>(n_seg);
    cv.take<uint2>((size_t)T * TILE_WORDS);
    cv.take<float>((size_t)max_workers * T * SUBS * SPEC_CAP);
    cv.take<float>(expl_capture_words(n, T, max_workers, n_seg, false));
    cv.take<uint32_t>((size_t)T * SAMPLE_PER);
    return align_up(cv.pos, 256);
}

const char* slimdp_last_error(const slimdp_ctx* ctx) { return ctx ? ctx->err.c_str() : g_create_error.c_str(); }

int slimdp_create(slimdp_ctx** out, uint64_t n, uint32_t max_workers, uint32_t n_seg, const uint64_t* seg_off,
                  uint64_t seed, void* hip_stream)
{
    if (!out) return fail(nullptr, SLIMDP_ERR_INVALID_ARG, "slimdp_create: out is NULL");
    *out = nullptr;
    if (n == 0 || n > SLIMDP_MAX_N) return fail(nullptr, SLIMDP_ERR_INVALID_ARG, "slimdp_create: n must be in [1, 2^31]");
    if (max_workers == 0 || max_workers > SLIMDP_MAX_WORKERS)
        return fail(nullptr, SLIMDP_ERR_INVALID_ARG, "slimdp_create: max_workers must be in [1, %u]", SLIMDP_MAX_WORKERS);
    if (!valid_shape(n, n_seg, seg_off))
        return fail(nullptr, SLIMDP_ERR_INVALID_ARG,
                    "slimdp_create: seg_off must be %u+1 strictly increasing offsets from 0 to n", n_seg);
    slimdp_ctx* c = new (std::nothrow) slimdp_ctx;
    if (!c) return fail(nullptr, SLIMDP_ERR_WORKSPACE, "slimdp_create: out of host memory");
    c->n = n; c->maxW = max_workers; c->n_seg = n_seg; c->seed = seed;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->seg_off.assign(seg_off, seg_off + n_seg + 1);
    c->tl = make_tiling(n, n_seg, seg_off);
    c->T = (uint32_t)c->tl.tile_seg.size();
    c->keys_stride = align_up(n, TILE) + TILE;
    c->pair_stride = (uint64_t)c->T * SUBS * PAIR_SLOT;
    c->list_first = list_starts(n_seg, seg_off);
    hipError_t e = hipGetDevice(&c->device);
    if (e != hipSuccess) { int rc = hip_fail(nullptr, e, "hipGetDevice (no usable GPU?)"); delete c; return rc; }
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, c->device);
    if (e != hipSuccess) { int rc = hip_fail(nullptr, e, "hipGetDeviceProperties"); delete c; return rc; }
    c->cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    Carver sizing(nullptr);
    carve(c, sizing);
    c->ws_bytes = align_up(sizing.pos, 256);
    e = hipMalloc(reinterpret_cast<void**>(&c->ws), c->ws_bytes);
    if (e != hipSuccess) {
        int rc = fail(nullptr, SLIMDP_ERR_WORKSPACE, "slimdp_create: hipMalloc(%zu bytes): %s", c->ws_bytes, hipGetErrorString(e));
        delete c;
        return rc;
    }
    Carver cv(c->ws);
    carve(c, cv);
    // A clear histogram; the tables, an empty prediction and the cleared flags, in one copy.  Both run on the default
    // stream, and the context's stream need not wait for that one (a non-blocking stream does not): the host waits here.
    e = hipMemset(c->c_hist, 0, (size_t)n_seg * H_STRIDE * 4);
    if (e == hipSuccess) {
        const size_t words = (size_t)(c->d_flags + 64 - c->d_tile_start);
        std::vector<uint32_t> up(words, 0u);
        auto at = [&](const uint32_t* d) { return up.begin() + (d - c->d_tile_start); };
        std::copy(c->tl.tile_start.begin(), c->tl.tile_start.end(), at(c->d_tile_start));
        std::copy(c->tl.tile_seg.begin(), c->tl.tile_seg.end(), at(c->d_tile_seg));
        std::copy(c->tl.seg_first_tile.begin(), c->tl.seg_first_tile.end(), at(c->d_seg_first_tile));
        std::copy(c->list_first.begin(), c->list_first.end(), at(c->d_list_first));
        std::fill_n(at(c->c_pred), n_seg, NONE);                              // no prediction yet
        e = hipMemcpy(c->d_tile_start, up.data(), words * 4, hipMemcpyHostToDevice);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking);      // default priority
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->ev_consumed, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->ev_drawn, hipEventDisableTiming);
    for (int j = 0; j < slimdp_ctx::N_PENDING && e == hipSuccess; ++j)
        e = hipEventCreateWithFlags(&c->pend[j].ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        int rc = hip_fail(nullptr, e, "slimdp_create: table upload, side stream");
        if (c->ev_consumed) (void)hipEventDestroy(c->ev_consumed);
        if (c->ev_drawn) (void)hipEventDestroy(c->ev_drawn);
        for (int j = 0; j < slimdp_ctx::N_PENDING; ++j)
            if (c->pend[j].ev) (void)hipEventDestroy(c->pend[j].ev);
        if (c->side) (void)hipStreamDestroy(c->side);
        (void)hipFree(c->ws);
        delete c;
        return rc;
    }
    *out = c;
    return SLIMDP_OK;
}

int slimdp_destroy(slimdp_ctx* ctx)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    (void)hipStreamSynchronize(ctx->side);
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipEventDestroy(ctx->ev_consumed);
    (void)hipEventDestroy(ctx->ev_drawn);
    for (int j = 0; j < slimdp_ctx::N_PENDING; ++j) (void)hipEventDestroy(ctx->pend[j].ev);
    (void)hipStreamDestroy(ctx->side);
    hipError_t e = hipFree(ctx->ws);
    if (ctx->spec.mem) (void)hipFree(ctx->spec.mem);
    if (ctx->spec.evals_mem) (void)hipFree(ctx->spec.evals_mem);
    if (ctx->e_cand_keys) (void)hipFree(ctx->e_cand_keys);
    delete ctx;
    return e == hipSuccess ? SLIMDP_OK : SLIMDP_ERR_HIP;
}

int slimdp_tile_starts(const slimdp_ctx* ctx, uint32_t* tile_start)
{
    if (!ctx || !tile_start) return SLIMDP_ERR_INVALID_ARG;
    memcpy(tile_start, ctx->tl.tile_start.data(), (ctx->T + 1) * sizeof(uint32_t));
    return SLIMDP_OK;
}

int slimdp_set_option(slimdp_ctx* ctx, const char* name, int64_t value)
{
    if (!ctx || !name) return SLIMDP_ERR_INVALID_ARG;
    if (strcmp(name, "explore_force_fallback") == 0) { ctx->opt_force_fallback = value; return SLIMDP_OK; }
    if (strcmp(name, "explore_per_tile_tail") == 0) { ctx->opt_per_tile_tail = value; return SLIMDP_OK; }
    if (strcmp(name, "strided_tiles") == 0 && (value == 0 || value == 1)) { ctx->opt_strided = value; return SLIMDP_OK; }
    if (strcmp(name, "side_blocks") == 0 && value >= 1 && value <= 8) { ctx->opt_side_blocks = value; return SLIMDP_OK; }
    if (strcmp(name, "explore_async") == 0 && value >= 0 && value <= 2) { ctx->opt_explore_async = value; return SLIMDP_OK; }
    if (strcmp(name, "explore_hint_mode") == 0 && (value == 0 || value == 1)) { ctx->opt_hint_mode = value; return SLIMDP_OK; }
    if (strcmp(name, "core_predict") == 0 && value >= 0 && value <= 2) { ctx->opt_core_predict = value; return SLIMDP_OK; }
    if (strcmp(name, "pack_core_blocks") == 0 && value >= 0 && value <= 64) { ctx->opt_pack_core_blocks = value; return SLIMDP_OK; }
    if (strcmp(name, "build_blocks") == 0 && value >= 1 && value <= 64) { ctx->opt_build_blocks = value; return SLIMDP_OK; }
    if (strcmp(name, "pack_nbuf") == 0 && (value == 1 || value == 2)) { ctx->opt_pack_nbuf = value; return SLIMDP_OK; }
    if (strcmp(name, "pack_kernel") == 0 && (value == 0 || value == 1)) { ctx->opt_pack_kernel = value; return SLIMDP_OK; }
    if (strcmp(name, "pull_kernel") == 0 && (value == 0 || value == 1)) { ctx->opt_pull_kernel = value; return SLIMDP_OK; }
    if (strcmp(name, "expected_core") == 0 && value >= -1 && (value < 0 || (uint64_t)value <= ctx->n)) { ctx->opt_expected_core = value; return SLIMDP_OK; }
    if (strcmp(name, "explore_keep") == 0 && value >= 0 && value <= 2) {
        const int rc = value == 2 ? ensure_expl_capture(ctx) : SLIMDP_OK;
        if (!rc) ctx->opt_explore_keep = value;
        return rc;
    }
    if (strcmp(name, "score_pipeline") == 0 && (value == 0 || value == 1)) { ctx->opt_score_pipeline = value; return SLIMDP_OK; }
    if (strcmp(name, "capture_estimate_bias") == 0) { ctx->opt_estimate_bias = value; return SLIMDP_OK; }
    if (strcmp(name, "speculative_pack") == 0) {
        ctx->spec.captured = false;
        if (value && !ctx->spec.mem) {
            const size_t S = ctx->n_seg;
            Carver sizing(nullptr);
            auto carve_spec = [&](Carver& cv) {
                ctx->spec.lo[0] = cv.take<uint32_t>(S);
                ctx->spec.lo[1] = cv.take<uint32_t>(S);
                ctx->spec.fail = cv.take<uint32_t>(S);
                ctx->spec.bits = cv.take<uint2>((size_t)ctx->T * TILE_WORDS);
                ctx->spec.vals = cv.take<float>((size_t)ctx->maxW * ctx->T * SUBS * SPEC_CAP);
                const size_t ew = expl_capture_words(ctx->n, ctx->T, ctx->maxW, ctx->n_seg, false);
                if (ew) ctx->spec.evals = cv.take<float>(ew);
                ctx->spec.sample = cv.take<uint32_t>((size_t)ctx->T * SAMPLE_PER);
            };
            carve_spec(sizing);
            hipError_t e = hipMalloc(reinterpret_cast<void**>(&ctx->spec.mem), align_up(sizing.pos, 256));
            if (e != hipSuccess) {
                ctx->spec.mem = nullptr;
                return fail(ctx, SLIMDP_ERR_WORKSPACE, "slimdp_set_option(speculative_pack): hipMalloc(%zu bytes): %s",
                            align_up(sizing.pos, 256), hipGetErrorString(e));
            }
            Carver cv(ctx->spec.mem);
            carve_spec(cv);
            // nothing captured, nothing trusted until a selection has set a bound
            int rc = fill(ctx, ctx->spec.lo[0], S, NONE);
            if (!rc) rc = fill(ctx, ctx->spec.lo[1], S, NONE);
            if (!rc) rc = fill(ctx, ctx->spec.fail, S, 1u);
            if (rc) return rc;
            ctx->spec.cur = 0;
            ctx->spec.next_written = false;
            ctx->spec.bound_valid = false;
        }
        if (value && ctx->opt_explore_keep == 2) { const int rc = ensure_expl_capture(ctx); if (rc) return rc; }
        ctx->spec.on = value != 0;
        return SLIMDP_OK;
    }
    return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_set_option: unknown option '%s'", name);
}

int slimdp_synchronize(slimdp_ctx* ctx)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    SLIMDP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    SLIMDP_HIP(ctx, hipStreamSynchronize(ctx->side));
    for (int j = 0; j < slimdp_ctx::N_PENDING; ++j) ctx->pend[j].live = false;
    ctx->side_pending = false;
    uint32_t flags[2] = {0, 0};
    SLIMDP_HIP(ctx, hipMemcpy(flags, ctx->d_flags, sizeof flags, hipMemcpyDeviceToHost));
    if (flags[1]) {
        SLIMDP_HIP(ctx, hipMemset(ctx->d_flags + 1, 0, 4));
        return fail(ctx, SLIMDP_ERR_DEVICE_STATUS, "device status 0x%x:%s%s", flags[1],
                    (flags[1] & 1u) ? " an emitted index list does not have the requested length;" : "",
                    (flags[1] & 2u) ? " a segment holds fewer eligible parameters than requested;" : "");
    }
    return SLIMDP_OK;
}

// ------------------------------------------------------------------------------------------
static int score_impl(slimdp_ctx* ctx, const float* w, const float* const* g, uint32_t W, float c, float* score, float* w_new,
                      float lr)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!w || !score) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_score: NULL array");
    if (W == 0 || W > ctx->maxW) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_score: W=%u outside [1, %u]", W, ctx->maxW);
    if (!table_ok(g, W)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_score: NULL update pointer");
    if (!(c >= 0.0f) || std::isinf(c)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_score: c must be finite and >= 0");
    ctx->hist_pending = false;
    ctx->cls_by_score = false;
    int rc = SLIMDP_OK;
    const bool known = device_state_known(ctx);
    if (!known || !ctx->hist_clean) { rc = fill(ctx, ctx->c_hist, (uint64_t)ctx->n_seg * H_STRIDE, 0u); if (rc) return rc; }
    ctx->hist_clean = false;
    PtrTab gt = make_tab<PtrTab>(g, W);
    int vec_ok = aligned16(w) && aligned16(score);
    for (uint32_t q = 0; q < W; ++q) vec_ok = vec_ok && aligned16(g[q]);
    // an announced explorer draw rides along if every segment has a narrow candidate bound
    PreArgs pre{};
    bool presample = false, pairs = false;
    uint32_t slots = 0;
    ctx->spec.expl_slots = 0;
    if (ctx->opt_hint_mode == 0) ctx->pre.valid = false;      // a draw made on the side stream stays valid
    if (ctx->hint.valid && ctx->opt_hint_mode == 0) {
        const slimdp_ctx::Plan& plan = ctx->plan;
        if (explorer_plan(ctx, "slimdp_score(hint)", ctx->hint.k_seg.data(), ctx->hint.m_seg.data(), ctx->hint.n_workers) == SLIMDP_OK &&
            plan.narrow && plan.M > 0 &&
            // tiles inside random blocks: the first request, not a scoring pass, allocates the wide buffer (until then
            // such an announcement goes unused and the request draws for itself)
            (plan.pairs || ctx->e_cand_keys || ctx->tl.quad_aligned)) {
            pairs = plan.pairs;
            rc = wait_for_side(ctx);         // the draw's buffers may still be read by work on the side stream
            if (rc) return rc;
            rc = init_states(ctx, ctx->e_state, ctx->e_state_holds, plan.init, known, false, 0, ctx->stream);
            if (rc) return rc;
            pre.nw = ctx->hint.n_workers; pre.worker0 = ctx->hint.worker0; pre.n_seg = ctx->n_seg;
            pre.states = ctx->e_state; pre.sure_bits = ctx->e_sure_bits; pre.cand_bits = ctx->e_cand_bits;
            if (!pairs) { rc = ensure_wide_keys(ctx); if (rc) return rc; }
            pre.cand_keys = pairs ? ctx->e_pair_keys : ctx->e_cand_keys; pre.cnt_cand = ctx->e_cnt_cand;
            pre.keys_stride = pairs ? ctx->pair_stride : ctx->keys_stride;
            pre.pk = PhiloxKey{(uint32_t)ctx->seed, (uint32_t)(ctx->seed >> 32), (uint32_t)ctx->hint.iteration,
                               (uint32_t)(ctx->hint.iteration >> 32)};
            slots = pairs && ctx->n_seg == 1 ? expl_slots(plan.init[0]) : 0;
            presample = true;
        }
    }
    // speculative packing: keep the update values of the parameters at or above the previous threshold
    SpecArgs sa{};
    // (not after a dense update: the pack that follows it belongs to the next iteration's updates)
    const bool capture = ctx->spec.on && !w_new && (W == 1 || W == 2 || W == 4 || W == 8 || W == 16);
    ctx->spec.captured = false;
    if (capture) {
        if (ctx->spec.next_written) { ctx->spec.cur ^= 1; ctx->spec.next_written = false; ctx->spec.bound_valid = true; }
        sa.lo = ctx->spec.lo[ctx->spec.cur]; sa.bits = ctx->spec.bits; sa.vals = ctx->spec.vals;
        // No selection has set a bound yet (first iteration of a context): estimate the coming threshold from a sample of
        // the very significances this pass computes, if the size of the coming core is known (announced draw, option, or
        // the previous selection).  Flat model, whole aligned tiles.
        const uint32_t T_full = (uint32_t)(ctx->n / TILE);
        int64_t expect = ctx->opt_expected_core;
        if (expect < 0 && ctx->hint.valid && ctx->n_seg == 1) expect = (int64_t)ctx->hint.k_seg[0];
        if (expect < 0 && ctx->have_last_K) expect = (int64_t)ctx->last_K;
        if (!ctx->spec.bound_valid && ctx->n_seg == 1 && vec_ok && T_full >= 64 && expect >= 0) {
            const uint32_t N = T_full * SAMPLE_PER;
            // rank of the threshold inside the sample, rounded up
            const uint64_t need = ((uint64_t)expect * N + ctx->n - 1) / ctx->n;
            hipLaunchKernelGGL(k_sample_keys, dim3((N + 255) / 256), dim3(256), 0, ctx->stream, w, gt, (int)W, c, T_full,
                               ctx->spec.sample);
            SLIMDP_LAUNCHED(ctx, "k_sample_keys");
            hipLaunchKernelGGL(k_sample_bound, dim3(1), dim3(1024), 0, ctx->stream, ctx->spec.sample, N, (uint32_t)need,
                               (long long)ctx->opt_estimate_bias, ctx->spec.lo[ctx->spec.cur], ctx->c_pred);
            SLIMDP_LAUNCHED(ctx, "k_sample_bound");
        }
    }
    // flat model, aligned arrays, a number of workers that the pipelined kernel is instantiated for (see there)
    if (ctx->n_seg == 1 && vec_ok && ctx->opt_strided && ctx->opt_score_pipeline && ctx->n < (1ull << 30) &&
        (W <= 8 || W == 16)) {
        const dim3 fgrid(persistent_blocks(ctx, SCOREF_MINB, 1)), fblock(BLOCK);
        // The explorers' values too, where that pays (expl_worth_keeping).  Fewer workers announced than scored: the draw for
        // its own sake.  A context with recorded calls: a replay may draw again between a scoring pass and its pack, unknown to
        // the host.
        if (!capture || !ctx->spec.evals || pre.nw < W || !known || ctx->opt_explore_keep == 0 ||
            (ctx->opt_explore_keep == 1 && !expl_worth_keeping(ctx->n, W)))
            slots = 0;
        pre.vals = ctx->spec.evals; pre.slots = slots;
        ctx->spec.expl_slots = slots;
        const ClsArgs cls{ctx->c_pred, ctx->c_used, (int)ctx->opt_core_predict, ctx->c_gt_bits, ctx->c_cand_bits, ctx->c_cand_keys, ctx->c_cnt_gt, ctx->c_cnt_cand};
#define LAUNCH_FLAT_Q(WT, PRE, SPEC, DENSE)                                                                           \
    hipLaunchKernelGGL((k_score_flat<WT, PRE, SPEC, DENSE>), fgrid, fblock, 0, ctx->stream, w, gt, c, score, ctx->n,  \
                       ctx->c_hist, pre, sa, cls, w_new, lr)
#define LAUNCH_FLAT_S(WT, SPEC, DENSE)                                                                                \
    do {                                                                                                              \
        if (presample && pairs && (SPEC) && slots) LAUNCH_FLAT_Q(WT, ((SPEC) ? 3 : 2), SPEC, DENSE);                  \
        else if (presample && pairs) LAUNCH_FLAT_Q(WT, 2, SPEC, DENSE);                                               \
        else if (presample) LAUNCH_FLAT_Q(WT, 1, SPEC, DENSE);                                                        \
        else LAUNCH_FLAT_Q(WT, 0, SPEC, DENSE);                                                                       \
    } while (0)
#define LAUNCH_FLAT(WT)                                                                                               \
    do {                                                                                                              \
        constexpr int CAP = (WT) == 1 || (WT) == 2 || (WT) == 4 || (WT) == 8 || (WT) == 16;                           \
        if (w_new) LAUNCH_FLAT_S(WT, 0, 1);                                                                           \
        else if (capture) LAUNCH_FLAT_S(WT, CAP, 0);                                                                  \
        else LAUNCH_FLAT_S(WT, 0, 0);                                                                                 \
    } while (0)
        switch (W) {
            case 1: LAUNCH_FLAT(1); break;
            case 2: LAUNCH_FLAT(2); break;
            case 3: LAUNCH_FLAT(3); break;
            case 4: LAUNCH_FLAT(4); break;
            case 5: LAUNCH_FLAT(5); break;
            case 6: LAUNCH_FLAT(6); break;
            case 7: LAUNCH_FLAT(7); break;
            case 8: LAUNCH_FLAT(8); break;
            default: LAUNCH_FLAT(16); break;
        }
#undef LAUNCH_FLAT
#undef LAUNCH_FLAT_S
#undef LAUNCH_FLAT_Q
        SLIMDP_LAUNCHED(ctx, "k_score_flat");
        ctx->cls_by_score = true;
        if (presample) { ctx->pre = ctx->hint; ctx->pre.pairs = pairs; }
        if (capture) {
            ctx->spec.captured = true; ctx->spec.score = score; ctx->spec.W = W; ctx->spec.core_epoch = 0;
            for (uint32_t q = 0; q < W; ++q) ctx->spec.g[q] = g[q];
        }
        ctx->hint.valid = false;
        ctx->hist_pending = true;
        ctx->hist_score = score;
        return SLIMDP_OK;
    }
    const uint32_t P = persistent_blocks(ctx, SCORE_MINB, 1);
    const dim3 grid(P), block(BLOCK);
    // flat model, up to 8 workers: every P-th tile per block (measured: 8 workers 1.38 -> 1.34 ms; 16 workers slower)
    const bool strided = ctx->n_seg == 1 && ctx->opt_strided && W <= 8;
#define LAUNCH_SCORE_Q(WT, PRE, SPEC, DENSE, STRIDED)                                                                 \
    hipLaunchKernelGGL((k_score<WT, PRE, SPEC, DENSE, STRIDED>), grid, block, 0, ctx->stream, w, gt, (int)W, c, score, \
                       ctx->d_tile_start, ctx->d_tile_seg, ctx->T, ctx->c_hist, pre, sa, w_new, lr)
#define LAUNCH_SCORE_P(WT, PRE, SPEC, DENSE)                                                                          \
    do {                                                                                                              \
        if constexpr ((WT) >= 1 && (WT) <= 8) {                                                                       \
            if (strided) LAUNCH_SCORE_Q(WT, PRE, SPEC, DENSE, 1);                                                     \
            else LAUNCH_SCORE_Q(WT, PRE, SPEC, DENSE, 0);                                                             \
        } else LAUNCH_SCORE_Q(WT, PRE, SPEC, DENSE, 0);                                                               \
    } while (0)
#define LAUNCH_SCORE_S(WT, SPEC, DENSE)                                                                               \
    do {                                                                                                              \
        if (presample && pairs) LAUNCH_SCORE_P(WT, 2, SPEC, DENSE);                                                   \
        else if (presample) LAUNCH_SCORE_P(WT, 1, SPEC, DENSE);                                                       \
        else LAUNCH_SCORE_P(WT, 0, SPEC, DENSE);                                                                      \
    } while (0)
#define LAUNCH_SCORE(WT)                                                                                              \
    do {                                                                                                              \
        if (w_new) LAUNCH_SCORE_S(WT, 0, 1);                                                                          \
        else if (capture) LAUNCH_SCORE_S(WT, 1, 0);                                                                   \
        else LAUNCH_SCORE_S(WT, 0, 0);                                                                                \
    } while (0)
    switch (W) {
        case 1: LAUNCH_SCORE(1); break;
        case 2: LAUNCH_SCORE(2); break;
        case 4: LAUNCH_SCORE(4); break;
        case 8: LAUNCH_SCORE(8); break;
        case 16: LAUNCH_SCORE(16); break;
        default:
            if (w_new) LAUNCH_SCORE_S(0, 0, 1);
            else LAUNCH_SCORE_S(0, 0, 0);
            break;
    }
#undef LAUNCH_SCORE_P
#undef LAUNCH_SCORE_Q
#undef LAUNCH_SCORE_S
#undef LAUNCH_SCORE
    SLIMDP_LAUNCHED(ctx, "k_score");
    if (presample) { ctx->pre = ctx->hint; ctx->pre.pairs = pairs; }
    if (capture) {
        ctx->spec.captured = true; ctx->spec.score = score; ctx->spec.W = W; ctx->spec.core_epoch = 0;
        for (uint32_t q = 0; q < W; ++q) ctx->spec.g[q] = g[q];
    }
    ctx->hint.valid = false;
    ctx->hist_pending = true;
    ctx->hist_score = score;
    return SLIMDP_OK;
}

int slimdp_score(slimdp_ctx* ctx, const float* w, const float* const* g, uint32_t W, float c, float* score)
{
    return score_impl(ctx, w, g, W, c, score, nullptr, 0.0f);
}

int slimdp_dense_update_score(slimdp_ctx* ctx, float* w, const float* const* g, uint32_t W, float lr, float c, float* score)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!std::isfinite(lr)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_dense_update_score: lr must be finite");
    if (w && score && static_cast<const void*>(w) == static_cast<const void*>(score))
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_dense_update_score: score aliases w");
    return score_impl(ctx, w, g, W, c, score, w, lr);
}

// The selection itself, for a context whose device pointers may also lie in the static scratch array.
static int select_core_impl(slimdp_ctx* ctx, const float* score, const uint64_t* k_seg, uint32_t flags, uint32_t* core_idx,
                            uint32_t* core_bits, uint32_t* core_off, uint64_t* core_epoch)
{
    if (!score || !k_seg || !core_bits || !core_off || !core_epoch)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_select_core: NULL argument");
    uint64_t K = 0;
    for (uint32_t s = 0; s < ctx->n_seg; ++s) {
        const uint64_t ns = ctx->seg_off[s + 1] - ctx->seg_off[s];
        if (k_seg[s] > ns)
            return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_select_core: k_seg[%u]=%llu exceeds the segment size %llu", s,
                        (unsigned long long)k_seg[s], (unsigned long long)ns);
        K += k_seg[s];
    }
    if (K > 0 && !core_idx) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_select_core: core_idx is NULL");
    const bool reuse = (flags & SLIMDP_SELECT_REUSE_HISTOGRAM) != 0;
    if (reuse && !(ctx->hist_pending && ctx->hist_score == score))
        return fail(ctx, SLIMDP_ERR_INVALID_ARG,
                    "slimdp_select_core: no histogram pending for this score buffer (call slimdp_score first)");
    ctx->hist_pending = false;
    const uint32_t T = ctx->T, S = ctx->n_seg;
    int rc = wait_for_side(ctx);             // an explorer request on the side stream may still read the bitmap this call rewrites
    if (rc) return rc;
    const bool known = device_state_known(ctx);
    CoreArgs a{};
    a.tile_start = ctx->d_tile_start; a.tile_seg = ctx->d_tile_seg; a.seg_first_tile = ctx->d_seg_first_tile;
    a.n = ctx->n; a.T = T; a.n_seg = S;
    a.groups = core_groups(T, (uint32_t)ctx->cus);
    a.k_flat = (uint32_t)K;
    a.plan = ctx->c_plan; a.hist = ctx->c_hist; a.state = ctx->c_state;
    a.gt_bits = ctx->c_gt_bits; a.cand_bits = ctx->c_cand_bits; a.cand_keys = ctx->c_cand_keys;
    a.cnt_gt = ctx->c_cnt_gt; a.cnt_cand = ctx->c_cnt_cand;
    a.tile_pre = ctx->c_tile_pre; a.group_tail = ctx->c_group_tail; a.flags = ctx->d_flags;
    if (S > 1 && (!known || !std::equal(k_seg, k_seg + S, ctx->c_plan_k.begin(), ctx->c_plan_k.end()))) {
        ctx->c_plan_k.clear();               // whatever happens below: what the device holds is not known yet
        uint32_t base = 0;
        for (uint32_t s0 = 0; s0 < S; s0 += PLAN_CHUNK) {
            CorePlanChunk chunk;
            const uint32_t cnt = std::min(S - s0, (uint32_t)PLAN_CHUNK);
            memset(&chunk, 0, sizeof chunk);
            for (uint32_t j = 0; j < cnt; ++j) { chunk.s[j] = CorePlan{(uint32_t)k_seg[s0 + j], base}; base += (uint32_t)k_seg[s0 + j]; }
            hipLaunchKernelGGL(k_core_plan, dim3(1), dim3(PLAN_CHUNK), 0, ctx->stream, ctx->c_plan, chunk, s0, cnt);
            SLIMDP_LAUNCHED(ctx, "k_core_plan");
        }
        ctx->c_plan_k.assign(k_seg, k_seg + S);
    }
    if (!reuse) {
        if (!known || !ctx->hist_clean) { rc = fill(ctx, ctx->c_hist, (uint64_t)S * H_STRIDE, 0u); if (rc) return rc; }
        ctx->hist_clean = false;
        uint32_t P0 = persistent_blocks(ctx, 4, 1);
        if (S == 1) P0 = (uint32_t)std::min<uint64_t>((uint64_t)ctx->cus * 4, (ctx->n / 4 + BLOCK - 1) / BLOCK + 1);
        hipLaunchKernelGGL(k_core_hist0, dim3(P0), dim3(BLOCK), 0, ctx->stream, score, a);
        SLIMDP_LAUNCHED(ctx, "k_core_hist0");
    }
    // did the scoring pass that made this histogram already sort the whole tiles against a predicted bin?
    const bool classified = reuse && ctx->cls_by_score;
    ctx->cls_by_score = false;
    ctx->hist_clean = false;
    const uint32_t P = persistent_blocks(ctx, (uint32_t)ctx->opt_build_blocks, 1);
    hipLaunchKernelGGL(k_core_build, dim3(P), dim3(BLOCK), 0, ctx->stream, score, a, ctx->c_used, (int)classified, (int)reuse,
                       (int)(S == 1 && ctx->opt_strided), S > 1 ? core_bits : nullptr);
    SLIMDP_LAUNCHED(ctx, "k_core_build");
    hipLaunchKernelGGL(k_core_hist2, dim3(a.groups), dim3(BLOCK), 0, ctx->stream, a);
    SLIMDP_LAUNCHED(ctx, "k_core_hist2");
    // speculative packing: this selection rates the capture of the scoring pass it reuses and sets the next bound
    const bool spec_sel = ctx->spec.on && ctx->spec.mem && ctx->spec.captured && reuse && ctx->spec.score == score;
    SpecTau sp{nullptr, nullptr, nullptr};
    if (spec_sel) sp = SpecTau{ctx->spec.lo[ctx->spec.cur], ctx->spec.lo[ctx->spec.cur ^ 1], ctx->spec.fail};
    hipLaunchKernelGGL(k_core_count, dim3(a.groups), dim3(BLOCK), 0, ctx->stream, a, sp, ctx->c_pred);
    SLIMDP_LAUNCHED(ctx, "k_core_count");
    const uint32_t per_group = ((T + a.groups - 1) / a.groups + 7) / 8;      // at most two tiles per wave and block
    hipLaunchKernelGGL(k_core_emit, dim3(a.groups * per_group), dim3(BLOCK), 0, ctx->stream, a, per_group, core_idx, core_off,
                       core_bits, (uint32_t)K);
    SLIMDP_LAUNCHED(ctx, "k_core_emit");
    ctx->hist_clean = known;                 // a recorded selection has cleared nothing yet
    *core_epoch = ++ctx->epoch;
    ctx->last_K = K; ctx->have_last_K = true;
    if (spec_sel) { ctx->spec.core_epoch = ctx->epoch; ctx->spec.next_written = true; }
    else ctx->spec.core_epoch = 0;
    return SLIMDP_OK;
}

int slimdp_select_core(slimdp_ctx* ctx, const float* score, const uint64_t* k_seg, uint32_t flags, uint32_t* core_idx,
                       uint32_t* core_bits, uint32_t* core_off, uint64_t* core_epoch)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    return select_core_impl(ctx, score, k_seg, flags, core_idx, core_bits, core_off, core_epoch);
}

// ------------------------------------------------------------------------------------------
// Core selection for callers that cannot allocate: no context, no hipMalloc.  The workspace is
// a file-scope array in device memory (one copy per GPU, held until the process ends); the
// host uses its per-device address obtained from the runtime, never the symbol itself.
// ------------------------------------------------------------------------------------------
#define SLIMDP_STATIC_SCRATCH_BYTES (5u << 20)
static __device__ __align__(256) unsigned char scratch[SLIMDP_STATIC_SCRATCH_BYTES];

namespace {
struct StaticDev { void* ptr = nullptr; int cus = 0; bool dirty = false; };   // dirty: the histogram may not be clear
constexpr int STATIC_MAX_DEVICES = 64;
StaticDev g_static[STATIC_MAX_DEVICES];
std::mutex g_static_mu;
}  // namespace

int slimdp_select_core_static(const float* score, uint64_t n, uint64_t k, uint32_t* core_idx, uint32_t* core_bits,
                              uint32_t* core_off, void* hip_stream)
{
    if (!score || !core_bits || !core_off || (k && !core_idx))
        return fail(nullptr, SLIMDP_ERR_INVALID_ARG, "slimdp_select_core_static: NULL argument");
    if (n == 0 || n > SLIMDP_STATIC_MAX_N)
        return fail(nullptr, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_select_core_static: n=%llu outside [1, %u] (the static workspace "
                    "serves at most SLIMDP_STATIC_MAX_N parameters; larger models need a context)",
                    (unsigned long long)n, (unsigned)SLIMDP_STATIC_MAX_N);
    if (k > n) return fail(nullptr, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_select_core_static: k exceeds n");
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return hip_fail(nullptr, e, "hipGetDevice");
    if (device < 0 || device >= STATIC_MAX_DEVICES)
        return fail(nullptr, SLIMDP_ERR_INVALID_ARG, "slimdp_select_core_static: device %d not supported", device);
    StaticDev sdv;
    {
        std::lock_guard<std::mutex> lock(g_static_mu);
        if (!g_static[device].ptr) {          // once per device, with that device current: this GPU's copy of the array
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) return hip_fail(nullptr, e, "hipGetSymbolAddress(scratch)");
            int cus = 0;
            e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
            if (e != hipSuccess) return hip_fail(nullptr, e, "hipDeviceGetAttribute");
            g_static[device].cus = cus > 0 ? cus : 256;
            g_static[device].ptr = p;
        }
        sdv = g_static[device];
    }
    // a context on the stack whose device pointers lie inside this GPU's array (host members only, nothing allocated on the device)
    slimdp_ctx tmp;
    const uint64_t so[2] = {0, n};
    tmp.n = n; tmp.maxW = 1; tmp.n_seg = 1; tmp.seed = 0;
    tmp.stream = static_cast<hipStream_t>(hip_stream);
    tmp.device = device; tmp.cus = sdv.cus;
    tmp.seg_off.assign(so, so + 2);
    tmp.T = (uint32_t)count_tiles(n, 1, so);
    tmp.keys_stride = align_up(n, TILE) + TILE;
    Carver cv(static_cast<char*>(sdv.ptr));
    carve_core(&tmp, cv);
    if (cv.pos > SLIMDP_STATIC_SCRATCH_BYTES)
        return fail(nullptr, SLIMDP_ERR_WORKSPACE, "slimdp_select_core_static: %zu bytes of workspace needed, %u available",
                    cv.pos, (unsigned)SLIMDP_STATIC_SCRATCH_BYTES);
    // the array keeps the previous call's contents: a flat model reads no tables, and the selection leaves the
    // histogram clear unless it was only recorded or a launch failed on the way
    tmp.hist_clean = !sdv.dirty;
    uint64_t epoch = 0;
    const int rc = select_core_impl(&tmp, score, &k, 0u, core_idx, core_bits, core_off, &epoch);
    if (rc) g_create_error = tmp.err;
    if (tmp.hist_clean == sdv.dirty) {
        std::lock_guard<std::mutex> lock(g_static_mu);
        g_static[device].dirty = !tmp.hist_clean;
    }
    return rc;
}

int slimdp_import_core(slimdp_ctx* ctx, const uint32_t* core_idx, const uint64_t* k_seg, uint32_t* core_bits,
                       uint32_t* core_off, uint64_t* core_epoch)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!k_seg || !core_bits || !core_off || !core_epoch) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_import_core: NULL argument");
    uint64_t K = 0;
    for (uint32_t s = 0; s < ctx->n_seg; ++s) {
        if (k_seg[s] > ctx->seg_off[s + 1] - ctx->seg_off[s])
            return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_import_core: k_seg[%u] exceeds the segment size", s);
        K += k_seg[s];
    }
    if (K && !core_idx) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_import_core: core_idx is NULL");
    int rc = wait_for_side(ctx);
    if (rc) return rc;
    rc = fill(ctx, core_bits, (ctx->n + 31) / 32, 0u);
    if (rc) return rc;
    if (K) {
        hipLaunchKernelGGL(k_bits_from_idx, dim3(fill_grid(K)), dim3(256), 0, ctx->stream, core_idx, K, ctx->n, core_bits);
        SLIMDP_LAUNCHED(ctx, "k_bits_from_idx");
    }
    hipLaunchKernelGGL(k_tile_offsets, dim3((ctx->T + 1 + 255) / 256), dim3(256), 0, ctx->stream, core_idx, K, ctx->d_tile_start,
                       ctx->T, ctx->n, core_off);
    SLIMDP_LAUNCHED(ctx, "k_tile_offsets");
    ctx->hist_pending = false;
    ctx->spec.core_epoch = 0;
    *core_epoch = ++ctx->epoch;
    ctx->last_K = K; ctx->have_last_K = true;
    return SLIMDP_OK;
}

int slimdp_sample_explore(slimdp_ctx* ctx, const uint32_t* core_bits, const uint64_t* k_seg, uint32_t worker0,
                          uint32_t n_workers, uint64_t iteration, const uint64_t* m_seg, uint32_t* const* expl_idx,
                          uint32_t* const* expl_off)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!core_bits || !k_seg || !m_seg) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_sample_explore: NULL argument");
    if (n_workers == 0 || n_workers > ctx->maxW)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_sample_explore: n_workers=%u outside [1, %u]", n_workers, ctx->maxW);
    if (!table_ok(expl_off, n_workers)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_sample_explore: NULL expl_off entry");
    int rc = explorer_plan(ctx, "slimdp_sample_explore", k_seg, m_seg, n_workers);
    if (rc) return rc;
    const uint64_t M = ctx->plan.M;
    const bool short_list = ctx->plan.pairs;
    if (M > 0 && !table_ok(expl_idx, n_workers)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_sample_explore: NULL expl_idx entry");
    const uint32_t T = ctx->T, S = ctx->n_seg, B = n_workers;
    const bool known = device_state_known(ctx);      // a recorded request draws again when it is replayed
    // zones already drawn inside slimdp_score for exactly this request, in the format this call wants?
    const bool cached = ctx->pre.same(iteration, worker0, n_workers, k_seg, m_seg, S) && ctx->pre.pairs == short_list;
    ctx->pre.valid = false;
    ctx->hint.valid = false;
    // Option "explore_async": the whole request runs on the library's side stream, beside whatever the caller enqueues
    // on the context's stream after this call; the calls that take the lists make the context's stream wait for them.
    const bool async = ctx->opt_explore_async != 0 && !stays_on_main(ctx, B, cached);
    ctx->asked_epoch = ctx->epoch;
    hipStream_t st = async ? ctx->side : ctx->stream;
    if (async) {
        // everything enqueued so far comes first: the selection that wrote core_bits, readers of the output arrays
        SLIMDP_HIP(ctx, hipEventRecord(ctx->ev_consumed, ctx->stream));
        SLIMDP_HIP(ctx, hipStreamWaitEvent(ctx->side, ctx->ev_consumed, 0));
        ctx->side_pending = false;       // a draw on the side stream precedes this request in stream order
    } else {
        rc = wait_for_side(ctx);         // an announced draw, or an earlier asynchronous request: their buffers are theirs until done
        if (rc) return rc;
    }
    rc = init_states(ctx, ctx->e_state, ctx->e_state_holds, ctx->plan.init, known, !known || !ctx->lists_clean, ctx->maxW, st);
    if (rc) return rc;
    ctx->lists_clean = false;
    const RerunFlag rerun = rerun_flag(ctx);
    const uint32_t P = persistent_blocks(ctx, 8, B);
    const uint32_t G = draw_group(ctx, 4, B);
    // a tile or a few to a block, so that no unit is left with a whole turn more than the others (20*10^6 parameters, 3 workers:
    // 36 us with at most eight blocks a unit, 33 with one tile to a block).  Beside other work one or two workers' draw leaves it more
    // room in few blocks (cached core keys, one iteration ahead, eight / thirty-two a unit, us: 20*10^6, 1 worker 86 / 88; 60*10^6, 1 220 /
    // 224; 64*10^6, 2 300 / 305), more workers' does not end in time (10^7 in 57 segments, 4 123 / 118; 30*10^6, 8 361 / 358).
    const dim3 draw_grid(persistent_blocks(ctx, async && B <= 2 ? 8 : 32, (B + G - 1) / G), (B + G - 1) / G);
    const uint32_t n_words = (uint32_t)((ctx->n + 31) / 32);
    const PhiloxKey pk{(uint32_t)ctx->seed, (uint32_t)(ctx->seed >> 32), (uint32_t)iteration, (uint32_t)(iteration >> 32)};
    MutPtrTab off_tab = make_tab<MutPtrTab>(expl_off, B);
    MutPtrTab idx_tab = make_tab<MutPtrTab>(expl_idx, B);
#define LAUNCH_DRAW(PAIRS)                                                                                               \
    do {                                                                                                                 \
        if (ctx->tl.quad_aligned)                                                                                        \
            hipLaunchKernelGGL((k_explore_keys<0, PAIRS>), draw_grid, dim3(BLOCK), 0, st, ctx->d_tile_start,        \
                               ctx->d_tile_seg, T, S, ctx->e_state, ctx->e_sure_bits, ctx->e_cand_bits,                  \
                               (PAIRS) ? ctx->e_pair_keys : ctx->e_cand_keys, ctx->e_cnt_cand,                           \
                               (PAIRS) ? ctx->pair_stride : ctx->keys_stride, worker0, B, G, pk);                        \
        else                                                                                                             \
            hipLaunchKernelGGL((k_explore_keys<1, PAIRS>), draw_grid, dim3(BLOCK), 0, st, ctx->d_tile_start,        \
                               ctx->d_tile_seg, T, S, ctx->e_state, ctx->e_sure_bits, ctx->e_cand_bits,                  \
                               (PAIRS) ? ctx->e_pair_keys : ctx->e_cand_keys, ctx->e_cnt_cand,                           \
                               (PAIRS) ? ctx->pair_stride : ctx->keys_stride, worker0, B, G, pk);                        \
        SLIMDP_LAUNCHED(ctx, "k_explore_keys");                                                                          \
    } while (0)
    const ExploreLists lists{ctx->e_list, ctx->e_list_count, ctx->d_list_first, ctx->list_first[S], (uint32_t)align_up(S, 32)};
    if (short_list) {
        constexpr int SBPW = 8;
        if (!cached) { ctx->spec.expl_slots = 0; LAUNCH_DRAW(1); }
        const uint32_t sure_blocks = ((T + 3) / 4) * ((B + SBPW - 1) / SBPW);
        const uint32_t gather_blocks = B * ((T + 63) / 64);
        hipLaunchKernelGGL(k_explore_collect<SBPW>, dim3(sure_blocks + gather_blocks), dim3(BLOCK), 0, st, core_bits, n_words, ctx->n,
                           ctx->d_tile_start, ctx->d_tile_seg, T, S, B, sure_blocks, ctx->e_sure_bits, ctx->e_cnt_sel,
                           ctx->e_pair_keys, ctx->pair_stride, ctx->e_cnt_cand, lists, rerun.now);
        SLIMDP_LAUNCHED(ctx, "k_explore_collect");
    } else {
        rc = ensure_wide_keys(ctx);
        if (rc) return rc;
        if (!cached) { ctx->spec.expl_slots = 0; LAUNCH_DRAW(0); }
        hipLaunchKernelGGL(k_explore_collect_wide, dim3(P, B), dim3(BLOCK), 0, st, core_bits, n_words, ctx->n, ctx->d_tile_start,
                           ctx->d_tile_seg, T, S, ctx->e_sure_bits, ctx->e_cnt_sel, ctx->e_cand_bits, ctx->e_cand_keys,
                           ctx->keys_stride, lists, rerun.now);
        SLIMDP_LAUNCHED(ctx, "k_explore_collect_wide");
    }
    // a block of 1024 threads has the shorter chain; small blocks where there are many more of them than run at a time
    if ((uint64_t)S * B <= 4ull * ctx->cus)
        hipLaunchKernelGGL(k_explore_select<1024>, dim3(S, B), dim3(1024), 0, st, ctx->e_state, ctx->d_seg_first_tile, T, S, lists,
                           ctx->e_cnt_sel, ctx->e_sure_bits, off_tab, rerun.now);
    else
        hipLaunchKernelGGL(k_explore_select<256>, dim3(S, B), dim3(256), 0, st, ctx->e_state, ctx->d_seg_first_tile, T, S, lists,
                           ctx->e_cnt_sel, ctx->e_sure_bits, off_tab, rerun.now);
    SLIMDP_LAUNCHED(ctx, "k_explore_select");
    constexpr int EBPW = 4;
#define LAUNCH_EMIT(NT)                                                                                                          \
    do {                                                                                                                         \
        const uint32_t blocks = (T + (NT) / 64 - 1) / ((NT) / 64);                                                               \
        hipLaunchKernelGGL((k_explore_emit<EBPW, NT>), dim3(std::max(blocks, (uint32_t)EBPW), (B + EBPW - 1) / EBPW), dim3(NT), 0, st,  \
                           core_bits, n_words, ctx->n, ctx->d_tile_start, ctx->d_tile_seg, ctx->d_seg_first_tile, T, S, B,       \
                           ctx->e_state, worker0, pk, ctx->e_sure_bits, off_tab, idx_tab, (uint32_t)M, rerun, ctx->d_flags);     \
        SLIMDP_LAUNCHED(ctx, "k_explore_emit");                                                                                  \
    } while (0)
    if (async) LAUNCH_EMIT(256); else LAUNCH_EMIT(1024);
#undef LAUNCH_EMIT
    ctx->lists_clean = known;                // a recorded request has cleared nothing yet
    ctx->rerun_turn ^= 1u;
#undef LAUNCH_DRAW
    if (async) {
        // a free slot, else the oldest one (the main stream then waits for that request first)
        int slot = -1;
        for (int j = 0; j < slimdp_ctx::N_PENDING && slot < 0; ++j)
            if (!ctx->pend[j].live) slot = j;
        if (slot < 0) {
            slot = 0;
            for (int j = 1; j < slimdp_ctx::N_PENDING; ++j)
                if (ctx->pend[j].seq < ctx->pend[slot].seq) slot = j;
            SLIMDP_HIP(ctx, hipStreamWaitEvent(ctx->stream, ctx->pend[slot].ev, 0));
        }
        slimdp_ctx::PendingExplore& p = ctx->pend[slot];
        SLIMDP_HIP(ctx, hipEventRecord(p.ev, ctx->side));
        p.live = true; p.seq = ++ctx->pend_seq; p.nw = B;
        p.idx_bytes = std::max<uint64_t>(M * 4, 4); p.off_bytes = ((uint64_t)T + 1) * 4;
        for (uint32_t q = 0; q < B; ++q) {
            p.idx[q] = reinterpret_cast<uintptr_t>(expl_idx ? expl_idx[q] : nullptr);
            p.off[q] = reinterpret_cast<uintptr_t>(expl_off[q]);
        }
    }
    return SLIMDP_OK;
}

int slimdp_explore_hint(slimdp_ctx* ctx, const uint64_t* k_seg, uint32_t worker0, uint32_t n_workers,
                        uint64_t iteration, const uint64_t* m_seg)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    ctx->hint.valid = false;
    if (!k_seg || !m_seg) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_explore_hint: NULL argument");
    if (n_workers == 0 || n_workers > ctx->maxW)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_explore_hint: n_workers=%u outside [1, %u]", n_workers, ctx->maxW);
    int rc = explorer_plan(ctx, "slimdp_explore_hint", k_seg, m_seg, n_workers);
    if (rc) return rc;
    const bool short_list = ctx->plan.pairs;
    ctx->hint.iteration = iteration; ctx->hint.worker0 = worker0; ctx->hint.n_workers = n_workers;
    ctx->hint.k_seg.assign(k_seg, k_seg + ctx->n_seg);
    ctx->hint.m_seg.assign(m_seg, m_seg + ctx->n_seg);
    if (ctx->opt_hint_mode == 0) {           // slimdp_score will draw
        ctx->hint.valid = true;
        return SLIMDP_OK;
    }
    if (!ctx->plan.narrow || ctx->plan.M == 0) return SLIMDP_OK;  // nothing worth drawing ahead: slimdp_sample_explore draws itself
    if (!short_list) { rc = ensure_wide_keys(ctx); if (rc) return rc; }
    if (draw_waits(ctx, n_workers)) return SLIMDP_OK;                // nor this: the request will draw
    const bool known = device_state_known(ctx);
    // the draw starts now on the side stream, once the previous draw's buffers have been read
    // (the event is recorded here, not after every slimdp_sample_explore: an event on a stream costs a gap between kernels)
    SLIMDP_HIP(ctx, hipEventRecord(ctx->ev_consumed, ctx->stream));
    SLIMDP_HIP(ctx, hipStreamWaitEvent(ctx->side, ctx->ev_consumed, 0));
    rc = init_states(ctx, ctx->e_draw_state, ctx->e_draw_holds, ctx->plan.init, known, false, 0, ctx->side);
    if (rc) return rc;
    ctx->spec.expl_slots = 0;
    // few waves keep the arithmetic units busy; the wave slots stay with the kernels of the main stream
    const uint32_t G = draw_group(ctx, (uint32_t)ctx->opt_side_blocks, n_workers), groups = (n_workers + G - 1) / G;
    const uint32_t P = persistent_blocks(ctx, (uint32_t)ctx->opt_side_blocks, groups);
    const PhiloxKey pk{(uint32_t)ctx->seed, (uint32_t)(ctx->seed >> 32), (uint32_t)iteration, (uint32_t)(iteration >> 32)};
    const dim3 grid(P, groups), block(BLOCK);
#define LAUNCH_SIDE_DRAW(MIS, PAIRS)                                                                                    \
    hipLaunchKernelGGL((k_explore_keys<MIS, PAIRS>), grid, block, 0, ctx->side, ctx->d_tile_start, ctx->d_tile_seg,    \
                       ctx->T, ctx->n_seg, ctx->e_draw_state, ctx->e_sure_bits, ctx->e_cand_bits,                       \
                       (PAIRS) ? ctx->e_pair_keys : ctx->e_cand_keys, ctx->e_cnt_cand,                                  \
                       (PAIRS) ? ctx->pair_stride : ctx->keys_stride, worker0, n_workers, G, pk)
    if (ctx->tl.quad_aligned) { if (short_list) LAUNCH_SIDE_DRAW(0, 1); else LAUNCH_SIDE_DRAW(0, 0); }
    else { if (short_list) LAUNCH_SIDE_DRAW(1, 1); else LAUNCH_SIDE_DRAW(1, 0); }
#undef LAUNCH_SIDE_DRAW
    SLIMDP_LAUNCHED(ctx, "k_explore_keys(side stream)");
    SLIMDP_HIP(ctx, hipEventRecord(ctx->ev_drawn, ctx->side));
    ctx->side_pending = ctx->draw_fresh = true;
    ctx->pre = ctx->hint;
    ctx->pre.valid = true;
    ctx->pre.pairs = short_list;
    return SLIMDP_OK;
}

int slimdp_tile_offsets(slimdp_ctx* ctx, const uint32_t* idx, uint64_t count, uint32_t* off)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!off || (count && !idx)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_tile_offsets: NULL argument");
    if (count > ctx->n) return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_tile_offsets: count exceeds n");
    hipLaunchKernelGGL(k_tile_offsets, dim3((ctx->T + 1 + 255) / 256), dim3(256), 0, ctx->stream, idx, count,
                       ctx->d_tile_start, ctx->T, ctx->n, off);
    SLIMDP_LAUNCHED(ctx, "k_tile_offsets");
    return SLIMDP_OK;
}

static int check_lists(slimdp_ctx* ctx, const char* who, uint32_t n_workers, const uint32_t* core_idx,
                       const uint32_t* core_off, uint64_t k, const uint32_t* const* expl_idx,
                       const uint32_t* const* expl_off, const uint64_t* m_w)
{
    if (n_workers == 0 || n_workers > ctx->maxW)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: n_workers=%u outside [1, %u]", who, n_workers, ctx->maxW);
    if (!core_off || (k && !core_idx) || !m_w) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: NULL argument", who);
    if (k > ctx->n) return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "%s: k exceeds n", who);
    if (!table_ok(expl_off, n_workers)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: NULL expl_off entry", who);
    for (uint32_t q = 0; q < n_workers; ++q) {
        if (m_w[q] > ctx->n - k) return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "%s: m_w[%u] exceeds n - k", who, q);
        if (m_w[q] && (!expl_idx || !expl_idx[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: NULL expl_idx entry", who);
    }
    return SLIMDP_OK;
}

int slimdp_pack(slimdp_ctx* ctx, uint32_t n_workers, const float* const* g, const uint32_t* core_idx,
                const uint32_t* core_off, uint64_t k, const uint32_t* const* expl_idx, const uint32_t* const* expl_off,
                const uint64_t* m_w, float* const* core_val, float* const* expl_val, uint64_t core_epoch, uint32_t flags)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (flags & ~SLIMDP_PACK_UPDATES_AS_SCORED) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pack: unknown flag bits 0x%x", flags);
    int rc = check_lists(ctx, "slimdp_pack", n_workers, core_idx, core_off, k, expl_idx, expl_off, m_w);
    if (rc) return rc;
    if (!table_ok(g, n_workers)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pack: NULL update pointer");
    for (uint32_t q = 0; q < n_workers; ++q) {
        if (k && (!core_val || !core_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pack: NULL core_val entry");
        if (m_w[q] && (!expl_val || !expl_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pack: NULL expl_val entry");
    }
    rc = check_epoch(ctx, core_epoch);
    if (rc) return rc;
    // The caller states that g is what the last scoring pass read.  That the contents are unchanged cannot be
    // checked here; that it is the same table can.
    const bool as_scored = (flags & SLIMDP_PACK_UPDATES_AS_SCORED) != 0;
    if (as_scored && ctx->spec.captured) {
        bool same = ctx->spec.W == n_workers;
        for (uint32_t q = 0; same && q < n_workers; ++q) same = ctx->spec.g[q] == g[q];
        if (!same)
            return fail(ctx, SLIMDP_ERR_INVALID_ARG,
                        "slimdp_pack: SLIMDP_PACK_UPDATES_AS_SCORED, but g is not the table of arrays the last slimdp_score read");
    }
    // the scoring pass of this very selection kept the core's update values: no second pass over the updates
    const bool spec = as_scored && ctx->spec.on && ctx->spec.captured && ctx->spec.core_epoch == core_epoch;
    if (spec) {
        ctx->spec.captured = false;      // one capture serves one pack
        bool side_busy = false;
        for (int j = 0; j < slimdp_ctx::N_PENDING; ++j) side_busy = side_busy || ctx->pend[j].live;
        uint64_t core_blocks = 0;
        if (k && ctx->n_seg == 1) {
            // many short blocks: work on the side stream (an asynchronous explorer request) gets its turn between them
            core_blocks = (k + 1023) / 1024;
            if (core_blocks > 32768) core_blocks = 32768;
            // while an explorer request runs on the side stream: few resident blocks, so that its small kernels find free
            // slots at once (measured: 2.54 -> 2.48 ms per step with one block per compute unit)
            const uint64_t per_cu = ctx->opt_pack_core_blocks > 0 ? (uint64_t)ctx->opt_pack_core_blocks : (side_busy ? 1u : 0u);
            if (per_cu > 0 && core_blocks > (uint64_t)ctx->cus * per_cu) core_blocks = (uint64_t)ctx->cus * per_cu;
        } else if (k) {
            core_blocks = (ctx->T + 3) / 4;
        }
        CountTab mt{};
        uint64_t mmax = 0;
        for (uint32_t q = 0; q < n_workers; ++q) { mt.c[q] = (uint32_t)m_w[q]; if (m_w[q] > mmax) mmax = m_w[q]; }
        uint64_t gather_blocks = (mmax + 1023) / 1024;
        if (gather_blocks > 2048) gather_blocks = 2048;
        auto launch = [&](uint64_t cb, uint64_t gb) {
            if (cb + gb == 0) return;
            const dim3 grid((uint32_t)(cb + gb * n_workers));
            auto go = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), 0, ctx->stream, (uint32_t)cb, (uint32_t)gb, make_tab<PtrTab>(g, n_workers), n_workers,
                                   ctx->n, ctx->d_tile_start, ctx->d_tile_seg, ctx->T, core_idx, core_off, (uint32_t)k, ctx->spec.bits,
                                   ctx->spec.vals, ctx->spec.fail, make_tab<MutPtrTab>(core_val, n_workers),
                                   make_tab<PtrTab>(expl_idx, n_workers), mt, make_tab<MutPtrTab>(expl_val, n_workers));
            };
            if (ctx->n_seg == 1) go(k_pack_spec<1>); else go(k_pack_spec<0>);
        };
        const bool kept = mmax && ctx->spec.expl_slots && device_state_known(ctx);
        // the core values do not need the explorer lists: while a request is on its way they go first
        if (side_busy || kept) { launch(core_blocks, 0); SLIMDP_LAUNCHED(ctx, "k_pack_spec"); core_blocks = 0; }
        rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
        if (rc) return rc;
        if (!kept) { launch(core_blocks, gather_blocks); SLIMDP_LAUNCHED(ctx, "k_pack_spec"); }
        if (kept) {
            hipLaunchKernelGGL(k_pack_expl_spec, dim3((ctx->T + 3) / 4, (n_workers + PEXP - 1) / PEXP), dim3(BLOCK), 0, ctx->stream,
                               make_tab<PtrTab>(g, n_workers), n_workers, ctx->n, ctx->T, (uint32_t)(ctx->n / TILE),
                               make_tab<PtrTab>(expl_idx, n_workers), make_tab<PtrTab>(expl_off, n_workers), mt, ctx->e_sure_bits,
                               ctx->e_pair_keys, ctx->pair_stride, ctx->e_cnt_cand, ctx->spec.evals, ctx->spec.expl_slots,
                               make_tab<MutPtrTab>(expl_val, n_workers));
            SLIMDP_LAUNCHED(ctx, "k_pack_expl_spec");
        }
        return SLIMDP_OK;
    }
    rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
    if (rc) return rc;
    if (ctx->opt_pack_kernel == 1) {
        hipLaunchKernelGGL(k_pack_stream_ws, dim3(8 * ((ctx->T + 7) / 8)), dim3(2 * BLOCK), 0, ctx->stream,
                           make_tab<PtrTab>(g, n_workers), n_workers, ctx->T, ctx->d_tile_start, core_idx, core_off,
                           make_tab<PtrTab>(expl_idx, n_workers), make_tab<PtrTab>(expl_off, n_workers),
                           make_tab<MutPtrTab>(core_val, n_workers), make_tab<MutPtrTab>(expl_val, n_workers));
        SLIMDP_LAUNCHED(ctx, "k_pack_stream_ws");
        return SLIMDP_OK;
    }
    int vec_ok = 1;
    for (uint32_t q = 0; q < n_workers; ++q) vec_ok = vec_ok && aligned16(g[q]);
    if (ctx->opt_pack_nbuf == 2)
        hipLaunchKernelGGL(k_pack_stream<2>, dim3(ctx->T), dim3(BLOCK), 0, ctx->stream, make_tab<PtrTab>(g, n_workers),
                           n_workers, ctx->d_tile_start, core_idx, core_off, make_tab<PtrTab>(expl_idx, n_workers),
                           make_tab<PtrTab>(expl_off, n_workers), make_tab<MutPtrTab>(core_val, n_workers),
                           make_tab<MutPtrTab>(expl_val, n_workers), vec_ok);
    else
        hipLaunchKernelGGL(k_pack_stream<1>, dim3(ctx->T), dim3(BLOCK), 0, ctx->stream, make_tab<PtrTab>(g, n_workers),
                           n_workers, ctx->d_tile_start, core_idx, core_off, make_tab<PtrTab>(expl_idx, n_workers),
                           make_tab<PtrTab>(expl_off, n_workers), make_tab<MutPtrTab>(core_val, n_workers),
                           make_tab<MutPtrTab>(expl_val, n_workers), vec_ok);
    SLIMDP_LAUNCHED(ctx, "k_pack_stream");
    return SLIMDP_OK;
}

int slimdp_merge(slimdp_ctx* ctx, float* w, float lr, uint64_t core_epoch, uint32_t n_workers, const uint32_t* core_idx,
                 const uint32_t* core_off, uint64_t k, const float* const* core_val, const uint32_t* const* expl_idx,
                 const uint32_t* const* expl_off, const float* const* expl_val, const uint64_t* m_w)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!w) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_merge: w is NULL");
    int rc = check_lists(ctx, "slimdp_merge", n_workers, core_idx, core_off, k, expl_idx, expl_off, m_w);
    if (rc) return rc;
    for (uint32_t q = 0; q < n_workers; ++q) {
        if (k && (!core_val || !core_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_merge: NULL core_val entry");
        if (m_w[q] && (!expl_val || !expl_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_merge: NULL expl_val entry");
    }
    rc = check_epoch(ctx, core_epoch);
    if (rc) return rc;
    rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
    if (rc) return rc;
    // Entries a tile is expected to hold, with six standard deviations: the variant that keeps them in registers (the staged
    // path costs 20*10^6 parameters, 3 workers, 1,776 entries a tile 79 us, eight entries per thread 66).  Sixteen take 104
    // registers, four blocks to a compute unit instead of seven: that pays only while the tiles are few enough to run in
    // two turns (8 workers, 3,200 a tile: 245 tiles 22.9 against 26.6 us staged, 1,954 tiles 63.7 against 66.8, but 2,100
    // tiles 81 against 69, 33,779 tiles 1,027 against 734).  With more tiles eight serve as long as half of them fit
    // (1,950 a tile, 138*10^6 parameters, 2 workers: 414 against 434 us staged and 593 with sixteen).
    double per_tile = 0.0;
    for (uint32_t q = 0; q < n_workers; ++q) per_tile += (double)m_w[q] * TILE / (double)ctx->n;
    const double room = per_tile + 6.0 * std::sqrt(per_tile);
    const bool few_tiles = ctx->T <= 8u * (uint32_t)ctx->cus;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(ctx->T), dim3(BLOCK), 0, ctx->stream, w, lr, n_workers, ctx->d_tile_start, core_idx, core_off,
                           make_tab<PtrTab>(core_val, n_workers), make_tab<PtrTab>(expl_idx, n_workers),
                           make_tab<PtrTab>(expl_off, n_workers), make_tab<PtrTab>(expl_val, n_workers), ctx->n, ctx->n_seg);
    };
    const bool lines = ctx->n_seg == 1 && aligned16(w);
#define LAUNCH_MERGE(R) do { if (lines) launch(k_merge<R, 1>); else launch(k_merge<R, 0>); } while (0)
    if (room <= 4.0 * BLOCK) LAUNCH_MERGE(4);
    else if ((few_tiles ? room : per_tile) <= 8.0 * BLOCK) LAUNCH_MERGE(8);
    else if (few_tiles && room <= 16.0 * BLOCK) LAUNCH_MERGE(16);
    else LAUNCH_MERGE(4);
#undef LAUNCH_MERGE
    SLIMDP_LAUNCHED(ctx, "k_merge");
    return SLIMDP_OK;
}

int slimdp_pull(slimdp_ctx* ctx, const float* w, uint64_t core_epoch, uint32_t n_workers, const uint32_t* core_idx,
                const uint32_t* core_off, uint64_t k, const uint32_t* const* expl_idx, const uint32_t* const* expl_off,
                const uint64_t* m_w, float* const* core_out, float* const* expl_out, float* const* w_local)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!w) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull: w is NULL");
    int rc = check_lists(ctx, "slimdp_pull", n_workers, core_idx, core_off, k, expl_idx, expl_off, m_w);
    if (rc) return rc;
    for (uint32_t q = 0; q < n_workers; ++q) {
        if (k && (!core_out || !core_out[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull: NULL core_out entry");
        if (m_w[q] && (!expl_out || !expl_out[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull: NULL expl_out entry");
        if (w_local && w_local[q] == w) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull: w_local aliases w");
    }
    rc = check_epoch(ctx, core_epoch);
    if (rc) return rc;
    rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
    if (rc) return rc;
    const float* src = w;
    bool any_local = false;
    for (uint32_t q = 0; w_local && q < n_workers; ++q) any_local = any_local || w_local[q] != nullptr;
    // The local models are patched by a pass that streams them (a scattered 4-byte write per value would touch nearly every
    // line of every local model, at a fraction of the rate); the values at the communication sets leave from the same pass.
    if (any_local && ctx->opt_pull_kernel == 1) {
        int vec_ok = aligned16(w);
        for (uint32_t q = 0; q < n_workers; ++q) vec_ok = vec_ok && (!w_local[q] || aligned16(w_local[q]));
        const uint32_t per = workers_per_block(ctx, n_workers);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(ctx->T, (n_workers + per - 1) / per), dim3(BLOCK), 0, ctx->stream, w,
                               make_tab<MutPtrTab>(w_local, n_workers), PtrTab{}, MutPtrTab{}, 0.0f, 1, n_workers, per, ctx->n,
                               ctx->d_tile_start, core_idx, core_off, make_tab<PtrTab>(expl_idx, n_workers),
                               make_tab<PtrTab>(expl_off, n_workers), make_tab<MutPtrTab>(core_out, n_workers),
                               make_tab<MutPtrTab>(expl_out, n_workers), vec_ok);
        };
        if (per < n_workers) launch(k_pull_local_step<0, 0, 1>);       // under 2^20 parameters: the caches hold them
        else if (local_streams(ctx, n_workers)) launch(k_pull_local_step<0, 1, 0>);
        else launch(k_pull_local_step<0, 0, 0>);
        SLIMDP_LAUNCHED(ctx, "k_pull_local_step<0>");
        return SLIMDP_OK;
    }
    hipLaunchKernelGGL(k_gather, dim3(ctx->T), dim3(BLOCK), 0, ctx->stream, make_tab<PtrTab, const float*>(&src, 1), 1,
                       n_workers, ctx->n, core_idx, core_off, make_tab<PtrTab>(expl_idx, n_workers),
                       make_tab<PtrTab>(expl_off, n_workers), make_tab<MutPtrTab>(core_out, n_workers),
                       make_tab<MutPtrTab>(expl_out, n_workers),
                       make_tab<MutPtrTab>(w_local, w_local ? n_workers : 0));
    SLIMDP_LAUNCHED(ctx, "k_gather(pull)");
    return SLIMDP_OK;
}

int slimdp_local_step(slimdp_ctx* ctx, uint32_t n_workers, float* const* w_local, const float* const* grad,
                      float* const* delta, float eta, uint32_t flags)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (flags & ~SLIMDP_LOCAL_FIRST) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step: unknown flag bits 0x%x", flags);
    if (n_workers == 0 || n_workers > ctx->maxW)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step: n_workers=%u outside [1, %u]", n_workers, ctx->maxW);
    if (!table_ok(w_local, n_workers) || !table_ok(grad, n_workers) || !table_ok(delta, n_workers))
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step: NULL array");
    if (!std::isfinite(eta)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step: eta must be finite");
    int vec_ok = 1;
    for (uint32_t q = 0; q < n_workers; ++q) {
        vec_ok = vec_ok && aligned16(w_local[q]) && aligned16(grad[q]) && aligned16(delta[q]);
        if (static_cast<const void*>(w_local[q]) == static_cast<const void*>(delta[q]) ||
            static_cast<const void*>(grad[q]) == static_cast<const void*>(delta[q]) ||
            static_cast<const void*>(grad[q]) == static_cast<const void*>(w_local[q]))
            return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step: arrays of worker %u alias", q);
    }
    uint64_t blocks = (ctx->n / 4 + 511) / 512;
    const uint64_t cap = (uint64_t)ctx->cus * 16 / n_workers + 1;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks, n_workers), dim3(256), 0, ctx->stream, make_tab<MutPtrTab>(w_local, n_workers),
                           make_tab<PtrTab>(grad, n_workers), make_tab<MutPtrTab>(delta, n_workers), ctx->n, eta,
                           (int)((flags & SLIMDP_LOCAL_FIRST) != 0), vec_ok);
    };
    if (local_streams(ctx, n_workers)) launch(k_local_step<1>); else launch(k_local_step<0>);
    SLIMDP_LAUNCHED(ctx, "k_local_step");
    return SLIMDP_OK;
}

int slimdp_local_step_pack(slimdp_ctx* ctx, uint32_t n_workers, float* const* w_local, const float* const* grad,
                           float* const* delta, float eta, uint32_t flags, const uint32_t* core_idx, const uint32_t* core_off,
                           uint64_t k, const uint32_t* const* expl_idx, const uint32_t* const* expl_off, const uint64_t* m_w,
                           float* const* core_val, float* const* expl_val, uint64_t core_epoch)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (flags & ~SLIMDP_LOCAL_FIRST) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: unknown flag bits 0x%x", flags);
    int rc = check_lists(ctx, "slimdp_local_step_pack", n_workers, core_idx, core_off, k, expl_idx, expl_off, m_w);
    if (rc) return rc;
    if (!table_ok(w_local, n_workers) || !table_ok(grad, n_workers) || !table_ok(delta, n_workers))
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: NULL array");
    if (!std::isfinite(eta)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: eta must be finite");
    int vec_ok = 1;
    for (uint32_t q = 0; q < n_workers; ++q) {
        vec_ok = vec_ok && aligned16(w_local[q]) && aligned16(grad[q]) && aligned16(delta[q]);
        if (static_cast<const void*>(w_local[q]) == static_cast<const void*>(delta[q]) ||
            static_cast<const void*>(grad[q]) == static_cast<const void*>(delta[q]) ||
            static_cast<const void*>(grad[q]) == static_cast<const void*>(w_local[q]))
            return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: arrays of worker %u alias", q);
        if (k && (!core_val || !core_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: NULL core_val entry");
        if (m_w[q] && (!expl_val || !expl_val[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_local_step_pack: NULL expl_val entry");
    }
    rc = check_epoch(ctx, core_epoch);
    if (rc) return rc;
    rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
    if (rc) return rc;
    const int first = (flags & SLIMDP_LOCAL_FIRST) != 0;
    const uint32_t per = workers_per_block(ctx, n_workers);
    const dim3 grid(ctx->T, (n_workers + per - 1) / per);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(BLOCK), 0, ctx->stream, make_tab<MutPtrTab>(w_local, n_workers),
                           make_tab<PtrTab>(grad, n_workers), make_tab<MutPtrTab>(delta, n_workers), eta, first, n_workers, per,
                           ctx->d_tile_start, core_idx, core_off, make_tab<PtrTab>(expl_idx, n_workers),
                           make_tab<PtrTab>(expl_off, n_workers), make_tab<MutPtrTab>(core_val, n_workers),
                           make_tab<MutPtrTab>(expl_val, n_workers), vec_ok);
    };
    const bool streams = fused_streams(ctx, n_workers, FUSED_PACK_HELD);
    if (per < n_workers) { if (ctx->opt_pack_nbuf == 2) launch(k_local_step_pack<2, 0, 1>); else launch(k_local_step_pack<1, 0, 1>); }
    else if (streams) { if (ctx->opt_pack_nbuf == 2) launch(k_local_step_pack<2, 1, 0>); else launch(k_local_step_pack<1, 1, 0>); }
    else { if (ctx->opt_pack_nbuf == 2) launch(k_local_step_pack<2, 0, 0>); else launch(k_local_step_pack<1, 0, 0>); }
    SLIMDP_LAUNCHED(ctx, "k_local_step_pack");
    return SLIMDP_OK;
}

int slimdp_pull_local_step(slimdp_ctx* ctx, const float* w, uint64_t core_epoch, uint32_t n_workers, const uint32_t* core_idx,
                           const uint32_t* core_off, uint64_t k, const uint32_t* const* expl_idx,
                           const uint32_t* const* expl_off, const uint64_t* m_w, float* const* w_local,
                           const float* const* grad, float* const* delta, float eta, uint32_t flags)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!w) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull_local_step: w is NULL");
    if (flags & ~SLIMDP_LOCAL_FIRST) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull_local_step: unknown flag bits 0x%x", flags);
    int rc = check_lists(ctx, "slimdp_pull_local_step", n_workers, core_idx, core_off, k, expl_idx, expl_off, m_w);
    if (rc) return rc;
    if (!table_ok(w_local, n_workers) || !table_ok(grad, n_workers) || !table_ok(delta, n_workers))
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull_local_step: NULL array");
    if (!std::isfinite(eta)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull_local_step: eta must be finite");
    int vec_ok = aligned16(w);
    for (uint32_t q = 0; q < n_workers; ++q) {
        vec_ok = vec_ok && aligned16(w_local[q]) && aligned16(grad[q]) && aligned16(delta[q]);
        const void *a = w_local[q], *b = grad[q], *c = delta[q];
        if (a == b || a == c || b == c || a == static_cast<const void*>(w) || c == static_cast<const void*>(w))
            return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_pull_local_step: arrays of worker %u alias", q);
    }
    rc = check_epoch(ctx, core_epoch);
    if (rc) return rc;
    rc = wait_for_lists(ctx, n_workers, expl_idx, expl_off, m_w);
    if (rc) return rc;
    const uint32_t per = workers_per_block(ctx, n_workers);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(ctx->T, (n_workers + per - 1) / per), dim3(BLOCK), 0, ctx->stream, w,
                           make_tab<MutPtrTab>(w_local, n_workers), make_tab<PtrTab>(grad, n_workers), make_tab<MutPtrTab>(delta, n_workers),
                           eta, (int)((flags & SLIMDP_LOCAL_FIRST) != 0), n_workers, per, ctx->n, ctx->d_tile_start, core_idx,
                           core_off, make_tab<PtrTab>(expl_idx, n_workers), make_tab<PtrTab>(expl_off, n_workers), MutPtrTab{}, MutPtrTab{},
                           vec_ok);
    };
    if (per < n_workers) launch(k_pull_local_step<1, 0, 1>);
    else if (fused_streams(ctx, n_workers, STREAMS_HELD)) launch(k_pull_local_step<1, 1, 0>);
    else launch(k_pull_local_step<1, 0, 0>);
    SLIMDP_LAUNCHED(ctx, "k_pull_local_step");
    return SLIMDP_OK;
}

static int quant_args(slimdp_ctx* ctx, const char* who, uint32_t n_workers, const void* const* a, const void* const* b,
                      const void* const* c, const uint64_t* count, Count64Tab* ct, uint64_t* cmax)
{
    if (n_workers == 0 || n_workers > ctx->maxW)
        return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: n_workers=%u outside [1, %u]", who, n_workers, ctx->maxW);
    if (!count || !a || !b || !c) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: NULL argument", who);
    *cmax = 0;
    for (uint32_t q = 0; q < n_workers; ++q) {
        if (count[q] > ctx->n) return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "%s: count[%u] exceeds n", who, q);
        if (count[q] && (!a[q] || !b[q] || !c[q])) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "%s: NULL array of worker %u", who, q);
        ct->c[q] = count[q];
        if (count[q] > *cmax) *cmax = count[q];
    }
    return SLIMDP_OK;
}

int slimdp_quantize(slimdp_ctx* ctx, uint32_t n_workers, uint32_t worker0, const float* const* val, const uint64_t* count,
                    uint32_t kind, uint64_t iteration, uint8_t* const* code, float* const* scale)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (kind > 1) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_quantize: kind must be 0 (core values) or 1 (explorer values)");
    Count64Tab ct{};
    uint64_t cmax = 0;
    int rc = quant_args(ctx, "slimdp_quantize", n_workers, reinterpret_cast<const void* const*>(val),
                        reinterpret_cast<const void* const*>(code), reinterpret_cast<const void* const*>(scale), count, &ct, &cmax);
    if (rc) return rc;
    if (cmax == 0) return SLIMDP_OK;
    int vec_ok = 1;
    for (uint32_t q = 0; q < n_workers; ++q)
        vec_ok = vec_ok && aligned16(val[q]) && (reinterpret_cast<uintptr_t>(code[q]) & 3u) == 0;
    const uint64_t buckets = (cmax + QB - 1) / QB;
    const PhiloxKey pk{(uint32_t)ctx->seed, (uint32_t)(ctx->seed >> 32), (uint32_t)iteration, (uint32_t)(iteration >> 32)};
    hipLaunchKernelGGL(k_quantize, dim3((uint32_t)((buckets + 3) / 4), n_workers), dim3(BLOCK), 0, ctx->stream,
                       make_tab<PtrTab>(val, n_workers), ct, kind, worker0, pk, make_tab<MutPtrTab>(code, n_workers),
                       make_tab<MutPtrTab>(scale, n_workers), vec_ok);
    SLIMDP_LAUNCHED(ctx, "k_quantize");
    return SLIMDP_OK;
}

int slimdp_dequantize(slimdp_ctx* ctx, uint32_t n_workers, const uint8_t* const* code, const float* const* scale,
                      const uint64_t* count, float* const* val)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    Count64Tab ct{};
    uint64_t cmax = 0;
    int rc = quant_args(ctx, "slimdp_dequantize", n_workers, reinterpret_cast<const void* const*>(code),
                        reinterpret_cast<const void* const*>(scale), reinterpret_cast<const void* const*>(val), count, &ct, &cmax);
    if (rc) return rc;
    if (cmax == 0) return SLIMDP_OK;
    int vec_ok = 1;
    for (uint32_t q = 0; q < n_workers; ++q)
        vec_ok = vec_ok && aligned16(val[q]) && (reinterpret_cast<uintptr_t>(code[q]) & 3u) == 0;
    uint64_t blocks = (cmax / 4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_dequantize, dim3((uint32_t)blocks, n_workers), dim3(256), 0, ctx->stream, make_tab<PtrTab>(code, n_workers),
                       make_tab<PtrTab>(scale, n_workers), ct, make_tab<MutPtrTab>(val, n_workers), vec_ok);
    SLIMDP_LAUNCHED(ctx, "k_dequantize");
    return SLIMDP_OK;
}

int slimdp_core_signature(slimdp_ctx* ctx, const uint32_t* core_idx, uint64_t k, uint64_t* sig)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (!sig || (k && !core_idx)) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_core_signature: NULL argument");
    if (k > ctx->n) return fail(ctx, SLIMDP_ERR_OUT_OF_RANGE, "slimdp_core_signature: k exceeds n");
    int rc = fill(ctx, reinterpret_cast<uint32_t*>(sig), 2, 0u);
    if (rc) return rc;
    if (k) {
        hipLaunchKernelGGL(k_signature, dim3(fill_grid(k)), dim3(256), 0, ctx->stream, core_idx, k,
                           reinterpret_cast<unsigned long long*>(sig));
        SLIMDP_LAUNCHED(ctx, "k_signature");
    }
    return SLIMDP_OK;
}

int slimdp_debug_philox(slimdp_ctx* ctx, uint64_t iteration, uint32_t worker, uint32_t i0, uint64_t count, uint32_t* out)
{
    if (!ctx) return SLIMDP_ERR_INVALID_ARG;
    if (count && !out) return fail(ctx, SLIMDP_ERR_INVALID_ARG, "slimdp_debug_philox: out is NULL");
    if (count == 0) return SLIMDP_OK;
    hipLaunchKernelGGL(k_debug_philox, dim3(fill_grid(count)), dim3(256), 0, ctx->stream, (uint32_t)ctx->seed,
                       (uint32_t)(ctx->seed >> 32), (uint32_t)iteration, (uint32_t)(iteration >> 32), worker, i0, count, out);
    SLIMDP_LAUNCHED(ctx, "k_debug_philox");
    return SLIMDP_OK;
}

}  // extern "C"
