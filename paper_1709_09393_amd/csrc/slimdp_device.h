// Device-side building blocks of libslimdp (gfx950, wave64).  Included only by slimdp.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "slimdp.h"

namespace slimdp {

constexpr uint32_t TILE = SLIMDP_TILE;            // parameters per tile
constexpr uint32_t TILE_WORDS = TILE / 32;        // bitmap words per tile
constexpr uint32_t SUB = 1024, SUB_WORDS = SUB / 32, SUBS = TILE / SUB;   // sub-tile: one wave's share of a tile
constexpr uint32_t NONE = 0xFFFFFFFFu;
constexpr int MAXW = SLIMDP_MAX_WORKERS;
constexpr int BLOCK = 256;                        // threads per block in the tile kernels
constexpr int EPT = TILE / BLOCK;                 // elements per thread per tile (16)

// Histogram storage per (batch, segment): level 0, level 1, level 2, and the second level-1 region of a core selection
// (the scoring pass counts into the first against a predicted bin, the selection's own pass into the second).
constexpr uint32_t H_L0 = 0, H_L1 = 8192, H_L2 = 12288, H_L1B = 12544, H_STRIDE = 16640;

// Core ranking key = raw bits of the score: 13 + 12 + 7 bits.
constexpr uint32_t CORE_SHIFT0 = 19, CORE_NB0 = 8192, CORE_SHIFT1 = 7, CORE_NB1 = 4096, CORE_NB2 = 128;

struct PtrTab { const void* p[MAXW]; };           // host pointer tables travel as kernel arguments
struct MutPtrTab { void* p[MAXW]; };

// Explorer request of one (batch, segment).  Words r <= sure_m1 (if has_gt) are taken unless in the core, words up to
// bound_m1 are candidates with key = bound_m1 - r.
struct SegState {
    uint32_t need0;     // number of elements to select
    uint32_t out_base;  // elements of the segments before this one
    uint32_t bound_m1, sure_m1, has_gt;
    uint32_t bits;      // candidate keys are below 2^bits
    uint32_t pad[2];
};
static_assert(sizeof(SegState) == 32, "SegState layout");

struct SegInit { uint32_t need, out_base, bound_m1, sure_m1, has_gt, bits; };
constexpr int INIT_CHUNK = 128;
struct SegInitChunk { SegInit s[INIT_CHUNK]; };

// ---------------------------------------------------------------------------------------
// wave / block primitives
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// Scans and reductions over a wave by data-parallel moves: shifts by 1, 2, 4, 8 lanes inside the rows of 16, then the last
// lane of a row, and of the lower half, to the rows above.  Six vector instructions, where six trips through the LDS
// crossbar take about 700 cycles, which the short kernels of a selection spend several times over in their chains.
// Every lane of the wave must be active.
template <class OP> __device__ __forceinline__ uint32_t wave_scan(uint32_t v, OP op)      // op(x, 0) == x
{
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true));       // row_shr:1
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true));
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false));      // row_bcast:15 into rows 1 and 3
    v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false));      // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) { return wave_scan(v, [](uint32_t a, uint32_t b) { return a + b; }); }
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return last_lane(wave_incl_scan(v)); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return last_lane(wave_scan(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; })); }

// Buffer addressing: a 128-bit descriptor in scalar registers (base, byte range, no stride)
// plus one 32-bit per-lane byte offset and a scalar offset.  Compared with flat 64-bit
// per-lane addresses this keeps the address arithmetic out of the vector registers, and
// accesses outside [0, bytes) are dropped by the hardware.  Callers pass 0 as the scalar
// offset and fold the wave's part into the lane offset: with a scalar-register offset the
// 16-byte forms were seen to store, now and then, a stale first dword on this target
// (caught by the several-tiles-per-block scoring test).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float4 buffer_load4(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, uint32_t wave_bytes)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, (int)wave_bytes, 0);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
// The same with a cache policy (the intrinsic's auxiliary operand must be a constant: 0 = default, 2 = non-temporal,
// for data that is touched once).
template <int AUX>
__device__ __forceinline__ float4 buffer_load4_aux(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, 0, AUX);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
template <int AUX>
__device__ __forceinline__ void buffer_store4_aux(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, float4 f)
{
    u32x4 v;
    v.x = __float_as_uint(f.x); v.y = __float_as_uint(f.y); v.z = __float_as_uint(f.z); v.w = __float_as_uint(f.w);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_bytes, 0, AUX);
}
__device__ __forceinline__ void buffer_store4(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, uint32_t wave_bytes, float4 f)
{
    u32x4 v;
    v.x = __float_as_uint(f.x); v.y = __float_as_uint(f.y); v.z = __float_as_uint(f.z); v.w = __float_as_uint(f.w);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_bytes, (int)wave_bytes, 0);
}

__device__ __forceinline__ void buffer_store1(__amdgpu_buffer_rsrc_t r, uint32_t lane_bytes, uint32_t v)
{
    __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)lane_bytes, 0, 0);
}

// OR over aligned groups of eight lanes, every lane of a group getting the result.  Three
// data-parallel-primitive moves inside a row of 16 lanes (swap neighbours, swap pairs, mirror
// each half row) instead of three trips through the LDS crossbar.
__device__ __forceinline__ uint32_t or_reduce8(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);      // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);      // quad_perm [2,3,0,1]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);     // row_half_mirror
    return v;
}

// Distances of four words above a bound, and whether they are below it: the borrow of the subtraction is shifted into acc
// by an addition with carry (the first word's ends up highest).  Eight instructions; from the comparisons the compiler
// makes masks, selects and ors, sixteen.  All four borrows are written before the first is read: a scalar that the
// vector unit wrote may be read by it two instructions later.  The compiler keeps that distance itself, but does not look
// into these blocks: where a scalar operand may come from a lane read just before (a spilled register), they begin by waiting.
struct Masks4 { uint64_t m0, m1, m2, m3; };
__device__ __forceinline__ Masks4 sub4_borrow(const uint32_t r[4], uint32_t bound, uint32_t d[4], uint32_t& acc)
{
    Masks4 m;
    asm("s_nop 1\n\t"
        "v_subrev_co_u32_e64 %0, %5, %9, %10\n\t"
        "v_subrev_co_u32_e64 %1, %6, %9, %11\n\t"
        "v_subrev_co_u32_e64 %2, %7, %9, %12\n\t"
        "v_subrev_co_u32_e64 %3, %8, %9, %13\n\t"
        "v_addc_co_u32_e64 %4, vcc, %4, %4, %5\n\t"
        "v_addc_co_u32_e64 %4, vcc, %4, %4, %6\n\t"
        "v_addc_co_u32_e64 %4, vcc, %4, %4, %7\n\t"
        "v_addc_co_u32_e64 %4, vcc, %4, %4, %8"
        : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "+&v"(acc), "=&s"(m.m0), "=&s"(m.m1), "=&s"(m.m2), "=&s"(m.m3)
        : "s"(bound), "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(r[3])
        : "vcc");
    return m;
}
// The component of x that belongs to the first of sub4_borrow's masks in which the lane is set (x.w if none is).
__device__ __forceinline__ float first_masked(const float4& x, const Masks4& m)
{
    float v;
    asm("s_nop 1\n\t"
        "v_cndmask_b32_e64 %0, %1, %2, %5\n\t"
        "v_cndmask_b32_e64 %0, %0, %3, %6\n\t"
        "v_cndmask_b32_e64 %0, %0, %4, %7"
        : "=&v"(v) : "v"(x.w), "v"(x.z), "v"(x.y), "v"(x.x), "s"(m.m2), "s"(m.m1), "s"(m.m0));
    return v;
}

// Four rounds of four flags a lane (bit 4 * round + i of v) to bitmap words: lanes 8j .. 8j+7 make word j of every round, and
// lane 8j + 2 * round (and the one beside it) gets it.  Nibbles are paired with the neighbouring lane's, the bytes then cross
// an 8-lane group in two exchanges (half-row mirror, lane pairs): ten instructions for four words, where a reduction
// for each of them took six.
__device__ __forceinline__ uint32_t transpose_spread(uint32_t v)             // one round a byte, in its low half
{
    const uint32_t lane = lane_id();
    v <<= 4u * (lane & 1u);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);       // quad_perm [1,0,3,2]
    // lanes 0..3 of a group keep rounds 0 and 1, lanes 4..7 rounds 2 and 3, of their pair and of the one mirrored (p and 3 - p)
    uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);      // row_half_mirror
    v = __builtin_amdgcn_perm(o, v, (lane & 4u) ? 0x03070206u : 0x05010400u);          // bytes: (lower pair, higher pair) of either round
    // of the two the lanes of pairs 0 and 2 keep the first, those of pairs 1 and 3 the second
    o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);        // quad_perm [2,3,0,1]
    // pairs in order: own (p, 3 - p) and the neighbour's
    const uint32_t sel = (lane & 2u) ? ((lane & 4u) ? 0x03070602u : 0x07030206u) : ((lane & 4u) ? 0x05010004u : 0x01050400u);
    return __builtin_amdgcn_perm(o, v, sel);
}

__device__ __forceinline__ uint32_t transpose_flags(uint32_t v)              // one round a nibble of the low half word
{
    v = (v | (v << 8)) & 0x00FF00FFu;
    return transpose_spread((v | (v << 4)) & 0x0F0F0F0Fu);
}

// Exclusive prefix sum over the block (NWAVES*64 threads, all must call).  wtot: NWAVES words
// of shared memory, free for reuse on return.
template <int NWAVES>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* wtot, uint32_t& total)
{
    const uint32_t lane = lane_id(), wid = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) wtot[wid] = incl;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
        const uint32_t t = wtot[w];
        if ((uint32_t)w < wid) base += t;
        tot += t;
    }
    __syncthreads();
    total = tot;
    return base + incl - v;
}

// Local element handled by (thread, slot j) of a tile.  Vector layout: four consecutive
// elements per thread and round (16-byte loads); scalar layout: one element per thread and round.
__device__ __forceinline__ uint32_t elem_vec(int j) { return (uint32_t)(j >> 2) * 1024u + threadIdx.x * 4u + (uint32_t)(j & 3); }
__device__ __forceinline__ uint32_t elem_scl(int j) { return (uint32_t)j * BLOCK + threadIdx.x; }

__device__ __forceinline__ uint32_t mask_below(uint32_t bit) { return (1u << bit) - 1u; }   // bit in 0..31

// Accesses to data that is touched once (streamed): NT != 0 marks them non-temporal, so that they do not
// push lines that will be used again out of the caches.  A non-temporal store must cover whole 128-byte lines
// per instruction (a partial one goes to memory as a read-modify-write).  Sixteen bytes from any address that a float
// may have: the hardware asks for no more than that of them, and the types say so to the compiler.
typedef float f32x4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4), aligned(4)));
template <int NT> __device__ __forceinline__ float4 ld4(const float* p)
{
    f32x4_t v;
    if (NT) v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p));
    else v = *reinterpret_cast<const f32x4_t*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
template <int NT> __device__ __forceinline__ uint4 ld4u(const uint32_t* p)
{
    u32x4_t v;
    if (NT) v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    else v = *reinterpret_cast<const u32x4_t*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <int NT> __device__ __forceinline__ void st4(float* p, float4 v)
{
    f32x4_t o; o.x = v.x; o.y = v.y; o.z = v.z; o.w = v.w;
    if (NT) __builtin_nontemporal_store(o, reinterpret_cast<f32x4_t*>(p));
    else *reinterpret_cast<f32x4_t*>(p) = o;
}
template <int NT, class Tp> __device__ __forceinline__ Tp ld1(const Tp* p)
{
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <int NT, class Tp> __device__ __forceinline__ void st1(Tp* p, Tp v)
{
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// ---------------------------------------------------------------------------------------
// Philox4x32 with 10 rounds (Salmon et al., SC'11): the explorer's random words.
// Counter (c0, c1, c2, c3), key (k0, k1).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        // three-input exclusive or in one instruction (truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The explorer's draw calls it for many workers with the same first word: word (c0, worker, it_lo, it_hi).  The worker enters
// at c1, and what the first three rounds do with the rest does not depend on it: of their six products per lane one is left
// to each worker (two more are the same for the whole wave).  What is left over from them, per lane and c0:
struct PhiloxCommon { uint32_t x, y, z, d; };
__device__ __forceinline__ PhiloxCommon philox_common(uint32_t c0, uint32_t it_lo, uint32_t it_hi, uint32_t k0, uint32_t k1)
{
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint32_t c2 = (uint32_t)(p0 >> 32) ^ (it_hi ^ k1);
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t c0b = (uint32_t)(p1 >> 32) ^ ((uint32_t)((uint64_t)0xCD9E8D57u * it_lo) ^ (k0 + 0x9E3779B9u));
    const uint64_t q = (uint64_t)0xD2511F53u * c0b;
    PhiloxCommon c;
    c.x = (uint32_t)p0 ^ (k1 + 0xBB67AE85u);
    c.y = (uint32_t)p1 ^ (k0 + 2u * 0x9E3779B9u);
    c.z = (uint32_t)(q >> 32) ^ (k1 + 2u * 0xBB67AE85u);
    c.d = (uint32_t)q;
    return c;
}
// The keys of the seven rounds that follow (key + round * Weyl constant).  A kernel that draws many words under one key
// computes them once and, made opaque to the compiler, keeps them in vector registers; left to itself the compiler holds
// them in scalar registers, runs out of those and reloads each with a lane read before every use.
struct PhiloxRoundKeys { uint32_t k0[7], k1[7]; };
template <bool HELD>
__device__ __forceinline__ PhiloxRoundKeys philox_round_keys(uint32_t k0, uint32_t k1)
{
    PhiloxRoundKeys rk;
#pragma unroll
    for (int r = 0; r < 7; ++r) {
        rk.k0[r] = k0 + (uint32_t)(r + 3) * 0x9E3779B9u;
        rk.k1[r] = k1 + (uint32_t)(r + 3) * 0xBB67AE85u;
        if (HELD) asm volatile("" : "+v"(rk.k0[r]), "+v"(rk.k1[r]));
    }
    return rk;
}
// The rest for one worker: v = the second round's product that only the worker decides.
__device__ __forceinline__ uint64_t philox_worker(uint32_t worker, uint32_t it_lo, uint32_t k0)
{
    return (uint64_t)0xD2511F53u * ((uint32_t)(((uint64_t)0xCD9E8D57u * it_lo) >> 32) ^ worker ^ k0);
}
__device__ __forceinline__ void philox_words(const PhiloxCommon& c, uint64_t v, const PhiloxRoundKeys& rk, uint32_t out[4])
{
    const uint64_t e = (uint64_t)0xCD9E8D57u * (c.x ^ (uint32_t)(v >> 32));
    uint32_t c0 = (uint32_t)(e >> 32) ^ c.y, c1 = (uint32_t)e, c2 = c.z ^ (uint32_t)v, c3 = c.d;
#pragma unroll
    for (int r = 0; r < 7; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, rk.k0[r], 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, rk.k1[r], 0x96);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Equation (1) with the rounding the interface promises: one fused multiply-add, canonical NaN.
__device__ __forceinline__ float significance(float w, float gsum, float c)
{
    float s = __builtin_fmaf(c, __builtin_fabsf(gsum), __builtin_fabsf(w));
    if (s != s) s = __uint_as_float(0x7FC00000u);
    return s;
}

}  // namespace slimdp
