// kernels.h -- gfx950 kernel of batched paged decode attention.
//
// One call = one launch of attn_kernel<G, kCheck, kAppend> on a persistent
// grid of W work groups (4 waves each); kCheck adds the optional input check
// (block ids against the pool, contexts against an explicit table row),
// kAppend the fused append of the current token's K/V.  Every work
// group
//   1. reads context_lens once and derives the partition of plan_policy.h on
//      its own (block sums, a prefix scan, the longest request for the tight
//      block-table stride; in every wave's registers for up to 512 requests,
//      by the group through LDS for more; 32-bit arithmetic unless the batch
//      is too large for it), so no planner kernel runs before it;
//   2. walks its contiguous range of (request b, kv-head g, block) units
//      (ranges of equal cost, a pair's cost being its blocks plus a fixed
//      start-up charge; for a small batch one part of one pair; with many
//      short pairs every wave takes whole pairs of its own) segment by
//      segment.  In a segment the four waves
//      take the blocks of one (b, g) pair round-robin; per 16-token block a
//      wave gathers the paged K/V rows with 128-bit loads (two blocks in
//      flight per wave), computes the G q-heads' scores as S^T = K Q^T with
//      four 16x16x32 fp16 MFMAs (q-heads padded to 16 columns), runs an
//      online softmax (running max and sum in base 2, log2(e) folded into
//      the scale), and accumulates O^T += V^T P^T in fp32 with sixteen
//      16x16x16 fp16 MFMAs -- the weights P as two fp16 parts, 22 bits --
//      V^T being assembled in registers with byte permutes.
//      Each wave's K/V pipeline runs on across segments: between two long
//      segments the last steps of one already load the next one's first
//      blocks, and the next segment's Q operand is loaded one segment ahead;
//   3. merges the waves' states in LDS and either writes the fp16 output rows
//      (the segment is the whole pair) or stores an fp32 partial
//      (accumulator, max, sum) and bumps the pair's arrival counter; the last
//      work group to arrive combines the pair's partials and writes the rows;
//   4. writes the zero rows of requests with no context (their share of them).
//
// The attention is the standard softmax attention that APEX runs for its
// GPU-resident decode requests over their paged KV (Sec. 3.1, Sec. 3.3,
// Sec. 4.1); splitting a pair's tokens is exact up to rounding: with per-range
// maxima m_s, sums l_s and unnormalised accumulators a_s,
//   out = sum_s 2^(m_s - M) a_s / sum_s 2^(m_s - M) l_s,   M = max_s m_s.
#pragma once

#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include <type_traits>

#include "plan_policy.h"

namespace apex {

typedef _Float16 f16;
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kAttnThreads = 256;
constexpr int kWaves = kAttnThreads / 64;
constexpr int kCachedLens = 2048;   // context_lens kept in LDS up to this batch size
constexpr int kStageFloats = 2048;  // LDS of one wave: its merged state, or the partials it combines
// Partials that the emitting threads combine on their own, all in flight at
// once; more are shared by the four waves, which end in another LDS merge.  What
// a thread takes per partial grows with the group: one element (G = 1 and 2),
// two (G = 4), four (G = 8).  G = 1, threads against waves: 7 and 8 partials 8.35
// and 7.96 us against 8.71 and 8.38 (one request of 700 tokens, 32 and 16 heads),
// 15 and 16 partials 11.10 and 25.94 against 11.39 and 26.24 (3000 and 16000
// tokens, 16 heads); with the line at 4 the fused call of one request on 32 heads
// was slower than before the waves shared the combine (2100 tokens: 12.2 us then,
// 12.7 with the line at 4, 12.3 at 16).  Four requests of 1024 tokens, G = 4, 4-5
// partials a pair: 9.5 us with the line at 4, 9.8 at 8.
template <int G>
constexpr int kFewPartials = G == 1 ? 16 : 4;

struct AttnParams {
    const f16* q;          // [B][Hq][D]
    const f16* k;          // [NB][Hkv][BS][D]
    const f16* v;
    f16* out;              // [B][Hq][D]
    float* lse;            // optional [B][Hq], natural log
    int32_t* counters;     // [B][Hkv] arrival counters, zero between calls
    float* pacc;           // [2W][G][D] partial accumulators
    float* pml;            // [2W][G][2] partial (max in log2 units, sum)
    int64_t bt_stride;     // 0 = tight: ceil(max L / BS)
    float scale_log2;      // scale * log2(e)
    int B;
    int Hq;
    int Hkv;
    int min_units;         // minimum units per active worker
    int seg_cost;          // cost positions charged per pair (plan_policy.h), 0 = equal units
    int cus;               // compute units for the one-group-per-CU rule (0 = off)
    int launched;          // work groups launched (the grid size)
    int64_t num_blocks;    // physical blocks in the caches (input check only)
    unsigned* error_word;  // input-check error bits (input check only)
    // Fused append (optional): the current token's K/V rows, [B][Hkv][D] with
    // new_stride elements between tokens.  The caches then hold the first
    // L - 1 tokens of a request; the current one is attended from these rows
    // and written to its slot (position L - 1) by the work group that emits
    // the pair.
    const f16* k_new;
    const f16* v_new;
    int64_t new_stride;
    f16* k_store;          // the caches, written by the fused append
    f16* v_store;
#ifdef APEX_TRACE_WORK_GROUPS
    uint64_t* trace;       // [trace_groups][kTraceWords] work-group timeline, or null
    int64_t trace_groups;
#endif
};

#ifdef APEX_TRACE_WORK_GROUPS
// Work-group timeline of the diagnostic build: per work group, in ticks of
// the 100 MHz real-time clock, its first instruction, the end of its
// partition prologue, the completion of wave 0's first tiles and its end;
// then its segments, the split ones among them, and its units.
constexpr int kTraceWords = 8;
__device__ inline uint64_t trace_clock() { return __builtin_amdgcn_s_memrealtime(); }
// the work group's row, kept in LDS while it runs (no register stays live
// across the block loop for it)
__shared__ uint64_t s_trace[kTraceWords];
#endif

// Input-check error bits (apex_decode.h: APEX_DEVICE_ERR_*).
constexpr unsigned kErrBlockId = 1u;      // a block id outside [0, num_blocks)
constexpr unsigned kErrTableRow = 2u;     // a context past its block-table row

__device__ inline void report_error(const AttnParams& p, unsigned bits)
{
    __hip_atomic_fetch_or(p.error_word, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Reinterpret one 32-bit word as two fp16 values.  Taken by value on purpose:
// clang's __builtin_bit_cast applied directly to a vector element expression
// (e.g. v.y) reads element 0 instead (seen in the gfx950 assembly).
__device__ inline f16x2 as_h2(unsigned int u)
{
    return __builtin_bit_cast(f16x2, u);
}

__device__ inline float wave_shfl_xor(float x, int mask)
{
    return __shfl_xor(x, mask, 64);
}

__device__ inline float exp2_fast(float x)
{
    return __builtin_amdgcn_exp2f(x);
}

// Inclusive prefix sum / max over the 64 lanes of a wave with DPP (row
// shifts within each 16-lane row, then the row broadcasts of lanes 15 and 31
// into the rows above): a few VALU cycles per step, where a cross-lane
// shuffle goes through the LDS crossbar.  Lane 63 ends with the wave's total.
__device__ inline int wave_incl_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2, 3
    return x;
}

// As wave_incl_sum for fp32 values (lane 63 ends with the wave's sum).
__device__ inline float wave_incl_sum_f32(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x111, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x112, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x114, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x118, 0xf, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x142, 0xa, 0xf, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x143, 0xc, 0xf, false));
    return x;
}

// As wave_incl_sum with max, for x >= 0.
__device__ inline int wave_incl_max(int x)
{
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
    return x;
}

// The value of one lane (the same lane index in every lane) as a scalar.
__device__ inline int lane_value(int x, int lane)
{
    return __builtin_amdgcn_readlane(x, lane);
}

// Max / sum of the values a lane's column holds in the four 16-lane rows of
// its wave (the rows' lanes l, l + 16, l + 32, l + 48), with the gfx950 row
// swaps: each swap returns the lane's own value and its partner's (rows
// paired as 0-1, 2-3, then halves as 0-32), so the pair's max / sum is the
// step of a xor-16 / xor-32 butterfly without the LDS crossbar of a shuffle.
__device__ inline float rows_max4(float x)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ inline float rows_sum4(float x)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline int uniform(int x)
{
    return __builtin_amdgcn_readfirstlane(x);
}

__device__ inline int64_t uniform64(int64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <typename T>
__device__ inline T* uniform_ptr(T* p)
{
    return (T*)uniform64((int64_t)p);
}

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Two fp16 halves from two words: the low (sel = kLoHalves) or high
// (sel = kHiHalves) half of a in the low half of the result, the same half of
// b in the high half.
constexpr unsigned kLoHalves = 0x05040100u;
constexpr unsigned kHiHalves = 0x07060302u;
__device__ inline unsigned pack_halves(unsigned a, unsigned b, unsigned sel)
{
    return __builtin_amdgcn_perm(b, a, sel);
}

// One (block, kv-head) slab of K or V: 16 rows of 128 fp16 values.
constexpr int kSlabBytes = kBlockSize * kHeadDim * 2;
// Buffer-resource word 3 for raw (untyped) buffer access on gfx9-family GPUs.
constexpr int kRawBufferWord3 = 0x00020000;
// Cache policy of the K/V loads: non-temporal (bit 1) -- each row is read
// exactly once per call, so it should not displace reusable lines.
constexpr int kStreamingLoad = 2;
// Cache policy of device-coherent accesses (sc1, the bit of relaxed atomics at
// agent scope): work groups on different XCDs, each with its own L2, see each
// other's values without any cache flush.
constexpr int kCoherent = 16;
// s_waitcnt operand: LDS (and scalar) accesses complete, others left in flight
constexpr int kWaitLds = 0xc07f;

// Operand layouts of one slab (lane = 16 q + c, q = lane / 16, c = lane % 16):
//   K: word i of lane (c, q) = token c, dims [32i + 8q, +8)   (A of S^T = K Q^T)
//   V: word e of lane (c, q) = token 4q + e, dims [8c, 8c + 8)
__device__ inline int k_lane_offset(int lane) { return (lane & 15) * 256 + (lane >> 4) * 16; }
__device__ inline int v_lane_offset(int lane) { return (lane >> 4) * 1024 + (lane & 15) * 16; }

// Loads a slab with buffer instructions: the slab base lives in scalar
// registers (a fresh resource per block), the lane offset in a VGPR that
// never changes.  The resource's extent bounds every access; an extent of 0
// turns the four loads into no-ops that return zeros, which lets a pipeline
// issue the same loads every step.
__device__ inline void load_slab(u32x4 (&w)[4], const f16* slab, int bytes, int lane_off,
                                 int stride)
{
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(slab), (short)0, bytes, kRawBufferWord3);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        w[i] = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + stride * i, 0, kStreamingLoad);
}

// This wave's share of one segment (blocks lo..hi-1 of pair (b, g)): its
// blocks are first, first + 4, ... < hi, n of them.  A wave with no block in
// the segment, and the "next segment" after a work group's last one, have
// n = 0.
struct WaveSeg {
    const int32_t* bt;   // block-table entry of the wave's first block
    const f16* kpair;    // K / V of kv-head g in block 0 (a block id adds id * step)
    const f16* vpair;
    const f16* qrow;     // this lane's Q^T operand row (q-head g*G + lane % 16, if < G)
    int first;           // the wave's first block (index into the pair's blocks)
    int n;
    int b, g;            // the pair
};

template <int G, int kStep>
__device__ inline WaveSeg wave_seg(const AttnParams& p, const int32_t* bt_row, int b, int g, int lo,
                                   int hi, int wave, int lane)
{
    WaveSeg s;
    s.first = uniform(kStep == 1 ? lo : lo + wave);
    s.n = s.first < hi ? (hi - s.first + kStep - 1) / kStep : 0;
    s.bt = bt_row + s.first;
    const size_t head_off = (size_t)uniform(g) * (kBlockSize * kHeadDim);
    s.kpair = uniform_ptr(p.k + head_off);
    s.vpair = uniform_ptr(p.v + head_off);
    const int col = lane & 15;
    s.qrow = p.q + ((size_t)b * p.Hq + (size_t)g * G + (col < G ? col : 0)) * kHeadDim + 8 * (lane >> 4);
    s.b = b;
    s.g = g;
    return s;
}

// Q^T operand: lane (h, q) holds head h's dims [32i + 8q, +8) for MFMA i;
// columns past the group are zero.
template <int G>
__device__ inline void load_q(f16x8 (&qop)[4], const WaveSeg& s, int lane)
{
    if ((lane & 15) < G) {
#pragma unroll
        for (int i = 0; i < 4; ++i) qop[i] = *(const f16x8*)(s.qrow + 32 * i);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) qop[i] = f16x8{0, 0, 0, 0, 0, 0, 0, 0};
    }
}

// The K/V pipeline of one wave, carried from segment to segment.  Tile t
// (t = 0, 1) holds the wave's blocks of parity t.  When a segment and the next
// both span at least kPrefetchBlocks blocks (every wave has at least four of
// each), a segment's last two steps refill the tiles with the next segment's
// blocks 0 and 1: they are in flight while the work group merges and emits
// the segment, and the next segment starts with its first loads issued long
// before.  Otherwise the next segment loads its first blocks itself.
constexpr int kPrefetchBlocks = 16;

struct WaveTiles {
    u32x4 kt0[4], vt0[4], kt1[4], vt1[4];
    int cur0, cur1;      // ids of the blocks in the tiles
    int nid0, nid1;      // ids of the blocks that refill the tiles next
    bool prefetched;     // the tiles hold the segment's blocks 0 and 1
    f16x8 qop[4];        // Q^T of the current segment
    f16x8 qnext[4];      // Q^T of the next segment (loaded one segment ahead)
};

// A wave's attention state over its blocks: lane (h = lane % 16, q = lane / 16)
// has head h's running max m (log2 units) and sum l of the weights of all of
// the wave's tokens, and P.V at dims 32q + 8i + t.
struct WaveState {
    float m, l;
    f32x4 acc[8];
};

// Fused append.  Scaled logits (log2 units) of the current token for the G
// q-heads of pair (b, g), computed by one wave (lane l takes dims 2l, 2l + 1):
// the loads, then (once they are complete) the sums.
template <int G>
struct NewTokenRows {
    f16x2 k2;
    f16x2 q2[G];
};

template <int G>
__device__ inline void load_new_token_rows(const AttnParams& p, int b, int g, int lane, NewTokenRows<G>& r)
{
    r.k2 = *(const f16x2*)(p.k_new + (size_t)b * p.new_stride + (size_t)g * kHeadDim + 2 * lane);
#pragma unroll
    for (int h = 0; h < G; ++h)
        r.q2[h] = *(const f16x2*)(p.q + ((size_t)b * p.Hq + (size_t)g * G + h) * kHeadDim + 2 * lane);
}

template <int G>
__device__ inline void new_token_logits(const AttnParams& p, const NewTokenRows<G>& r, int lane, float* s_new,
                                        int first, int stride)
{
#pragma unroll
    for (int h = 0; h < G; ++h) {
        if (h % stride != first) continue;
        const float x = wave_incl_sum_f32(fmaf((float)r.q2[h][0], (float)r.k2[0], (float)r.q2[h][1] * (float)r.k2[1]));
        if (lane == 63) s_new[h] = x * p.scale_log2;
    }
}

// Elements of a (request, kv-head) pair's G output rows that one thread of the
// merge and emit owns: consecutive dims of one head, so that the whole work
// group covers the rows in one pass (G = 1: its first half).  The merge is
// bound by its instructions: one pass with vector LDS reads takes 0.25-0.3 us
// where G / 2 passes over single elements took 0.65 (G = 4) and 0.95 (G = 8).
template <int G>
constexpr int kEmitElems = G >= 2 ? G * kHeadDim / kAttnThreads : 1;

template <typename T, int N>
struct vec_of {
    typedef T type __attribute__((ext_vector_type(N)));
};

// The current token's K and V elements [dim, dim + N) of kv-head g of request
// b and the id of the block that holds its slot (position Lc - 1, Lc = the
// full length), loaded ahead of the emit that needs them.  With the input
// check a position past an explicit table row (a context cut to its row,
// already reported) has no slot: the row's last slot holds a cached token.
// The slot's table entry is the same for the whole work group, so it is read
// through the constant address space (the scalar path); `safe` is any
// readable entry, read instead when there is no slot.  (dim is a multiple of
// N <= 4 and every row starts at a multiple of 8 elements: aligned vectors.)
template <int N>
struct NewTokenElems {
    typename vec_of<f16, N>::type kn, vn;
    int id;
    bool in_row;
};

template <bool kCheck, int N>
__device__ inline NewTokenElems<N> load_new_token_elems(const AttnParams& p, const int32_t* bt_row,
                                                        const int32_t* safe, int b, int g, int Lc, int dim)
{
    typedef typename vec_of<f16, N>::type f16xN;
    NewTokenElems<N> e;
    const size_t src = (size_t)b * p.new_stride + (size_t)g * kHeadDim + dim;
    e.kn = *(const f16xN*)(p.k_new + src);
    e.vn = *(const f16xN*)(p.v_new + src);
    e.in_row = !(kCheck && p.bt_stride > 0 && (int64_t)((Lc - 1) / kBlockSize) >= p.bt_stride);
    const int32_t* a = e.in_row ? bt_row + (Lc - 1) / kBlockSize : safe;
    e.id = *(const __attribute__((address_space(4))) int32_t*)a;
    return e;
}

// Issues the loads of a segment's blocks 0 and 1 (tile 0 first) and of the ids
// that follow them, for a segment that the pipeline does not run on into.
template <bool kCheck, int kStep>
__device__ inline void load_first_tiles(const AttnParams& p, const WaveSeg& cs, const int32_t* safe, WaveTiles& st,
                                        int lane)
{
    const int n = cs.n;
    const uint32_t step = (uint32_t)((size_t)p.Hkv * kBlockSize * kHeadDim);
    const int koff = k_lane_offset(lane), voff = v_lane_offset(lane);
    auto id_at = [&](int pos) -> int {
        const int32_t* a = pos < n ? cs.bt + kStep * pos : safe;
        return *(const __attribute__((address_space(4))) int32_t*)a;
    };
    auto id_ok = [&](int id) -> bool { return !kCheck || (id >= 0 && (int64_t)id < p.num_blocks); };
    st.cur0 = id_at(0);
    st.cur1 = id_at(1);
    st.nid0 = id_at(2);
    st.nid1 = id_at(3);
    const int nb0 = n > 0 && id_ok(st.cur0) ? kSlabBytes : 0;
    const int nb1 = n > 1 && id_ok(st.cur1) ? kSlabBytes : 0;
    load_slab(st.kt0, cs.kpair + (uint64_t)(uint32_t)st.cur0 * step, nb0, koff, 64);
    load_slab(st.vt0, cs.vpair + (uint64_t)(uint32_t)st.cur0 * step, nb0, voff, 256);
    load_slab(st.kt1, cs.kpair + (uint64_t)(uint32_t)st.cur1 * step, nb1, koff, 64);
    load_slab(st.vt1, cs.vpair + (uint64_t)(uint32_t)st.cur1 * step, nb1, voff, 256);
}

// Per-wave attention over its blocks of segment cs; ns is the work group's
// next segment (n = 0 if none), `safe` any readable block-table entry, pf_next
// whether the tiles continue into ns, cur_row the block-table row of cs's
// request (with the fused append, ne receives this thread's elements of the
// current token for the emit).  Lane
// (h = lane % 16, q = lane / 16) keeps m (running max of head h, log2 units,
// equal on the four lanes of h), l (sum of the weights of its tokens) and
// acc[t][i] (running P.V of head h at dim 32q + 8i + t).  The wave takes every
// kStep-th block: kWaves when the four waves share a segment, 1 when it has one
// of its own.  On return its state is in ws and the tiles hold (in flight) the
// next segment's first blocks.
template <int G, bool kCheck, bool kAppend, int kStep>
__device__ inline void wave_attend(const AttnParams& p, const WaveSeg& cs, const WaveSeg& ns,
                                   const int32_t* safe, bool pf_next, int L, WaveTiles& st, int wave,
                                   int lane, WaveState& ws,
                                   float* s_new, const int32_t* cur_row, NewTokenElems<kEmitElems<G>>& ne)
{
    constexpr int D = kHeadDim;
    constexpr int BS = kBlockSize;
    const int q = lane >> 4;
    const int n = cs.n;

    const uint32_t step = (uint32_t)((size_t)p.Hkv * BS * D);
    const int koff = k_lane_offset(lane);
    const int voff = v_lane_offset(lane);
    // with the input check, a block id outside the pool is never read: its
    // loads get a zero extent like those past the end
    auto id_ok = [&](int id) -> bool { return !kCheck || (id >= 0 && (int64_t)id < p.num_blocks); };
    // block id at position pos of this (here) or the next segment's wave
    // list; `ok` false reads the safe entry (the id is then unused).  The
    // table is read-only during the call: reading it through the constant
    // address space keeps the load on the scalar path.
    auto id_at = [&](bool here, int pos, bool ok) -> int {
        const int32_t* a = ok ? (here ? cs.bt : ns.bt) + kStep * pos : safe;
        return *(const __attribute__((address_space(4))) int32_t*)a;
    };
    // the tiles continue into the next segment (the work group's choice:
    // both segments are long)
    const bool pf = kStep == kWaves && pf_next;

    // Everything loaded before the loop (the tiles, mostly issued during the
    // previous segment's last steps, and this segment's Q^T, issued one
    // segment ahead) is complete from here on, so the loop's own waits are
    // those of its two-deep pipeline alone.
    __builtin_amdgcn_s_waitcnt(0);
#ifdef APEX_TRACE_WORK_GROUPS
    if (wave == 0 && lane == 0 && s_trace[2] == 0) s_trace[2] = trace_clock();
#endif
#pragma unroll
    for (int i = 0; i < 4; ++i) st.qop[i] = st.qnext[i];
    if (kStep == kWaves) load_q<G>(st.qnext, ns, lane);   // used by the next segment only
    // With the fused append: the rows of the current token's logits for this
    // pair (wave 0 sums them after the loop; the merge reads them) and this
    // thread's elements for the emit.  Issued after the wait above, they
    // complete during the block loop instead of adding a round trip to the
    // segment's entry and to its emit.  Every wave issues the row loads, a
    // few hundred bytes: with a branch on the wave around them the compiler's
    // wait placement could not tell that every path passes the loop's waits.
    NewTokenRows<G> nt;
    if (kAppend) {
        load_new_token_rows<G>(p, cs.b, cs.g, lane, nt);
        if (kStep == kWaves)
            ne = load_new_token_elems<kCheck, kEmitElems<G>>(p, cur_row, safe, cs.b, cs.g, L + 1,
                                                             (wave * 64 + lane) * kEmitElems<G> % D);
    }

    float m = -INFINITY, l = 0.f;
    f32x4 (&acc)[8] = ws.acc;
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // One block: consume (kt, vt) holding block k (id cur) of tile t = k % 2,
    // refill them with the tile's next element (id nid: this segment's block
    // k + 2, else the next segment's block t), look up the id of the element
    // after that.  Slab addresses are formed in scalar registers only, block
    // ids arrive through the scalar path ahead of use, and every step issues
    // eight loads (zero-extent when there is no element) so the compiler can
    // wait for exactly the oldest slab.
    auto block_step = [&](u32x4 (&kt)[4], u32x4 (&vt)[4], int k, int& cur, int& nid) {
        const int t = k & 1;
        // refill: this segment's block k + 2, else the next segment's block
        // t (with pf), else nothing
        const bool r_here = k + 2 < n;
        const bool r_ok = r_here || pf;
        // the id of the tile's element after that: block k + 4 here, else the
        // next segment's block t or t + 2
        const bool l_here = k + 4 < n;
        const int l_pos = l_here ? k + 4 : (r_here ? t : t + 2);
        const int id_next = id_at(l_here, l_pos, l_here || pf);
        const int id2 = nid;
        const f16* kbase = r_here ? cs.kpair : ns.kpair;
        const f16* vbase = r_here ? cs.vpair : ns.vpair;
        const int nbytes = r_ok && id_ok(id2) ? kSlabBytes : 0;
        const int tok0 = (cs.first + kStep * k) * BS;
        const int cur_id = cur;
        cur = id2;
        nid = id_next;
        if (kCheck && !id_ok(cur_id)) {
            // skip the block (its tokens take no part), keep the pipeline going
            if (lane == 0) report_error(p, kErrBlockId);
            load_slab(kt, kbase + (uint64_t)(uint32_t)id2 * step, nbytes, koff, 64);
            load_slab(vt, vbase + (uint64_t)(uint32_t)id2 * step, nbytes, voff, 256);
            return;
        }
        // S^T = K Q^T: lane (h, q) gets the scores of tokens 4q..4q+3 of head h
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, kt[i]), st.qop[i], s, 0, 0, 0);
        // K is consumed: refill it (in place: the barrier keeps the scheduler
        // from issuing the loads above the products that read the tile)
        __builtin_amdgcn_sched_barrier(0);
        load_slab(kt, kbase + (uint64_t)(uint32_t)id2 * step, nbytes, koff, 64);

        float sv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[i] = s[i] * p.scale_log2;
        const bool tail = tok0 > L - BS;   // the pair's last, partial block (no overflow at L near 2^31)
        if (tail) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (tok0 + 4 * q + i >= L) sv[i] = -INFINITY;
        }
        const float bm = rows_max4(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])));
        const float mnew = fmaxf(m, bm);   // finite: the block holds a valid token
        const float alpha = exp2_fast(m - mnew);
        f32x4 pw;
#pragma unroll
        for (int i = 0; i < 4; ++i) pw[i] = exp2_fast(sv[i] - mnew);
        // the weights as two fp16 MFMA operands: ph = pw rounded to fp16 and
        // pl = the rest rounded to fp16, together 22 significant bits (the
        // rest pw - ph is exact in fp32); the normaliser sums the same parts
        const f16x4 ph = __builtin_convertvector(pw, f16x4);
        const f32x4 ph32 = __builtin_convertvector(ph, f32x4);
        const f16x4 pl = __builtin_convertvector(pw - ph32, f16x4);
        const f32x4 pq = ph32 + __builtin_convertvector(pl, f32x4);
        l = l * alpha + ((pq[0] + pq[1]) + (pq[2] + pq[3]));
        m = mnew;

        // V^T operands in registers: tile t row c is dim 8c + t, its k index
        // is token 4q + e; rows of masked tokens are zeroed (they may hold NaN)
        unsigned a[8][2];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const unsigned sel = (t & 1) ? kHiHalves : kLoHalves;
            const int w = t >> 1;
            a[t][0] = pack_halves(vt[0][w], vt[1][w], sel);
            a[t][1] = pack_halves(vt[2][w], vt[3][w], sel);
        }
        // V is consumed: refill it (in place)
        __builtin_amdgcn_sched_barrier(0);
        load_slab(vt, vbase + (uint64_t)(uint32_t)id2 * step, nbytes, voff, 256);
        if (tail) {
            const bool ok0 = tok0 + 4 * q + 0 < L, ok1 = tok0 + 4 * q + 1 < L;
            const bool ok2 = tok0 + 4 * q + 2 < L, ok3 = tok0 + 4 * q + 3 < L;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                a[t][0] = (ok0 ? a[t][0] & 0x0000ffffu : 0u) | (ok1 ? a[t][0] & 0xffff0000u : 0u);
                a[t][1] = (ok2 ? a[t][1] & 0x0000ffffu : 0u) | (ok3 ? a[t][1] & 0xffff0000u : 0u);
            }
        }
        if (alpha != 1.f) {
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] *= alpha;
        }
        // O^T += V^T P^T, eight 16-dim tiles, the high parts of P, then the
        // low parts (independent accumulators between the two passes)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const u32x2 av = {a[t][0], a[t][1]};
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, av), ph, acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const u32x2 av = {a[t][0], a[t][1]};
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, av), pl, acc[t], 0, 0, 0);
        }
    };

    // pairs of blocks, then an odd last block on tile 0 (a loop with a single
    // exit keeps both tiles in the same registers from one segment to the next)
    int k = 0;
    for (; k + 1 < n; k += 2) {
        block_step(st.kt0, st.vt0, k, st.cur0, st.nid0);
        block_step(st.kt1, st.vt1, k + 1, st.cur1, st.nid1);
    }
    if (k < n) block_step(st.kt0, st.vt0, k, st.cur0, st.nid0);
    st.prefetched = pf;
    // (the waves that share a segment share the heads: a head's sum is a chain of
    // cross-lane adds, and with all G on one wave the merge waited for them:
    // 8 requests of 2000-4000 tokens, G = 8, 12.4 -> 12.0 us; one of 2100, G = 4,
    // 10.15 -> 9.95)
    if (kAppend) new_token_logits<G>(p, nt, lane, s_new, kStep == 1 ? 0 : uniform(wave), kStep);
    ws.m = m;
    ws.l = rows_sum4(l);   // over the four token groups
}

// A wave's state of a segment, to be merged with the other waves'.
template <int G>
__device__ inline void store_wave_state(const WaveState& ws, int wave, int lane, float (*s_acc)[kStageFloats],
                                        float (*s_m)[G], float (*s_l)[G])
{
    const int col = lane & 15, q = lane >> 4;
    if (col < G) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float* dst = &s_acc[wave][col * kHeadDim + 32 * q + 8 * i];
            *(f32x4*)dst = f32x4{ws.acc[0][i], ws.acc[1][i], ws.acc[2][i], ws.acc[3][i]};
            *(f32x4*)(dst + 4) = f32x4{ws.acc[4][i], ws.acc[5][i], ws.acc[6][i], ws.acc[7][i]};
        }
        if (q == 0) {
            s_m[wave][col] = ws.m;
            s_l[wave][col] = ws.l;
        }
    }
}

// A whole pair's rows from one wave's state (lane (h, q): head h, dims
// 32q + 8i + t), with the fused append the current token's fold and store.
template <int G, bool kCheck, bool kAppend>
__device__ inline void emit_wave(const AttnParams& p, WaveState& ws, int b, int g, int Lc, int lane,
                                 const float* s_new, const int32_t* bt_row, const int32_t* safe)
{
    const int col = lane & 15, q = lane >> 4;
    float M = ws.m, den = ws.l;
    if (kAppend) {
        const size_t src = (size_t)b * p.new_stride + (size_t)g * kHeadDim;
        f16x8 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const f16x8*)(p.v_new + src + 32 * q + 8 * i);
        // lane 63 has just written the logits that all lanes read.  Without the
        // fence a lane's own view allows the read first: for G = 1, where both
        // are one address, the compiler read the previous pair's logit in the
        // lanes that do not write
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const float sn = s_new[col < G ? col : 0];
        const float M2 = fmaxf(M, sn);
        const float f = M == -INFINITY ? 0.f : exp2_fast(M - M2);
        const float wgt = exp2_fast(sn - M2);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < 8; ++t) ws.acc[t][i] = fmaf(wgt, (float)v[i][t], ws.acc[t][i] * f);
        den = fmaf(den, f, wgt);
        M = M2;
        // lanes 0-15 store the K row, lanes 16-31 the V row
        if (lane < 32) {
            const NewTokenElems<8> e = load_new_token_elems<kCheck, 8>(p, bt_row, safe, b, g, Lc, 8 * col);
            if (e.in_row && !(kCheck && !(e.id >= 0 && (int64_t)e.id < p.num_blocks))) {
                const size_t dst =
                    (((size_t)(uint32_t)e.id * p.Hkv + g) * kBlockSize + (Lc - 1) % kBlockSize) * kHeadDim + 8 * col;
                *(f16x8*)&(q == 0 ? p.k_store : p.v_store)[dst] = q == 0 ? e.kn : e.vn;
            } else if (kCheck && e.in_row && lane == 0) {
                report_error(p, kErrBlockId);
            }
        }
    }
    if (col < G) {
        const int head = g * G + col;
        f16* row = p.out + ((size_t)b * p.Hq + head) * kHeadDim + 32 * q;
        // one reciprocal per head; a quotient with one correction step is
        // within half an ulp and a rounding of the division's.  An infinite
        // numerator (an infinite V value) has no remainder (inf - inf): the
        // maximum turns that NaN into a number and the quotient stays infinite.
        const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f16x8 o;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float a = ws.acc[t][i], y = a * inv;
                const float z = fmaf(fmaxf(fmaf(-y, den, a), -FLT_MAX), inv, y);
                o[t] = (f16)(den > 0.f ? z : 0.f);
            }
            *(f16x8*)(row + 8 * i) = o;
        }
        if (p.lse && q == 0)
            p.lse[(size_t)b * p.Hq + head] = den > 0.f ? (M + __log2f(den)) * 0.69314718055994531f : -INFINITY;
    }
}

// N consecutive dims of one head's merged state: running max M (log2 units;
// -inf when empty), numerators and denominator relative to it.
template <int N>
struct RowState {
    float M, den;
    typename vec_of<float, N>::type num;
};

template <int N>
__device__ inline void write_row(const AttnParams& p, int b, int head, int dim, const RowState<N>& r)
{
    typename vec_of<f16, N>::type o;
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = (f16)(r.den > 0.f ? r.num[i] / r.den : 0.f);
    *(typename vec_of<f16, N>::type*)&p.out[((size_t)b * p.Hq + head) * kHeadDim + dim] = o;
    if (p.lse && dim == 0)
        p.lse[(size_t)b * p.Hq + head] =
            r.den > 0.f ? (r.M + __log2f(r.den)) * 0.69314718055994531f : -INFINITY;
}

// Folds the current token (logit sn in log2 units, values vn) into a merged
// state with its fp32 weight.
template <int N>
__device__ inline void fold_new_token(float sn, typename vec_of<f16, N>::type vn, RowState<N>& r)
{
    const float M2 = fmaxf(r.M, sn);
    const float f = r.M == -INFINITY ? 0.f : exp2_fast(r.M - M2);
    const float wgt = exp2_fast(sn - M2);
#pragma unroll
    for (int i = 0; i < N; ++i) r.num[i] = fmaf(wgt, (float)vn[i], r.num[i] * f);
    r.den = fmaf(r.den, f, wgt);
    r.M = M2;
}

// Writes those elements to the slot (with the input check, a block id outside
// the pool is reported and not written).
template <bool kCheck, int N>
__device__ inline void store_new_token(const AttnParams& p, const NewTokenElems<N>& e, int g, int Lc, int dim)
{
    if (!e.in_row) return;
    if (kCheck && !(e.id >= 0 && (int64_t)e.id < p.num_blocks)) {
        if (dim == 0) report_error(p, kErrBlockId);
        return;
    }
    const size_t dst = (((size_t)(uint32_t)e.id * p.Hkv + g) * kBlockSize + (Lc - 1) % kBlockSize) * kHeadDim + dim;
    *(typename vec_of<f16, N>::type*)&p.k_store[dst] = e.kn;
    *(typename vec_of<f16, N>::type*)&p.v_store[dst] = e.vn;
}

// The four waves' states of head h (s_acc, s_m, s_l) at dims [dim, dim + N),
// merged.
template <int G, int N>
__device__ inline RowState<N> merge_waves(const float (*s_acc)[kStageFloats], const float (*s_m)[G],
                                          const float (*s_l)[G], int h, int dim)
{
    typedef typename vec_of<float, N>::type f32xN;
    RowState<N> r;
    r.M = s_m[0][h];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) r.M = fmaxf(r.M, s_m[q][h]);
    const float Ms = r.M == -INFINITY ? 0.f : r.M;
    r.den = 0.f;
    r.num = 0.f;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
        const float f = exp2_fast(s_m[q][h] - Ms);
        const f32xN a = *(const f32xN*)&s_acc[q][h * kHeadDim + dim];
        r.den = fmaf(f, s_l[q][h], r.den);
#pragma unroll
        for (int i = 0; i < N; ++i) r.num[i] = fmaf(f, a[i], r.num[i]);
    }
    return r;
}

// The partials of a split pair: contributor c (work group wf + c) left its
// accumulators and (max, sum) pairs in slot 2 (wf + c), the first one in slot
// 2 wf + 1 (partial_slot).  Resources over up to n contributors from c0 on;
// offsets past them read zeros.
template <int G>
struct Partials {
    static constexpr int kRow = G * kHeadDim * 4, kMl = G * 8;   // bytes of a slot in pacc and pml
    __amdgpu_buffer_rsrc_t acc, ml;
    int c0;
    __device__ inline Partials(const AttnParams& p, int wf, int c0_, int n) : c0(c0_)
    {
        const int64_t slot = 2 * (int64_t)(wf + c0_);
        acc = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(p.pacc + slot * (G * kHeadDim)), (short)0,
                                                n * 2 * kRow, kRawBufferWord3);
        ml = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(p.pml + slot * (G * 2)), (short)0, n * 2 * kMl,
                                               kRawBufferWord3);
    }
    // slot of contributor c0 + j, counted from contributor c0's even slot
    __device__ inline int slot(int j) const { return 2 * j + (j == 0 && c0 == 0); }
};


__device__ inline void store_coherent(float* p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Stores elements [e0, e0 + N) of a work group's partial (all of head h; with
// `first` also the head's max and sum), device-coherent.  A coherent store goes
// through to memory by itself, so with N > 1 (G = 4 and 8) single words wrote
// every line N times, and one vector store does it once: 48 requests of
// 512-8192 tokens, G = 4, 22.7 -> 22.4 us, 12 of 2048-16384, G = 8, 79.1 ->
// 78.4.  With N = 1 (G = 1 and 2) the plain store needs no resource: 4 requests
// of 17-511 tokens 8.72 us, 8.97 through one.
template <int G, int N>
__device__ inline void store_partial(const AttnParams& p, int64_t slot, int e0, int h, bool first,
                                     const RowState<N>& r)
{
    if constexpr (N == 1) {
        store_coherent(&p.pacc[slot * (G * kHeadDim) + e0], r.num[0]);
        if (first) {
            store_coherent(&p.pml[((size_t)slot * G + h) * 2 + 0], r.M);
            store_coherent(&p.pml[((size_t)slot * G + h) * 2 + 1], r.den);
        }
    } else {
        const auto acc = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(p.pacc + slot * (G * kHeadDim)),
                                                           (short)0, Partials<G>::kRow, kRawBufferWord3);
        if constexpr (N == 2)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r.num), acc, e0 * 4, 0, kCoherent);
        else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, r.num), acc, e0 * 4, 0, kCoherent);
        if (first) {
            const auto ml = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(p.pml + slot * (G * 2)), (short)0,
                                                              Partials<G>::kMl, kRawBufferWord3);
            const u32x2 v = {__float_as_uint(r.M), __float_as_uint(r.den)};
            __builtin_amdgcn_raw_buffer_store_b64(v, ml, h * 8, 0, kCoherent);
        }
    }
}

// Rescales r to the running max of C more (max, sum) pairs and adds their
// sums; cf gets the contributors' factors.
template <int N, int C>
__device__ inline void fold_sums(const u32x2 (&ml)[C], int n, RowState<N>& r, float (&cf)[C])
{
    float Mn = r.M;
#pragma unroll
    for (int j = 0; j < C; ++j) {
        cf[j] = j < n ? __uint_as_float(ml[j][0]) : -INFINITY;
        Mn = fmaxf(Mn, cf[j]);
    }
    const float Ms = Mn == -INFINITY ? 0.f : Mn;
    const float f0 = exp2_fast(r.M - Ms);
    r.den *= f0;
    r.num *= f0;
    r.M = Mn;
#pragma unroll
    for (int j = 0; j < C; ++j) {
        cf[j] = exp2_fast(cf[j] - Ms);
        r.den = fmaf(cf[j], __uint_as_float(ml[j][1]), r.den);
    }
}

// Combines up to C partials of a pair at elements [e0, e0 + N) of its rows
// (all of head h), all in flight at once (C <= kFewPartials).
template <int G, int N, int C>
__device__ inline void combine_few(const AttnParams& p, int wf, int nc, int e0, int h, RowState<N>& r)
{
    typedef typename vec_of<float, N>::type f32xN;
    const Partials<G> ps(p, wf, 0, nc);
    u32x2 ml[C];
    f32xN a[C];
#pragma unroll
    for (int j = 0; j < C; ++j) {
        ml[j] = __builtin_amdgcn_raw_buffer_load_b64(ps.ml, h * 8 + ps.slot(j) * ps.kMl, 0, kCoherent);
        const int off = e0 * 4 + ps.slot(j) * ps.kRow;
        if constexpr (N == 1)
            a[j] = __builtin_bit_cast(f32xN, __builtin_amdgcn_raw_buffer_load_b32(ps.acc, off, 0, kCoherent));
        else if constexpr (N == 2)
            a[j] = __builtin_bit_cast(f32xN, __builtin_amdgcn_raw_buffer_load_b64(ps.acc, off, 0, kCoherent));
        else
            a[j] = __builtin_bit_cast(f32xN, __builtin_amdgcn_raw_buffer_load_b128(ps.acc, off, 0, kCoherent));
    }
    float cf[C];
    fold_sums<N, C>(ml, nc, r, cf);
#pragma unroll
    for (int j = 0; j < C; ++j)
#pragma unroll
        for (int i = 0; i < N; ++i) r.num[i] = fmaf(cf[j], a[j][i], r.num[i]);
}

// 16 bytes per lane from offset `off` of r (device-coherent) straight into LDS
// at dst + 16 * lane, without passing through registers.
__device__ inline void load_to_lds(__amdgpu_buffer_rsrc_t r, float* dst, int off)
{
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0,
                                             kCoherent);
#endif
}

// Combines contributors [c0, c1) of a pair into this wave's state in LDS (as
// wave_attend leaves it).  What bounds a combine is the round trips to the
// partials (about 0.6 us each) and then the instructions, not bytes: one
// thread per output element walking all contributors in eights took 4 us for
// the 32 of a 131072-token pair.  So the four waves share the contributors,
// every lane owns 2 G consecutive elements, and the rows go straight into the
// wave's LDS stage (the registers are taken by the tiles).  Kernel time,
// before -> after: one 131071-token request 87.6 -> 84.5 us, one 4096-token
// pair of G = 8 13.6 -> 10.2, one 131072-token pair (512 contributors) 95.7
// -> 37.6.  A stage of 64 KiB instead of 32 per group saves another 5 us there
// and costs every launch 0.1 us.
template <int G>
__device__ inline void combine_wave(const AttnParams& p, int wf, int c0, int c1, int wave, int lane,
                                    float (*s_acc)[kStageFloats], float (*s_m)[G], float (*s_l)[G])
{
    constexpr int N = G * kHeadDim / 64;                       // elements per lane
    constexpr int kLoads = (G * kHeadDim * 4 + 1023) / 1024;   // 1 KiB loads per row
    constexpr int C = G == 8 ? 2 : 4;                          // rows in flight (the stage holds them)
    static_assert(C * kLoads * 256 <= kStageFloats && G * kHeadDim <= kStageFloats, "the stage is too small");
    float* stage = s_acc[wave];
    const int h = lane * N / kHeadDim, dim = lane * N % kHeadDim;
    RowState<N> r;
    r.M = -INFINITY;
    r.den = 0.f;
    r.num = 0.f;
    for (; c0 < c1; c0 += C) {
        const int n = c1 - c0 < C ? c1 - c0 : C;
        const Partials<G> ps(p, wf, c0, n);
        // the reads of the round before are complete before its rows are
        // overwritten: what a load writes to LDS is not ordered behind them
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        u32x2 ml[C];
#pragma unroll
        for (int j = 0; j < C; ++j) {
            ml[j] = __builtin_amdgcn_raw_buffer_load_b64(ps.ml, h * 8 + ps.slot(j) * ps.kMl, 0, kCoherent);
            if (j < n) {
#pragma unroll
                for (int k = 0; k < kLoads; ++k)
                    load_to_lds(ps.acc, stage + (j * kLoads + k) * 256, lane * 16 + k * 1024 + ps.slot(j) * ps.kRow);
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        float cf[C];
        fold_sums<N, C>(ml, n, r, cf);
#pragma unroll
        for (int j = 0; j < C; ++j) {
            if (j < n) {
#pragma unroll
                for (int i = 0; i < N; ++i)
                    r.num[i] = fmaf(cf[j], stage[j * kLoads * 256 + lane * N + i], r.num[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) stage[lane * N + i] = r.num[i];
    if (dim == 0) {
        s_m[wave][h] = r.M;
        s_l[wave][h] = r.den;
    }
}

// What a wave's own partition gives a work group (all scalar).
struct WavePlan {
    bool planned = false;      // false: the group-wide partition decides
    bool all_nonempty = false;
    int short_pairs = 0;       // > 0: single waves take whole pairs, this many in all
    int part_units = 0;        // > 0: pair cut, units of the group's part,
    int cut_first = 0, cut_last = 0;   // and the work groups of its pair
    int b = 0, g = 0, blk = 0, L = 0;  // the group's first segment
    int64_t V = 0, W = 0, v0 = 0, v1 = 0, vf = 0, stride = 0;
};

template <int G, bool kCheck, bool kAppend>
__global__ __launch_bounds__(kAttnThreads) __attribute__((amdgpu_waves_per_eu(2))) void attn_kernel(AttnParams p,
                                                        const int32_t* __restrict__ bt,
                                                        const int32_t* __restrict__ lens)
{
    constexpr int D = kHeadDim;
    __shared__ __align__(16) float s_acc[kWaves][kStageFloats];   // a wave's state: its first G * D floats
    __shared__ float s_m[kWaves][G];
    __shared__ float s_l[kWaves][G];
    __shared__ int s_lens[kCachedLens];
    __shared__ int s_wsum[kWaves];
    __shared__ int s_wmax[kWaves];
    __shared__ int s_wcnt[kWaves];
    __shared__ int s_loc_b;
    __shared__ int s_loc_g;
    __shared__ int s_loc_blk;
    __shared__ int64_t s_loc_vf;
    __shared__ int s_last;
    __shared__ float s_new[kWaves][G];
    __shared__ int s_order[kShortRequests];   // the non-empty requests, in order

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t w = blockIdx.x;
    const int B = p.B;
    const bool cached = B <= kCachedLens;
#ifdef APEX_TRACE_WORK_GROUPS
    if (tid < kTraceWords) s_trace[tid] = tid == 0 ? trace_clock() : 0;
#endif

    // 1. partition (positions on the cost line of plan_policy.h: every
    // non-empty pair's K cost positions, then its blocks)
    // with the input check, a context longer than an explicit table row is
    // cut to the row (and reported)
    const int64_t row_tokens = p.bt_stride * kBlockSize;
    auto is_cut = [&](int L) -> bool { return kCheck && p.bt_stride > 0 && L > row_tokens; };
    // Tokens the partition covers: the cached ones.  With the fused append
    // the current token (position L - 1) comes from the new rows, so the
    // caches hold the first L - 1; a context cut to its row keeps every token
    // of the row, and its current token, whose position lies past the row,
    // is attended but has no slot to be stored in.  The tight table stride
    // follows the (cut) full lengths.
    constexpr bool append = kAppend;
    auto cached_len = [&](int L) -> int {
        if (is_cut(L)) return (int)row_tokens;
        return append && L > 0 ? L - 1 : L;
    };
    auto len_of = [&](int b) -> int { return cached ? s_lens[b] : cached_len(lens[b]); };
    const int K = p.seg_cost;

    // The prologue is serial code of every work group: no K/V byte is asked
    // for before its end, and a wave issues one instruction in four cycles at
    // best, so its time is its instruction count.  For a batch of up to
    // 64 R requests every wave derives the partition on its own, lane i
    // holding R consecutive requests (R = 1 up to 64 requests, 4 up to 256, 8 up to 512): one
    // scan of the requests' cost, ballots and lane reads, no barrier and no
    // LDS round trip, all results in scalar registers, products in 32 bits.
    // Returns false, with nothing decided, when 32 bits do not hold them
    // (plan bound: V (launched + 1) < 2^32).  Against the group-wide form
    // below, a work group's time from its start to its first segment falls
    // from 1.9 to 1.1 us for 16 requests and from 1.7 to 1.0 us for 4.
    auto plan_in_wave = [&](auto runs) -> WavePlan {
        constexpr int R = decltype(runs)::value;
        WavePlan r;
        int raws[R], Ls[R], nbs[R];
        unsigned cost = 0;
        int maxb = 0, maxnb = 0, nonempty = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) raws[i] = 0;
        if (R > 1 && lane * R + R <= B) {
            // (context_lens is 4-byte aligned; such vector loads are allowed)
            typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
            for (int i = 0; i + 3 < R; i += 4) {
                const i32x4_any v = *(const i32x4_any*)(lens + lane * R + i);
                raws[i] = v[0];
                raws[i + 1] = v[1];
                raws[i + 2] = v[2];
                raws[i + 3] = v[3];
            }
        } else if (lane * R < B) {
#pragma unroll
            for (int i = 0; i < R; ++i)
                if (lane * R + i < B) raws[i] = lens[lane * R + i];
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int raw = raws[i];
            if (is_cut(raw)) report_error(p, kErrTableRow);
            Ls[i] = cached_len(raw);
            // blocks_of in 32 bits (no length is near 2^32)
            nbs[i] = (int)(((unsigned)max(Ls[i], 0) + kBlockSize - 1) / kBlockSize);
            const int full = is_cut(raw) ? (int)row_tokens : raw;
            maxb = max(maxb, (int)(((unsigned)max(full, 0) + kBlockSize - 1) / kBlockSize));
            maxnb = max(maxnb, nbs[i]);
            nonempty += __popcll(__ballot(nbs[i] > 0));
            cost += nbs[i] > 0 ? (unsigned)(nbs[i] + K) : 0u;
            if (lane * R < B) s_lens[lane * R + i] = Ls[i];   // (past B: never read, inside the array)
        }
        // every wave writes the same values and reads back what it wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const unsigned hi = (unsigned)wave_incl_sum((int)cost), lo = hi - cost;
        const unsigned total = (unsigned)lane_value((int)hi, 63);
        // the tight table follows the full lengths, the rules below the cached
        // ones: with the fused append a request may have a block fewer of them
        const int longest = lane_value(wave_incl_max(append ? maxnb : maxb), 63);
        r.stride = p.bt_stride > 0 ? p.bt_stride : append ? lane_value(wave_incl_max(maxb), 63) : longest;
        nonempty = uniform(nonempty);
        r.all_nonempty = nonempty == B;
        const uint64_t V64 = (uint64_t)total * (unsigned)p.Hkv;
        if ((V64 >> 32) != 0 || V64 * ((unsigned)p.launched + 1ull) > 0xffffffffull) return r;
        r.planned = true;
        const unsigned hk = (unsigned)p.Hkv, V32 = (unsigned)V64;
        const unsigned units = V32 - (unsigned)K * (unsigned)nonempty * hk;
        // a small batch of the default grid is cut by pairs (plan_policy.h): one
        // segment per work group
        const unsigned floor_units = p.cus > 0 && 64 * R <= kPairCutRequests
                                         ? pair_cut_floor(units, (uint32_t)nonempty * hk, (uint32_t)longest,
                                                          (uint32_t)p.cus, (uint32_t)p.launched)
                                         : 0;
        if (floor_units > 0) {
            unsigned T[R], parts[R], sum = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                T[i] = (unsigned)nbs[i];
                parts[i] = nbs[i] > 0;
            }
            if (floor_units < (unsigned)longest) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    if (nbs[i] == 0) continue;
                    T[i] = pair_part_units((uint32_t)nbs[i], floor_units, G);
                    parts[i] = ((unsigned)nbs[i] + T[i] - 1) / T[i];
                }
            }
#pragma unroll
            for (int i = 0; i < R; ++i) sum += parts[i];
            const unsigned phi = (unsigned)wave_incl_sum((int)sum), plo = phi - sum;
            const uint64_t hit = __ballot(plo * hk <= (unsigned)w && (unsigned)w < phi * hk);
            if (hit == 0) return r;   // no part is left for this work group
            const int ln = __builtin_ctzll(hit);
            unsigned rest = (unsigned)w - (unsigned)lane_value((int)plo, ln) * hk;
            unsigned c = (unsigned)lane_value((int)parts[0], ln);
            int nb = lane_value(nbs[0], ln), per = lane_value((int)T[0], ln);
            r.L = lane_value(Ls[0], ln);
            r.b = ln * R;
#pragma unroll
            for (int i = 1; i < R; ++i) {
                if (rest >= c * hk) {
                    rest -= c * hk;
                    c = (unsigned)lane_value((int)parts[i], ln);
                    nb = lane_value(nbs[i], ln);
                    per = lane_value((int)T[i], ln);
                    r.L = lane_value(Ls[i], ln);
                    ++r.b;
                }
            }
            r.g = hk <= 64 ? __popcll(__ballot((unsigned)lane < hk && (unsigned)lane * c <= rest)) - 1
                         : uniform((int)(rest / c));
            const int part = (int)rest - r.g * (int)c;
            r.blk = part * per;
            r.part_units = min(per, nb - r.blk);
            r.cut_first = (int)w - part;
            r.cut_last = r.cut_first + (int)c - 1;
            r.v1 = 1;   // the group has work
            return r;
        }
        if (p.cus > 0 && waves_take_pairs(units, (uint32_t)nonempty * hk, (uint32_t)longest, (uint32_t)p.launched)) {
            int mine = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) mine += nbs[i] > 0;
            int at = wave_incl_sum(mine) - mine;
#pragma unroll
            for (int i = 0; i < R; ++i)
                if (nbs[i] > 0) s_order[at++] = lane * R + i;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            r.short_pairs = nonempty * (int)hk;
            return r;
        }
        const unsigned W32 = clamp_workers<uint32_t>(units >> __builtin_ctz((unsigned)p.min_units), units,
                                                     (uint32_t)p.launched, (uint32_t)nonempty * hk, (uint32_t)p.cus);
        r.V = V32;
        r.W = W32;
        if (units == 0 || (unsigned)w >= W32) return r;
        const unsigned ends = ((unsigned)w + (lane & 1)) * V32 / W32;   // lane 0: start, lane 1: end
        const unsigned u0 = (unsigned)lane_value((int)ends, 0);
        r.v0 = u0;
        r.v1 = (unsigned)lane_value((int)ends, 1);
        // the lane whose requests hold u0, the request, the pair
        const int ln = __builtin_ctzll(__ballot(lo * hk <= u0 && u0 < hi * hk));
        unsigned vpre = (unsigned)lane_value((int)lo, ln) * hk;
        int nb = lane_value(nbs[0], ln);
        r.L = lane_value(Ls[0], ln);
        r.b = ln * R;
#pragma unroll
        for (int i = 1; i < R; ++i) {
            const unsigned span = nb > 0 ? (unsigned)(nb + K) * hk : 0u;
            if (u0 >= vpre + span) {
                vpre += span;
                nb = lane_value(nbs[i], ln);
                r.L = lane_value(Ls[i], ln);
                ++r.b;
            }
        }
        const unsigned per = (unsigned)(nb + K);
        // kv-head: pair g of the request starts at vpre + g per
        r.g = hk <= 64 ? __popcll(__ballot((unsigned)lane < hk && vpre + (unsigned)lane * per <= u0)) - 1
                     : uniform((int)((u0 - vpre) / per));
        const unsigned first = vpre + (unsigned)r.g * per + (unsigned)K;   // position of the pair's block 0
        r.vf = first;
        r.blk = u0 > first ? (int)(u0 - first) : 0;
        return r;
    };
    WavePlan plan;
    if (B <= 64)
        plan = plan_in_wave(std::integral_constant<int, 1>());
    else if (B <= 256)
        plan = plan_in_wave(std::integral_constant<int, 4>());
    else if (B <= kShortRequests)
        plan = plan_in_wave(std::integral_constant<int, 8>());

    const int short_pairs = plan.short_pairs, part_units = plan.part_units;
    const int cut_first = plan.cut_first, cut_last = plan.cut_last;
    bool all_nonempty = plan.all_nonempty;
    int b = plan.b, g = plan.g, blk = plan.blk, L = plan.L;
    int64_t V = plan.V, W = plan.W, v0 = plan.v0, v1 = plan.v1, vf = plan.vf, stride = plan.stride;

    // More than kShortRequests requests (and partitions past 32 bits):
    // context_lens is read once by the group, each thread sums the blocks of a
    // contiguous run of requests (and keeps the lengths in LDS when they fit);
    // wave-level scans plus one barrier give the prefix sums, the total, the
    // longest request and the non-empty requests.
    if (!plan.planned) {
    const int seg = (B + kAttnThreads - 1) / kAttnThreads;
    const int r0 = min(B, tid * seg);
    const int r1 = min(B, r0 + seg);
    int tsum = 0, tmax = 0, tcnt = 0;
    for (int b = r0; b < r1; ++b) {
        const int raw = lens[b];
        if (is_cut(raw)) report_error(p, kErrTableRow);
        const int L = cached_len(raw);
        if (cached) s_lens[b] = L;
        const int nb = (int)blocks_of(L, kBlockSize);
        tsum += nb;
        tmax = max(tmax, (int)blocks_of(is_cut(raw) ? (int)row_tokens : raw, kBlockSize));
        tcnt += nb > 0;
    }
    const int own_cnt = tcnt;
    int incl = wave_incl_sum(tsum);
    tmax = wave_incl_max(tmax);
    int incl_cnt = wave_incl_sum(tcnt);
    if (lane == 63) {
        s_wsum[wave] = incl;
        s_wmax[wave] = tmax;
        s_wcnt[wave] = incl_cnt;
    }
    __syncthreads();
    int total = 0, maxb = 0, nonempty = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
        if (v < wave) {
            incl += s_wsum[v];
            incl_cnt += s_wcnt[v];
        }
        total += s_wsum[v];
        maxb = max(maxb, s_wmax[v]);
        nonempty += s_wcnt[v];
    }
    const int64_t units = (int64_t)uniform(total) * p.Hkv;
    const int64_t pairs = (int64_t)uniform(nonempty) * p.Hkv;
    stride = p.bt_stride > 0 ? p.bt_stride : (int64_t)uniform(maxb);
    V = units + (int64_t)K * pairs;
    // When V (launched + 1) < 2^32 (any batch below about 8 M units at the
    // default grid) every product below fits 32 bits and the partition runs in
    // 32-bit arithmetic, else in 64-bit; both give the same ranges.  Lanes 0
    // and 1 find the range's two ends in one division.
    const bool narrow = ((uint64_t)V >> 32) == 0 && (uint64_t)V * ((uint64_t)p.launched + 1) <= 0xffffffffull;
    if (narrow) {
        const uint32_t W32 = active_workers_t<uint32_t>((uint32_t)units, (uint32_t)p.launched, (uint32_t)p.min_units,
                                                        (uint32_t)pairs, (uint32_t)p.cus);
        const uint32_t ends = units > 0 && w < W32 ? (uint32_t)(w + (lane & 1)) * (uint32_t)V / W32 : 0u;
        W = W32;
        v0 = (uint32_t)__builtin_amdgcn_readlane((int)ends, 0);
        v1 = (uint32_t)__builtin_amdgcn_readlane((int)ends, 1);
    } else {
        W = active_workers(units, (int64_t)p.launched, p.min_units, pairs, p.cus);
        const int64_t ends = units > 0 && w < W ? worker_start(w + (lane & 1), V, W) : 0;
        v0 = ((int64_t)__builtin_amdgcn_readlane((int)(ends >> 32), 0) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)ends, 0);
        v1 = ((int64_t)__builtin_amdgcn_readlane((int)(ends >> 32), 1) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)ends, 1);
    }

    // The worker's blocks are those whose positions lie in [v0, v1).  Request
    // b's positions start at Hkv (pre_b + K pp_b) (pre_b blocks and pp_b
    // non-empty requests before it) and number Hkv (nb_b + K); the thread
    // whose requests hold v0 finds the pair there and its first block at or
    // after v0 (block 0 when v0 is one of the pair's cost positions), and
    // publishes the pair, that block and the position of the pair's block 0.
    // (In I = uint32_t every position is below V < 2^32.)
    auto locate = [&](auto at) {
        using I = decltype(at);
        const I hk = (I)p.Hkv, Kc = (I)K;
        const I lo = (I)(incl - tsum) + Kc * (I)(incl_cnt - own_cnt);
        const I hi = (I)incl + Kc * (I)incl_cnt;
        if (lo * hk <= at && at < hi * hk) {
            I vpre = lo * hk;
            for (int b = r0; b < r1; ++b) {
                // with one request per thread, its block count is the scan's
                const I nb = seg == 1 ? (I)tsum : (I)blocks_of(len_of(b), kBlockSize);
                if (nb == 0) continue;
                const I span = (nb + Kc) * hk;
                if (at < vpre + span) {
                    const I g = div_floor(at - vpre, nb + Kc);
                    const I vf = vpre + g * (nb + Kc) + Kc;   // position of the pair's block 0
                    s_loc_b = b;
                    s_loc_g = (int)g;
                    s_loc_blk = (int)(at > vf ? at - vf : 0);
                    s_loc_vf = (int64_t)vf;
                    break;
                }
                vpre += span;
            }
        }
    };
    if (v0 < v1) {
        if (narrow)
            locate((uint32_t)v0);
        else
            locate(v0);
    }
    __syncthreads();

    if (v0 < v1) {
        b = uniform(s_loc_b);
        g = uniform(s_loc_g);
        blk = uniform(s_loc_blk);
        vf = uniform64(s_loc_vf);
        L = uniform(len_of(b));
    }
    all_nonempty = uniform(nonempty) == B;
    }

    if (short_pairs > 0) {
        // every wave takes whole pairs of its own: no barrier, no merge, the rows
        // straight from its registers.  The k-th run of `launched` pairs goes to
        // wave k mod 4 of the work groups, shifted by kPairSkew groups a wave; the
        // last one, unless whole, to the groups that start first
#ifdef APEX_TRACE_WORK_GROUPS
        __syncthreads();   // the row is cleared before the waves count into it
        if (tid == 0) s_trace[1] = trace_clock();
#endif
        const int wv = uniform(wave);
        const int skew = p.launched > kWaves * kPairSkew ? wv * kPairSkew : 0;
        for (int first = wv * p.launched; first < short_pairs; first += kWaves * p.launched) {
            const int from = first + p.launched <= short_pairs ? skew : 0;
            const int i = first + ((int)w + from < p.launched ? (int)w + from : (int)w + from - p.launched);
            if (i >= short_pairs) break;
            const int k = uniform((int)((unsigned)i / (unsigned)p.Hkv));
            const int bp = uniform(s_order[k]), Lp = uniform(s_lens[bp]);
            const int32_t* row = bt + (size_t)bp * (size_t)stride;
            const WaveSeg cs = wave_seg<G, 1>(p, row, bp, i - k * p.Hkv, 0, (int)blocks_of(Lp, kBlockSize), 0, lane);
            WaveTiles st;
            WaveState ws;
            NewTokenElems<kEmitElems<G>> unused;
            load_first_tiles<kCheck, 1>(p, cs, bt, st, lane);
            load_q<G>(st.qnext, cs, lane);
            wave_attend<G, kCheck, kAppend, 1>(p, cs, cs, bt, false, Lp, st, wave, lane, ws, s_new[wv], row, unused);
            emit_wave<G, kCheck, kAppend>(p, ws, bp, cs.g, Lp + 1, lane, s_new[wv], row, bt);
#ifdef APEX_TRACE_WORK_GROUPS
            if (lane == 0) {
                atomicAdd((unsigned long long*)&s_trace[4], 1ull);
                atomicAdd((unsigned long long*)&s_trace[6], (unsigned long long)cs.n);
            }
#endif
        }
    }

    // A segment is the worker's blocks of one pair: from block blk of the pair
    // whose block 0 lies at position vf, up to the pair's end or the worker's
    // range end v1, whichever comes first (none when v1 falls on or before
    // the block: the range ends among cost positions).
    auto seg_take = [&](int nb_, int blk_, int64_t vf_) -> int {
        const int64_t left = v1 - (vf_ + blk_);
        return left <= 0 ? 0 : (int)min((int64_t)(nb_ - blk_), left);
    };
    int nb = 0, take = 0;
    if (v0 < v1) {
        nb = (int)blocks_of(L, kBlockSize);
        take = part_units > 0 ? part_units : seg_take(nb, blk, vf);
    }

    if (take > 0) {
    // Moves a segment cursor past its segment to the worker's next one;
    // false when the worker's range is done.
    auto advance = [&](int& b_, int& L_, int& nb_, int& g_, int& blk_, int64_t& vf_, int take_) -> bool {
        blk_ += take_;
        if (blk_ < nb_) return false;   // the range ended inside the pair
        const int64_t vnext = vf_ + nb_ + K;   // the next pair's block 0
        if (v1 <= vnext) return false;
        blk_ = 0;
        vf_ = vnext;
        if (++g_ == p.Hkv) {
            g_ = 0;
            do {
                ++b_;
            } while (b_ < B && len_of(b_) <= 0);
            if (b_ >= B) return false;   // unreachable: positions remain after the current pair
            L_ = uniform(len_of(b_));
            nb_ = (int)blocks_of(L_, kBlockSize);
        }
        return true;
    };

    // 2. segments.  Each one is announced to the waves together with the
    // next, so their K/V pipelines run on from one to the other.
#ifdef APEX_TRACE_WORK_GROUPS
    if (tid == 0) s_trace[1] = trace_clock();
#endif
    WaveSeg cs = wave_seg<G, kWaves>(p, bt + (size_t)uniform(b) * (size_t)stride, b, g, blk, blk + take, wave, lane);
    WaveTiles st;
    st.prefetched = false;
    st.cur0 = st.cur1 = st.nid0 = st.nid1 = 0;
    load_q<G>(st.qnext, cs, lane);
    while (true) {
        int b2 = b, L2 = L, nb2 = nb, g2 = g, blk2 = blk;
        int64_t vf2 = vf;
        // the loads of a segment that the pipeline did not run on into go out
        // before the next segment is looked up
        if (!st.prefetched) load_first_tiles<kCheck, kWaves>(p, cs, bt, st, lane);
        const bool more = part_units == 0 && advance(b2, L2, nb2, g2, blk2, vf2, take);
        const int take2 = more ? seg_take(nb2, blk2, vf2) : 0;
        WaveSeg ns = cs;
        ns.n = 0;
        if (more)
            ns = wave_seg<G, kWaves>(p, bt + (size_t)uniform(b2) * (size_t)stride, b2, g2, blk2, blk2 + take2, wave,
                             lane);
        // the pair's first and last work groups: this one, unless the range
        // cuts the pair (found here, while the loads are in flight)
        const int wf = part_units > 0 ? cut_first : blk == 0 ? (int)w : uniform((int)worker_of(vf, V, W));
        const int wl = part_units > 0      ? cut_last
                       : blk + take == nb ? (int)w
                                          : uniform((int)worker_of(vf + nb - 1, V, W));
        NewTokenElems<kEmitElems<G>> ne;
        {
            WaveState ws;
            wave_attend<G, kCheck, kAppend, kWaves>(p, cs, ns, bt,
                                                    more && take >= kPrefetchBlocks && take2 >= kPrefetchBlocks, L,
                                                    st, wave, lane, ws, s_new[0],
                                                    bt + (size_t)uniform(b) * (size_t)stride, ne);
            store_wave_state<G>(ws, wave, lane, s_acc, s_m, s_l);
        }
        __syncthreads();
#ifdef APEX_TRACE_WORK_GROUPS
        if (tid == 0) {
            ++s_trace[4];
            s_trace[6] += take;
        }
#endif

        // 3. merge the waves, emit rows or a partial
        const int64_t slot = partial_slot(w, wf);
        constexpr int N = kEmitElems<G>;
        const int h = tid * N / D, dim = tid * N % D;
        const bool emits = G >= 2 || tid < D;
        auto emit = [&](RowState<N>& r) {
            if (append) {
                fold_new_token<N>(s_new[0][h], ne.vn, r);
                if (h == 0) store_new_token<kCheck, N>(p, ne, g, L + 1, dim);
            }
            write_row<N>(p, b, g * G + h, dim, r);
        };
        if (emits) {
            RowState<N> r = merge_waves<G, N>(s_acc, s_m, s_l, h, dim);
            if (wf == wl) {
                emit(r);
            } else {
                store_partial<G, N>(p, slot, tid * N, h, dim == 0, r);
            }
        }
        if (wf != wl) {
#ifdef APEX_TRACE_WORK_GROUPS
            if (tid == 0) ++s_trace[5];
#endif
            // The partials are written with device-coherent stores; waiting for
            // them to complete before the arrival is counted makes them visible
            // to the last arriver's device-coherent loads, on whichever XCD it
            // runs, without writing back or invalidating the L2.
            asm volatile("" ::: "memory");   // (no store moves past the wait)
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) {
                int32_t* cnt = &p.counters[(size_t)b * p.Hkv + g];
                const int old = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int last = old == wl - wf;
                if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_last = last;
            }
            __syncthreads();
            if (s_last) {
                // combine the pair's partials: a few by the threads that own
                // the output elements, more by the four waves, whose states
                // are then merged like those of a segment
                const int nc = wl - wf + 1;
                RowState<N> r;
                r.M = -INFINITY;
                r.den = 0.f;
                r.num = 0.f;
                constexpr int few = kFewPartials<G>;
                if (nc <= few) {
                    if (emits) {
                        if (nc <= 2)
                            combine_few<G, N, 2>(p, wf, nc, tid * N, h, r);
                        else if (nc <= 4)
                            combine_few<G, N, 4>(p, wf, nc, tid * N, h, r);
                        else if (nc <= 8 && few >= 8)
                            combine_few<G, N, few < 8 ? few : 8>(p, wf, nc, tid * N, h, r);
                        else
                            combine_few<G, N, few>(p, wf, nc, tid * N, h, r);
                        emit(r);
                    }
                } else {
                    const int per = (nc + kWaves - 1) / kWaves;
                    const int c0 = uniform(wave) * per;
                    combine_wave<G>(p, wf, c0, c0 + per < nc ? c0 + per : nc, uniform(wave), lane, s_acc, s_m, s_l);
                    __syncthreads();
                    if (emits) {
                        r = merge_waves<G, N>(s_acc, s_m, s_l, h, dim);
                        emit(r);
                    }
                }
            }
        }
        __syncthreads();

        if (!more) break;
        b = b2;
        vf = vf2;
        L = L2;
        nb = nb2;
        g = g2;
        blk = blk2;
        take = take2;
        cs = ns;
    }
    }

    // rows of empty requests are zeros (and lse = -inf); with the fused
    // append a request whose only token is the current one returns its V row
    // (lse = its scaled logit) and stores its K/V
    for (int b = all_nonempty ? B : (int)w; b < B; b += (int)gridDim.x) {
        if (len_of(b) > 0) continue;
        if (append && lens[b] == 1) {
            const size_t nrow = (size_t)b * p.new_stride;
            for (int i = tid; i < p.Hq * D; i += kAttnThreads) {
                const int h = i / D, dim = i % D;
                p.out[((size_t)b * p.Hq + h) * D + dim] = p.v_new[nrow + (size_t)(h / (p.Hq / p.Hkv)) * D + dim];
            }
            if (p.lse) {
                for (int h = wave; h < p.Hq; h += kWaves) {
                    const f16x2 k2 = *(const f16x2*)(p.k_new + nrow + (size_t)(h / (p.Hq / p.Hkv)) * D + 2 * lane);
                    const f16x2 q2 = *(const f16x2*)(p.q + ((size_t)b * p.Hq + h) * D + 2 * lane);
                    float x = fmaf((float)q2[0], (float)k2[0], (float)q2[1] * (float)k2[1]);
#pragma unroll
                    for (int m = 32; m >= 1; m >>= 1) x += wave_shfl_xor(x, m);
                    if (lane == 0) p.lse[(size_t)b * p.Hq + h] = x * p.scale_log2 * 0.69314718055994531f;
                }
            }
            for (int i = tid; i < p.Hkv * D; i += kAttnThreads)
                store_new_token<kCheck, 1>(
                    p, load_new_token_elems<kCheck, 1>(p, bt + (size_t)b * stride, bt, b, i / D, 1, i % D), i / D, 1,
                    i % D);
        } else {
            RowState<1> r;
            r.M = 0.f;
            r.den = 0.f;
            r.num = 0.f;
            for (int i = tid; i < p.Hq * D; i += kAttnThreads) write_row<1>(p, b, i / D, i % D, r);
        }
    }
#ifdef APEX_TRACE_WORK_GROUPS
    __syncthreads();   // every wave has counted
    if (p.trace && tid == 0 && w < p.trace_groups) {
        uint64_t* t = p.trace + w * kTraceWords;
        t[0] = s_trace[0];
        t[1] = s_trace[1];
        t[2] = s_trace[2];
        t[3] = trace_clock();
        t[4] = s_trace[4];
        t[5] = s_trace[5];
        t[6] = s_trace[6];
        t[7] = 0;
    }
#endif
}

}  // namespace apex
