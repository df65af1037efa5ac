// plan_policy.h -- work partition of batched paged decode attention.
//
// Decode attention streams every cached K/V row of every request once (APEX
// Sec. 2.2 and Sec. 2.3: it is the memory-bandwidth-bound part of a decode
// step).  A batch is ragged -- a few long requests next to many short ones --
// so the work is cut by amount, not by request.  One unit is one block of one
// kv-head (16 tokens: 4 KiB of K plus 4 KiB of V at d = 128); the units are
// laid out in (request b, kv-head g, block) order.  Besides its units, a
// worker pays a fixed cost for every (request, kv-head) pair it attends --
// the block-id and first-tile latency, the merge and the emit -- so each
// non-empty pair is charged K = kSegmentCostUnits extra positions: on a line
// of V = U + K P positions (P pairs) every pair has its K cost positions
// followed by its blocks, and worker w of W takes the positions
// [floor(w V / W), floor((w + 1) V / W)).  The blocks among them form a
// contiguous range of units, so every worker walks consecutive units as
// before, and a run of short pairs no longer lands on one worker.  A
// (request, kv-head) pair whose units straddle workers is finished by a
// log-sum-exp combine of the workers' partial results.  Each worker has at
// most two partial segments (its first and its last), which fixes where
// they are stored.  Forced grids (tests) take K = 0: equal units.
//
// These functions are compiled for both the host (inspection, tests) and the
// device (every worker runs them on its own), so both see the same partition.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace apex {

constexpr int kHeadDim = 128;
constexpr int kBlockSize = 16;
constexpr int kMinUnitsPerWorker = 16;  // four blocks per wave of a 4-wave work group
static_assert((kMinUnitsPerWorker & (kMinUnitsPerWorker - 1)) == 0, "the kernel divides by it with a shift");
constexpr int64_t kUnitsPerCuForOne = 1024;   // 8 MiB of K/V per CU
// Cost of a pair's segment in units: a short segment takes about 2-3 us of
// latency (block ids, first tiles, merge, emit), the time a work group
// streams about eight blocks in.
constexpr int kSegmentCostUnits = 8;

// floor(a / b) for a >= 0, b > 0.  A 64-bit division is a long software
// sequence on the GPU; the partition's operands nearly always fit in 32 bits,
// where the hardware-assisted 32-bit sequence gives the same quotient.  The
// 64-bit one is kept out of line, so that the code a work group runs before
// its first load stays short.
__host__ __device__ __attribute__((noinline)) inline int64_t div_floor_wide(int64_t a, int64_t b)
{
    return a / b;
}

__host__ __device__ inline int64_t div_floor(int64_t a, int64_t b)
{
    if (__builtin_expect(((uint64_t)a | (uint64_t)b) <= 0xffffffffull, 1))
        return (int64_t)((uint32_t)a / (uint32_t)b);
    return div_floor_wide(a, b);
}

__host__ __device__ inline uint32_t div_floor(uint32_t a, uint32_t b) { return a / b; }

__host__ __device__ inline int64_t blocks_of(int32_t len, int bs)
{
    return len > 0 ? ((int64_t)len + bs - 1) / bs : 0;
}

// Workers that get units: at most the launched ones; enough that each has
// about min_units units, but never fewer than the non-empty (request,
// kv-head) pairs -- a small batch would otherwise queue several short pairs
// on one work group, one after another, while most of the device idles.
// With cus > 0 (the device's compute units), a batch of at most one pair per
// CU and at most kUnitsPerCuForOne units per CU uses only the first `cus`
// work groups: one per CU (work groups are handed out round-robin over the
// XCDs and then over their CUs), no pair split between two groups, and no
// second group sharing the CU.
// The integer type I is int64_t, or uint32_t where the caller has shown that
// every operand and cus * kUnitsPerCuForOne fit (the kernel's 32-bit path).
// clamp_workers takes the quotient units / min_units from the caller.
template <typename I>
__host__ __device__ inline I clamp_workers(I w, I units, I launched, I pairs, I cus)
{
    if (cus > 0 && pairs <= cus && units <= cus * (I)kUnitsPerCuForOne && launched > cus) launched = cus;
    if (w < pairs) w = pairs;
    if (w < 1) w = 1;
    return w < launched ? w : launched;
}

template <typename I>
__host__ __device__ inline I active_workers_t(I units, I launched, I min_units, I pairs, I cus)
{
    return clamp_workers<I>(div_floor(units, min_units > 0 ? min_units : (I)1), units, launched, pairs, cus);
}

__host__ __device__ inline int64_t active_workers(int64_t units, int64_t launched, int min_units,
                                                  int64_t pairs, int64_t cus)
{
    return active_workers_t<int64_t>(units, launched, min_units, pairs, cus);
}

// First position of worker w on the cost line of `positions` positions (the
// range of w is [worker_start(w), worker_start(w+1))).
__host__ __device__ inline int64_t worker_start(int64_t w, int64_t positions, int64_t workers)
{
    return div_floor(w * positions, workers);
}

// The worker whose range holds position v (0 <= v < positions).
__host__ __device__ inline int64_t worker_of(int64_t v, int64_t positions, int64_t workers)
{
    return div_floor((v + 1) * workers - 1, positions);
}

// Position of the first block of the pair with index `pair` (in (request,
// kv-head) order over the non-empty pairs) whose units start at unit p0:
// every pair up to and including it adds its K cost positions.
__host__ __device__ inline int64_t first_block_position(int64_t p0, int64_t pair, int64_t K)
{
    return p0 + K * (pair + 1);
}

// Partial slot that worker w uses for a split pair whose first contributor
// is wf: the first contributor holds the pair's start and runs past its
// range, so the pair is its last segment (slot 2w + 1); every later one
// starts inside the pair, so the pair is its first segment (slot 2w).
__host__ __device__ inline int64_t partial_slot(int64_t w, int64_t wf)
{
    return w == wf ? 2 * w + 1 : 2 * w;
}

// Pair cut: small batches.  The cost line cuts anywhere, so in a small batch
// nearly every work group gets the end of one pair and the start of another:
// two segments in a row, each with its first-tile latency, and two combines,
// which is most of a launch of 10 us.  When every pair fits the work groups in
// parts of at most kPairCutMaxPart units, a work group takes one part of one
// pair instead.  Kernel time, line -> parts: MHA of 17-511 tokens 10.3 -> 8.0
// us, 8 pairs of 300 tokens 10.8 -> 7.2, 512 pairs of 20-200 tokens 13.5 ->
// 10.8.  With longer parts the uneven last ones cost what the combine saves: of
// 300 batches those with 12 to 24 units per free work group take 0.94 to 0.98 of
// the line's time on average in parts, with 24 to 26 0.98, with 26 to 30 1.01 to
// 1.03 and up to 1.14 (270 pairs of 116 and 676 tokens in turn, parts of 29: 21.0
// us, 18.8 on the line).  Pairs of up to kWholePairUnits stay whole: up to four
// blocks per wave cost less than a combine; so do pairs of up to kWholeAloneUnits
// where the parts do not fit (20 such batches: 0.98 of their time in parts of 24
// to 32 units, never above).  The part grows with the pair (pair_part_units), since a pair's last
// work group reads all its parts' partials, sooner for G = 8, whose partials
// are the largest.
constexpr uint32_t kPairCutMaxPart = 24;
constexpr uint32_t kWholePairUnits = 16;
constexpr uint32_t kWholeAloneUnits = 32;

// The cut is derived in the kernel's in-register partition, up to four requests
// per lane.  (More requests have at most 512 pairs with one kv-head only.)
constexpr int kPairCutRequests = 256;

// Least units per part that keep the parts of all pairs within the work groups
// (sum ceil(nb / T) <= units / T + pairs); at least `longest` (the longest
// pair's units) = no pair is cut; 0 = the pair cut does not apply.
__host__ __device__ inline uint32_t pair_cut_floor(uint32_t units, uint32_t pairs, uint32_t longest, uint32_t cus,
                                                   uint32_t launched)
{
    const uint32_t groups = pairs <= cus ? (cus < launched ? cus : launched) : launched;
    if (pairs == 0 || pairs > groups) return 0;
    const uint32_t room = groups - pairs;
    if (units > room * kPairCutMaxPart) return longest <= kWholeAloneUnits ? longest : 0;
    if (longest <= kWholePairUnits) return longest;
    return (units + room - 1) / room;
}

// Units per part of a pair of nb blocks (the last part may have fewer).
__host__ __device__ inline uint32_t pair_part_units(uint32_t nb, uint32_t floor_units, uint32_t group)
{
    if (nb <= kWholePairUnits) return nb;
    const uint32_t low = nb < 256 ? nb : 256;
    const uint32_t T = (group == 8 ? 8 + low / 32 : 4 + low * 3 / 64) + (nb - low) / 128;
    return T > floor_units ? T : floor_units;
}

// Short pairs: with more pairs than work groups, a group attends several one
// after the other, and a pair of a few blocks costs it a first-tile latency, a
// join and a merge (7 us and half a microsecond a block on the line) for one or
// two blocks per wave.  Instead every wave takes whole pairs of its own: 3 us
// and 1.2 us a block for the longest, all waves at once, no barrier, no merge.
// Kernel time, line -> waves: 2048 pairs of 20-60 tokens 21.2 -> 11.5 us, 2400
// of 16-48 22.6 -> 13.2, 1280 of 16-130 (G = 8) 21.9 -> 13.2, 2048 of 200-256
// 46.3 -> 38.7.  The rule compares the two estimates, which place the line up to
// one pair per wave (2048 on 256 CUs): it keeps 640 pairs of 200-256 on the line
// (20.9 us, 27.2 by waves).  They know neither the bytes nor a second round, in
// which a wave may get two of the longest and end alone.  Up to 24 blocks, and
// past two rounds, the waves still win.  Above, in the second round, they do where
// most pairs are short or all are alike, else the line balances better (over 570
// batches of 17 to 32 blocks, periodic ones among them, the rule's choice takes
// 0.80 of the time before there were pairs by waves, at worst 1.06 and 1.015): 2304
// pairs of 16-512 tokens, 17.3 blocks on average, 62.7 us on the line, 66.1 by
// waves; 2624 of 310 and 478 in turn, 25: 89.4, 97.5; but 2304 of 128, every
// sixteenth of 512, 9.5: 46.0, 37.3; 4112 of 512: 175.1, 170.4.  Past 32 blocks the
// streaming hides the line's cost and whole pairs only balance worse (2048 pairs
// of 512-2048 tokens 204.6 on the line, 220.6 by waves).
//
// Which wave takes which pair: pairs follow each other request by request, and
// the work groups XCD by XCD and CU by CU, both in powers of two.  With pair i on
// work group i mod launched in every run, a batch with a long request in every
// second, fourth or eighth place put all its long pairs on a part of the CUs (or
// XCDs).  So wave k's whole runs start k kPairSkew groups further on: its
// multiples by 0 to 3 lie about evenly in any 8, 16, ... 256 places.  120 requests,
// one of 476 tokens to seven of 18, 32 heads: 111 -> 64 us (line 60); 136, one of
// 403 to seven of 77, 16 heads: 61.6 -> 36.4 (line 40.0).  Batches without a
// period are 1 % slower on average (273 of them, 0.94 to 1.15), which is their
// luck with the other order.
constexpr int kPairSkew = 77;

// The order of the non-empty requests comes out of the in-register partition,
// eight per lane at most, so larger batches stay on the line, also where waves
// would be faster (500 requests of 100 tokens, 8 kv-heads, G = 4: 41.6 us, 62.7
// before there were pairs by waves).
constexpr int kShortRequests = 512;
constexpr uint32_t kShortPairUnits = 32;
constexpr uint32_t kLaterRoundUnits = 24;
constexpr uint32_t kMostlyShortUnits = 12;

__host__ __device__ inline bool waves_take_pairs(uint32_t units, uint32_t pairs, uint32_t longest, uint32_t launched)
{
    if (pairs <= launched || longest > kShortPairUnits ||
        (30 + 12 * longest) * (uint64_t)launched > 70 * (uint64_t)pairs + 5 * (uint64_t)units)
        return false;
    const uint32_t waves = 4 * launched;
    return pairs <= waves || pairs > 2 * waves || longest <= kLaterRoundUnits ||
           units <= (uint64_t)kMostlyShortUnits * pairs || 8 * (uint64_t)units > 7 * (uint64_t)longest * pairs;
}

}  // namespace apex
