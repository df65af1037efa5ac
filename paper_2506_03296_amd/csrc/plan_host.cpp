// plan_host.cpp -- host mirrors of the work partition (apex_decode_plan_host
// and apex_decode_plan_pairs_host in include/apex_decode.h): the same plan_policy.h arithmetic the kernel's
// prologue runs, over host context_lens, for inspection and tests.  Plain
// host C++ (no HIP kernels), so it also builds with g++ under sanitizers.
#include <stdint.h>

#include "apex_decode.h"
#include "plan_policy.h"
#include "status.h"

using apex::fail;

extern "C" {

int apex_decode_plan_host(const int32_t* context_lens, int B, int Hkv, int block_size,
                          int launched_workers, int forced, int cus, int32_t* contributors_out,
                          int64_t* units_out, int64_t* active_out, int64_t* partials_out)
{
    apex::clear_error();
    if (B < 0 || Hkv <= 0 || launched_workers <= 0 || cus < 0)
        return fail(APEX_ERR_INVALID_ARG, "bad partition arguments");
    if (B > 0 && !context_lens) return fail(APEX_ERR_INVALID_ARG, "context_lens is NULL");
    if (block_size != apex::kBlockSize)
        return fail(APEX_ERR_UNSUPPORTED, "block_size %d unsupported (only 16)", block_size);
    int64_t blocks = 0, nonempty = 0;
    for (int b = 0; b < B; ++b) {
        blocks += apex::blocks_of(context_lens[b], block_size);
        nonempty += context_lens[b] > 0;
    }
    const int64_t units = blocks * Hkv;
    const int64_t pairs = nonempty * Hkv;
    const int64_t W = apex::active_workers(units, launched_workers,
                                           forced ? 1 : apex::kMinUnitsPerWorker, pairs,
                                           forced ? 0 : cus);
    const int64_t K = forced ? 0 : apex::kSegmentCostUnits;
    const int64_t V = units + K * pairs;
    int64_t partials = 0, pre = 0, pp = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t nb = apex::blocks_of(context_lens[b], block_size);
        for (int g = 0; g < Hkv; ++g) {
            int64_t n = 0;
            if (nb > 0) {
                const int64_t vf = apex::first_block_position(pre * Hkv + (int64_t)g * nb, pp * Hkv + g, K);
                n = apex::worker_of(vf + nb - 1, V, W) - apex::worker_of(vf, V, W) + 1;
                if (n > 1) partials += n;
            }
            if (contributors_out) contributors_out[(size_t)b * Hkv + g] = (int32_t)n;
        }
        pre += nb;
        pp += nb > 0;
    }
    if (units_out) *units_out = units;
    if (active_out) *active_out = units > 0 ? W : 0;
    if (partials_out) *partials_out = partials;
    return APEX_OK;
}

int apex_decode_plan_pairs_host(const int32_t* context_lens, int B, int Hq, int Hkv, int block_size,
                                int launched_workers, int cus, int32_t* parts_out, int32_t* part_units_out,
                                int64_t* active_out)
{
    apex::clear_error();
    if (B < 0 || Hkv <= 0 || Hq <= 0 || Hq % Hkv != 0 || launched_workers <= 0 || cus < 0)
        return fail(APEX_ERR_INVALID_ARG, "bad partition arguments");
    if (B > 0 && !context_lens) return fail(APEX_ERR_INVALID_ARG, "context_lens is NULL");
    if (block_size != apex::kBlockSize)
        return fail(APEX_ERR_UNSUPPORTED, "block_size %d unsupported (only 16)", block_size);
    uint64_t blocks = 0, nonempty = 0, longest = 0;
    for (int b = 0; b < B; ++b) {
        const uint64_t nb = (uint64_t)apex::blocks_of(context_lens[b], block_size);
        blocks += nb;
        nonempty += nb > 0;
        longest = nb > longest ? nb : longest;
    }
    // the line's positions, whose 32-bit arithmetic the kernel's rule shares
    const uint64_t units = blocks * (uint64_t)Hkv, pairs = nonempty * (uint64_t)Hkv;
    const uint64_t V = units + apex::kSegmentCostUnits * pairs;
    uint32_t floor_units = 0;
    bool by_waves = false;
    if (cus > 0 && (V >> 32) == 0 && V * ((uint64_t)launched_workers + 1) <= 0xffffffffull) {
        if (B <= apex::kPairCutRequests)
            floor_units = apex::pair_cut_floor((uint32_t)units, (uint32_t)pairs, (uint32_t)longest, (uint32_t)cus,
                                               (uint32_t)launched_workers);
        by_waves = B <= apex::kShortRequests && floor_units == 0 &&
                   apex::waves_take_pairs((uint32_t)units, (uint32_t)pairs, (uint32_t)longest, (uint32_t)launched_workers);
    }
    if (by_waves) floor_units = (uint32_t)longest;   // every pair is one part
    int64_t active = 0;
    for (int b = 0; b < B; ++b) {
        const uint32_t nb = (uint32_t)apex::blocks_of(context_lens[b], block_size);
        uint32_t T = 0, parts = 0;
        if (floor_units > 0 && nb > 0) {
            T = floor_units < longest ? apex::pair_part_units(nb, floor_units, (uint32_t)(Hq / Hkv)) : nb;
            parts = (nb + T - 1) / T;
        }
        active += (int64_t)parts * Hkv;
        if (parts_out) parts_out[b] = (int32_t)parts;
        if (part_units_out) part_units_out[b] = (int32_t)T;
    }
    if (by_waves) active = launched_workers;   // pairs > launched_workers
    if (active_out) *active_out = active;
    return APEX_OK;
}

}  // extern "C"
