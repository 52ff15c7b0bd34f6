// The planner of a prefetch step, for the kernels that plan.
#pragma once
#include "kvc_device.h"

namespace kvc {
namespace {

// Prefetch planner, Algorithm 1 of the paper without the token predictor: for every (layer, sequence) the k
// predicted logical blocks in order -- translate through the block table (TranslateAddress), skip what is already
// in L1 or in the L2 prefetch buffer (the residency test), otherwise claim a slot of the half being filled and
// list the pool block for the decode launch (IssueDMA).
//
// KMAX lanes per (layer, sequence), lane j holding prediction j and slot j of both halves.  The planner is a
// short chain of memory trips and little else, so every value is read by one coalesced load and nothing is read
// behind a branch (indices beyond their range read entry 0 and are sorted out afterwards): two trips, predictions
// and tags first, then the table entries.  The walk over the predictions then runs on ballots.  (With a thread per
// (layer, sequence) that translated its k predictions behind branches the planner took 10.5 us for 64 sequences of
// 8 -- as long as the decode launch it plans.)
//
// plan_row: one row per KMAX lanes, layer l and sequence sq (in range where `there`); -> what becomes of this lane's slot.
// plan_write puts it down (-> whether the slot is fetched).  tag_bits: upper bits of the tag of the row's first slot that are
// not the tag's (see k_prefetch_decompress).
struct PlanSlot {
    bool live;           // there is such a slot
    int64_t at;          // its place in loc and fetch,
    int64_t tag_at;      // and in the tags
    int32_t loc, fetch;  // what they become,
    int32_t tag, had;    // and the tag; what that was
};
template <int KMAX>
__device__ __forceinline__ PlanSlot plan_row(const PlanArgs& a, bool there, int32_t l, int32_t sq, int tag_bits = 0) {
    const int lane = lane_id();
    const int j = lane % KMAX;
    const int k = a.k;
    const bool live = there && j < k;
    const int64_t n_slots = (int64_t)a.n_layers * a.n_seq * k;
    const int64_t base = ((int64_t)l * a.n_seq + sq) * k;
    const int64_t fill0 = (int64_t)a.fill_half * n_slots + base, other0 = (int64_t)(1 - a.fill_half) * n_slots + base;

    int32_t lb = -1, t_fill = -1, t_other = -1, l1 = INT32_MAX;
    if (live) {
        lb = a.pred[(int64_t)sq * k + j];
        t_fill = a.tags[fill0 + j];
        t_other = a.tags[other0 + j];
        if (a.l1_first) l1 = a.l1_first[sq];
    }
    if (tag_bits != 0 && j == 0) t_fill = (int32_t)((uint32_t)t_fill << tag_bits) >> tag_bits;
    const int32_t held = t_fill;
    int32_t e = -1;
    if (live) e = a.block_table[(int64_t)sq * a.max_blocks + (lb >= 0 && lb < a.max_blocks ? lb : 0)];
    // the pool block (>= 0), -1 for "no block", -2 for "in L1" (held in the GPU-local cache)
    const bool in_l1 = a.l1_first && lb >= l1;
    const bool bad = live && (lb >= a.max_blocks || (lb >= 0 && !in_l1 && e >= a.pool_blocks_per_layer));
    int32_t want = -1;
    if (live && lb >= 0 && lb < a.max_blocks) want = in_l1 ? -2 : (e < 0 || bad) ? -1 : (int32_t)((int64_t)l * a.pool_blocks_per_layer + e);

    // this row's part of a ballot, bit j2 = lane j2 of the row
    // (the half of the ballot by masks: of a selection the compiler may make a 64-bit shift by a lane's own amount)
    const int lane0 = lane - j;
    const uint32_t upper = 0u - (uint32_t)(lane >> 5);
    auto of_row = [&](bool c) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(c);
        const uint32_t half = ((uint32_t)m & ~upper) | ((uint32_t)(m >> 32) & upper);
        return KMAX == 32 ? half : (half >> (lane0 & 31)) & ((1u << (KMAX & 31)) - 1u);
    };
    auto of_row_lane = [&](int32_t v, int j2) { return __builtin_amdgcn_ds_bpermute((lane0 + j2) << 2, v); };
    int32_t wants[KMAX];
#pragma unroll
    for (int j2 = 0; j2 < KMAX; ++j2) wants[j2] = of_row_lane(want, j2);
    int32_t fetch = -1, loc = want == -2 ? -2 : -1;
    if (a.policy == 0) {
        // Algorithm 1 as printed: prediction jj owns slot jj of the half being filled
#pragma unroll
        for (int jj = 0; jj < KMAX; ++jj) {
            const int32_t pb = wants[jj];
            const uint32_t other = of_row(t_other == pb), settled = of_row(t_fill == pb) & ((1u << jj) - 1u);  // slots already settled in this step
            if (j == jj && pb >= 0) {  // lowest matching slot wins
                loc = (int32_t)(other ? other0 + __builtin_ctz(other) : settled ? fill0 + __builtin_ctz(settled) : fill0 + jj);
                if (!other && !settled && t_fill != pb) t_fill = fetch = pb;
            }
        }
    } else {
        // Slot reuse: blocks wanted by this step stay where they are; a block that is in neither half
        // takes the lowest slot whose content this step does not want.
        bool wanted = false, dup = false;  // a slot is kept if it is the first one holding a wanted block
#pragma unroll
        for (int j2 = 0; j2 < KMAX; ++j2) {
            const int32_t t = of_row_lane(t_fill, j2);  // (read by every lane, outside any condition)
            wanted = wanted || wants[j2] == t_fill;
            dup = dup || (t == t_fill && j2 < j);
        }
        bool keep = (t_fill >= 0 && wanted && !dup) || j >= k;  // slots beyond k do not exist: never claimable
#pragma unroll
        for (int jj = 0; jj < KMAX; ++jj) {
            const int32_t pb = wants[jj];
            const uint32_t other = of_row(t_other == pb), held = of_row(keep && j < k && t_fill == pb), unwanted = of_row(!keep);
            if (pb >= 0) {
                const int slot = __builtin_ctz(held ? held : unwanted ? unwanted : 1u);
                if (j == jj) loc = (int32_t)(other ? other0 + __builtin_ctz(other) : fill0 + slot);
                if (!other && !held && j == slot) {  // claim it: it now holds a wanted block
                    keep = true;
                    t_fill = fetch = pb;
                }
            }
        }
    }
    if (bad) atomicOr(&a.st->status, KVC_ST_BAD_INDEX);
    return PlanSlot{live, base + j, fill0 + j, loc, fetch, t_fill, held};
}
__device__ __forceinline__ bool plan_write(const PlanArgs& a, const PlanSlot& r) {
    if (r.live) {
        a.loc[r.at] = r.loc;
        a.fetch[r.at] = r.fetch;
        if (r.fetch >= 0) a.tags[r.tag_at] = r.tag;
    }
    return r.live && r.fetch >= 0;
}

}  // namespace
}  // namespace kvc
