// hsga_layout.hpp -- a surface's layout worked out by one wavefront from the
// site rule's constant-time tables (Distributed Phylogenetic Tracking:
// deposit times follow from the site index and the generation count).
#pragma once

#include "hsga_rule.hpp"

namespace hsga {

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

// rule_item_at for a tilted sub-surface, its site `site` (>= m: none) per
// lane, after U items (the same U in all 64 lanes).  The epoch's events are
// loaded 64 at a time, one per lane, which also works out the item that the
// event's chain leaves behind; walking them is then two readlanes and four
// selects each, where a walk by every lane for itself waits for three loads
// per event (MRCA prepare at 32 tilted sites 13.3 -> 9.5 us, the general
// route's 4,096 layouts 11.2 -> 9.7 us).
__device__ __forceinline__ uint32_t tilted_item_at_wave(const RuleTable& R, uint64_t U,
                                                        uint32_t site) {
    const uint32_t m = R.m;
    if (U <= m) return site < U && site < m ? site : kRuleEmptyItem;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t u = U - 1;                        // the newest item
    const uint32_t e = rule_bitlen(u + 1) - R.first;
    const uint32_t r = R.r[e];
    uint32_t key = site < m ? R.chain_of[e][site] : kRuleNoSite;
    uint32_t held = site < m ? R.layout0[e][site] : kRuleEmptyItem;
    const uint32_t end = R.evt_begin[e + 1];
    for (uint32_t i0 = R.evt_begin[e]; i0 < end; i0 += 64) {
        uint32_t ue = kRuleEmptyItem, move = 0, left = 0;
        if (i0 + lane < end) {
            ue = R.evt_u[i0 + lane];
            move = R.evt_key[i0 + lane] | (uint32_t)R.evt_site[i0 + lane] << 8;
            const uint32_t h = (uint32_t)__builtin_ctzll((uint64_t)ue + 1);
            const uint64_t c = ((uint64_t)ue + 1) >> (h + 1);
            left = (uint32_t)(((2 * (c - r) + 1) << h) - 1);
        }
        // events are in time order: those up to u are the first lanes
        const uint32_t n = (uint32_t)__popcll(__ballot(i0 + lane < end && ue <= u));
        for (uint32_t j = 0; j < n; ++j) {
            const uint32_t mv = lane_value(move, j), lv = lane_value(left, j);
            const uint32_t k = mv & 0xffu, s = mv >> 8;
            if (key == k && site != s) {
                key = kRuleNoSite;
                held = lv;
            }
            if (site == s) key = k;
        }
        if (n < 64) break;
    }
    if (key == kRuleNoSite) return site < m ? held : kRuleEmptyItem;
    const uint32_t h = key / r, q = key % r;
    const uint64_t cmax = ((U >> h) - 1) / 2;        // newest level-h index below U
    const uint64_t c = cmax - (cmax + r - q) % r;
    return (uint32_t)(((2 * c + 1) << h) - 1);
}

// scheme_item_at(rules, kind, S, tau, lane) for each lane of a wavefront.
// All 64 lanes call it with the same tau.
__device__ __forceinline__ uint32_t scheme_layout_wave(const RuleTable* rules, uint32_t kind,
                                                       uint32_t S, uint64_t tau) {
    const uint32_t lane = threadIdx.x & 63u;
    if (kind == 0) return rule_item_at(rules[0], tau, lane);
    if (kind == 1) return tilted_item_at_wave(rules[0], tau, lane);
    const uint32_t h = S >> 1;
    const uint32_t lo = rule_item_at(rules[0], (tau + 1) >> 1, lane);
    const uint32_t hi = tilted_item_at_wave(rules[1], tau >> 1, lane - h);
    if (lane < h) return lo == kRuleEmptyItem ? lo : 2 * lo;
    return lane < S && hi != kRuleEmptyItem ? 2 * hi + 1 : kRuleEmptyItem;
}

}  // namespace hsga
