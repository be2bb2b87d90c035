// Members per VB work unit when large units are split over several
// workgroups that meet at a device-scope barrier after every colour class.
// Host code only (no HIP), so that the allocation can be checked on the CPU.
//
// A unit's cost per sweep is weighed as n (10 + chains): its graph (adjacency
// stream and spin words per vertex) dominates and is shared by its chains,
// a chain adding about a tenth of it (whole units, us per sweep on MI355X:
// one chain of 985767 spins 560, six chains of 65536 spins 67).  Splitting
// shortens a launch only if no unit left whole outlasts the split ones, so
// the automatic plan splits the units above twice a CU's share of the cost
// only when all of them get at least two members, or else the largest
// leading group of them with three times the cost of every unit left whole, or
// else as many of the costliest as there is room for, in two each, if that shortens
// the longest launch by a sixth and more (sizes spread over decades: 256 graphs of
// 2^10 to 2^20 spins with 2 replicas 444 us per sweep, 614 whole).
// Their members are shared out in proportion to cost, so that every member
// carries about the same part of a sweep, with a floor per member that rises
// with the number of split units: members of many split units meet at their
// barriers at the same time, and thin members then wait more than they
// compute.  Measured, us per sweep: graphs of 65536 spins with 6 chains,
// 1 graph 13 members 34 (8: 37, whole: 67), 4 graphs 8 members 44 (4: 48), 16
// graphs 4 members 57 (6: 68, 8: 82), 64 graphs whole 69 (2 members: 73); one
// request of 985767 spins with 2 chains (two units), 32 members each 66 (16: 76,
// 64: 75, whole: 560).  Sizes below about 2^15 are split although they are faster
// whole by now (one graph of 16384 spins, 6 chains, 26 against 21): the floors are
// older than the sweep loop.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <numeric>
#include <vector>

namespace sg {

// the least cost a member carries with at most two, at most eight and more
// split units (about 5, 9 and 17 us of a sweep on MI355X), and the most
// members of one unit
constexpr int64_t kSplitMemberCostFew = 75000;
constexpr int64_t kSplitMemberCostSome = 130000;
constexpr int64_t kSplitMemberCostMany = 260000;
constexpr int kSplitMaxMembers = 32;
// what a member of a unit split in two adds to half its cost (one chain of 10^6 spins,
// us per sweep: whole 560, two members 374 for one such unit and 436 for 32 at once)
constexpr int64_t kSplitPairCost = 2500000;

// Blocks of 64 positions in the chunks of a split unit with `slots` chain slots, whose
// members have `waves` wavefronts together: two, whose latencies overlap, or one where
// two would leave wavefronts without a chunk, or with half the work of others, in the
// largest colour class (`largest` positions).  Measured with 8 slots, us per sweep with
// one / two blocks and the chunks of two per wavefront: graphs of 65536 spins, 6 chains,
// 13 members each (0.8) 34.4 / 35.3, 8 members (1.4) 42.6 / 44.6, 4 (2.8) 60.6 / 57.0;
// of 131072 spins, 28 (0.8) 35.0 / 35.8, 16 (1.4) 56.1 / 59.0, 4 (5.6) 85 / 77.  With
// fewer slots a chunk of two is as quick as one of one (2 chains, 0.8: 29.1 / 28.6).
inline int split_chunk_blocks(int slots, int64_t largest, int64_t waves)
{
    return slots == 8 && (largest + 127) / 128 < 2 * waves ? 1 : 2;
}

struct SplitUnit {
    int64_t cost;        // n (10 + chains)
    bool resident;       // adjacency kept in LDS: never split
    int64_t chunk_cap;   // most members with two blocks of 64 positions per wavefront in the largest class
};

// Members of every unit (1: whole) for `budget` workgroups of split members
// and a CU's share `share` of the batch's cost.  forced: 0 automatic, 1
// never split, k >= 2 every non-resident unit that has the blocks for k
// members, within the budget.  Returns the members used (those of split
// units).
inline int plan_split(const std::vector<SplitUnit>& units, int64_t share, int budget, int forced,
                      std::vector<int>& members)
{
    members.assign(units.size(), 1);
    if (forced == 1 || budget < 2) return 0;
    std::vector<size_t> by_cost(units.size());
    std::iota(by_cost.begin(), by_cost.end(), (size_t)0);
    std::stable_sort(by_cost.begin(), by_cost.end(),
                     [&](size_t a, size_t b) { return units[a].cost > units[b].cost; });
    size_t n_auto = 0;
    if (forced == 0) {
        size_t cand = 0;
        while (cand < by_cost.size() && !units[by_cost[cand]].resident && units[by_cost[cand]].cost >= 2 * share)
            ++cand;
        for (size_t m = std::min(cand, (size_t)(budget / 2)); m >= 1; --m) {
            const int64_t rest = by_cost.size() > m ? units[by_cost[m]].cost : 0;
            if (m == cand || units[by_cost[m - 1]].cost >= 3 * rest) {
                n_auto = m;
                break;
            }
        }
    }
    // no such group: the costliest units in two, when that shortens the longest
    // launch by a sixth and more
    if (forced == 0 && n_auto == 0 && by_cost.size() > 1) {
        size_t cand = 0;
        while (cand < by_cost.size() && !units[by_cost[cand]].resident && units[by_cost[cand]].cost >= 2 * share &&
               units[by_cost[cand]].chunk_cap >= 2)
            ++cand;
        const size_t m = std::min(cand, (size_t)(budget / 2));
        if (m >= 1) {
            const int64_t most = units[by_cost[0]].cost;
            const int64_t rest = by_cost.size() > m ? units[by_cost[m]].cost : 0;
            if (6 * std::max(rest, most / 2 + kSplitPairCost) <= 5 * most) {
                members.assign(units.size(), 1);
                for (size_t r = 0; r < m; ++r) members[by_cost[r]] = 2;
                return 2 * (int)m;
            }
        }
    }
    int64_t split_cost = 0;
    for (size_t r = 0; r < n_auto; ++r) split_cost += units[by_cost[r]].cost;
    const int64_t floor_cost = n_auto <= 2 ? kSplitMemberCostFew : n_auto <= 8 ? kSplitMemberCostSome
                                                                                : kSplitMemberCostMany;
    const int64_t per_member = std::max<int64_t>({share, (split_cost + budget - 1) / budget, floor_cost});
    int used = 0;
    for (size_t r = 0; r < by_cost.size(); ++r) {
        const SplitUnit& u = units[by_cost[r]];
        if (u.resident || (forced == 0 && r >= n_auto)) continue;
        int64_t want = forced >= 2 ? forced
                                   : std::min<int64_t>(kSplitMaxMembers, (u.cost + per_member / 2) / per_member);
        want = std::min<int64_t>(want, std::min<int64_t>(u.chunk_cap, budget));
        if (want >= 2) {
            members[by_cost[r]] = (int)want;
            budget -= (int)want;
            used += (int)want;
        }
    }
    return used;
}

}  // namespace sg
