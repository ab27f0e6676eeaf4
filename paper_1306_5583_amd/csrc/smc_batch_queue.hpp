// smc_batch_queue.hpp -- the work queue of the persistent batched step:
// item kinds, the dependency counters, and the host-side builder that lists
// one step's items so that every item comes after all the items it waits
// for (the condition that lets workgroups taking tickets in order always
// make progress).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace smc {

// Kinds of work item (see smc_persist.hip for what each does).
enum : int32_t {
    IT_PF_MOVE = 0,
    IT_GMM_REWEIGHT = 1,
    IT_FINAL = 2,
    IT_RESAMPLE = 3,
    IT_GMM_STEP = 4,
    IT_MONITOR = 5  // mixture sampler: path-sampling integrand after all its M items
};

struct QItem {
    int32_t kind;
    int32_t prob;
    int32_t tile;   // 1024-particle tile (A, R), Metropolis tile (M); 0 for F
    int32_t count;  // M: consecutive Metropolis tiles of the item; monitor: the
                    // problem's Metropolis tiles; 1 otherwise
};

// Per-problem completion counters (uint32 each, DEP_STRIDE per problem):
// DEP_A counts finished A tiles, DEP_F finished normalisations, DEP_R
// finished resampling tiles of mixture samplers, DEP_M the Metropolis tiles
// of their finished Metropolis items (an item adds its tile count, so the
// targets do not depend on the item size a schedule chooses).  At step t the
// targets are t * tiles (A, R), t (F) and t * Metropolis tiles (the
// monitor).
enum : int { DEP_A = 0, DEP_F = 1, DEP_R = 2, DEP_M = 3, DEP_STRIDE = 4 };
// Launch-wide words: the ticket counter and the abort flag.
enum : int { SYNC_TICKET = 0, SYNC_ABORT = 1, SYNC_WORDS = 64 };

// Mixture samplers of the persistent step have at most this many components.
constexpr int BATCH_MAX_K = 8;

// Orders of the queue the autotuner chooses between.
enum : int32_t {
    // mixture samplers' A, F, R items, then their Metropolis tiles with the
    // most expensive problems first and their monitors, then the tracking
    // filters' items (which fill the workgroups freed at the tail of the
    // Metropolis phase)
    ORDER_COST_FIRST = 0,
    // phase by phase in problem order: every A item, every F, every R, then
    // the Metropolis tiles and the monitors
    ORDER_PHASES = 1
};

struct QProblem {
    bool gmm;
    int64_t tiles;     // 1024-particle tiles
    int64_t mtiles;    // Metropolis tiles of 64 >> lsl particles
    double cost;       // relative cost of one of them
    int lsl = 0;       // 2^lsl lanes share a particle's data
};

// A step ends when its longest chain of items does, so a sampler whose
// 64-particle tiles each cost more than a workgroup slot gets on average has
// them split, 2^lsl lanes to a particle, while a lane keeps at least 64
// points per block (every item repeats the proposals in every lane and
// publishes its tile).  Twelve filters and four samplers of 1550 to 9430
// particles: 712 us a step with whole tiles, 431 split like this, 488 with
// half the cost and 32 points for the line; four filters and two samplers
// 1404 -> 313.
// A step index is as far as the 32-bit tickets and counters reach, and more
// items bring that nearer: a batch of so many steps that they could not index
// the last with its tiles split keeps them whole.
inline void split_tiles(std::vector<QProblem> &pr, const std::vector<int64_t> &n,
                        const std::vector<int64_t> &n_data, int64_t steps)
{
    const std::vector<QProblem> whole_tiles = pr;
    constexpr double SLOTS = 512;  // two workgroups a compute unit
    constexpr int WAVES = 4, MIN_POINTS = 64;
    double total = 0.0;
    for (const QProblem &p : pr)
        if (p.gmm)
            total += (double)p.mtiles * p.cost;
    for (size_t i = 0; i < pr.size(); ++i) {
        QProblem &p = pr[i];
        if (!p.gmm)
            continue;
        const double limit = total / SLOTS, whole = p.cost;
        while (p.lsl < 6 && p.cost > limit &&
               n_data[i] >= ((int64_t)WAVES * MIN_POINTS << (p.lsl + 1)))
            p.cost = whole / (double)(1 << ++p.lsl);
        const int64_t per = 64 >> p.lsl;
        p.mtiles = (n[i] + per - 1) / per;
    }
    // a step's tickets: its items and no more workgroups than items
    uint64_t items = 0, longest = 0;
    for (const QProblem &p : pr) {
        items += (uint64_t)(p.gmm ? 2 * p.tiles + 2 + p.mtiles : 2 * p.tiles + 1);
        longest = std::max(longest, (uint64_t)p.mtiles);
    }
    if ((uint64_t)steps > 0xFFFFFFFFull / std::max(2 * items, longest))
        pr = whole_tiles;
}

// One step's items.  `per_item` Metropolis tiles make one Metropolis item.
inline std::vector<QItem> build_queue(const std::vector<QProblem> &pr, int32_t order,
                                      int per_item)
{
    std::vector<QItem> q;
    const int np = (int)pr.size();
    std::vector<int> gm, pf;
    for (int p = 0; p < np; ++p)
        (pr[p].gmm ? gm : pf).push_back(p);
    auto phase_a = [&](const std::vector<int> &ps) {
        for (int p : ps)
            for (int64_t b = 0; b < pr[p].tiles; ++b)
                q.push_back(QItem{pr[p].gmm ? IT_GMM_REWEIGHT : IT_PF_MOVE, p, (int32_t)b, 1});
    };
    auto phase_f = [&](const std::vector<int> &ps) {
        for (int p : ps)
            q.push_back(QItem{IT_FINAL, p, 0, 1});
    };
    auto phase_r = [&](const std::vector<int> &ps) {
        for (int p : ps)
            for (int64_t b = 0; b < pr[p].tiles; ++b)
                q.push_back(QItem{IT_RESAMPLE, p, (int32_t)b, 1});
    };
    auto phase_m = [&](const std::vector<int> &ps) {
        for (int p : ps)
            for (int64_t b = 0; b < pr[p].mtiles; b += per_item)
                q.push_back(QItem{IT_GMM_STEP, p, (int32_t)b,
                                  (int32_t)std::min<int64_t>(per_item, pr[p].mtiles - b)});
    };
    auto phase_mon = [&](const std::vector<int> &ps) {
        for (int p : ps)
            q.push_back(QItem{IT_MONITOR, p, 0, (int32_t)pr[p].mtiles});
    };
    if (order == ORDER_PHASES) {
        std::vector<int> all(np);
        for (int p = 0; p < np; ++p)
            all[p] = p;
        phase_a(all);
        phase_f(all);
        phase_r(all);
        phase_m(gm);
        phase_mon(gm);
    } else {
        std::vector<int> byc = gm;
        std::stable_sort(byc.begin(), byc.end(),
                         [&](int a, int b) { return pr[a].cost > pr[b].cost; });
        phase_a(byc);
        phase_f(byc);
        phase_r(byc);
        phase_m(byc);
        phase_mon(byc);
        phase_a(pf);
        phase_f(pf);
        phase_r(pf);
    }
    return q;
}

}  // namespace smc
