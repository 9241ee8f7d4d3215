// Host bookkeeping of the batched form, free of HIP so that the library and a
// sanitizer build on the CPU compile the same code: the split of a class's
// work into tiles, the per-integrand ranges of block partials, the number of
// shares of a class and the spread of the classes over streams; and the times
// by which launch geometries are compared.
#pragma once

#include <stdint.h>

#include <math.h>

#include <algorithm>
#include <utility>
#include <vector>

namespace mcubes {

// Work items [w_begin, w_end) of integrand `item`; its (sum S_c, sum var_c)
// go to partials[2 partial], [2 partial + 1].
struct BatchTile {
    uint32_t item, w_begin, w_end, partial;
};

// Splits the samples of the class's integrands (in the order of `items`;
// integrand i has m[i] cubes of p[i] samples) into `shares` equal contiguous
// shares, a share ending inside an integrand at a cube boundary, and appends
// one tile per (share, integrand) pair with work.  A tile's partial slot is
// its index in `tiles`, so the tiles of an integrand are consecutive.
inline void split_tiles(const std::vector<int> &items, const int64_t *m, const int64_t *p,
                        int shares, std::vector<BatchTile> &tiles) {
    const int k = (int)items.size();
    std::vector<int64_t> off(k + 1, 0);
    for (int q = 0; q < k; ++q) off[q + 1] = off[q] + m[items[q]] * p[items[q]];
    const int64_t S = off[k];
    // position of sample offset T: (item slot, first cube starting at or after T)
    auto position = [&](int64_t T) {
        const int q = (int)(std::upper_bound(off.begin(), off.end(), T) - off.begin()) - 1;
        if (q >= k) return std::make_pair(k, (int64_t)0);
        const int i = items[q];
        const int64_t w = (T - off[q] + p[i] - 1) / p[i];
        if (w >= m[i]) return std::make_pair(q + 1, (int64_t)0);
        return std::make_pair(q, w);
    };
    auto lo = position(0);
    for (int b = 0; b < shares; ++b) {
        const int64_t Tb = (int64_t)(((unsigned __int128)S * (uint64_t)(b + 1)) / (uint64_t)shares);
        const auto hi = position(Tb);
        for (int q = lo.first; q <= hi.first && q < k; ++q) {
            const int64_t wb = q == lo.first ? lo.second : 0;
            const int64_t we = q == hi.first ? hi.second : m[items[q]];
            if (we > wb) {
                BatchTile t;
                t.item = (uint32_t)items[q];
                t.w_begin = (uint32_t)wb;
                t.w_end = (uint32_t)we;
                t.partial = (uint32_t)tiles.size();
                tiles.push_back(t);
            }
        }
        lo = hi;
    }
}

// [begin[i], end[i]) = the partial slots of integrand i's tiles (0, 0 for an
// integrand without tiles).  Returns the index of the first tile whose
// integrand's tiles are not consecutive, or -1.
inline int64_t part_ranges(const std::vector<BatchTile> &tiles, int n, uint32_t *begin,
                           uint32_t *end) {
    for (int i = 0; i < n; ++i) begin[i] = end[i] = 0;
    std::vector<char> seen(n, 0);
    for (size_t t = 0; t < tiles.size(); ++t) {
        const uint32_t i = tiles[t].item;
        if (!seen[i]) {
            seen[i] = 1;
            begin[i] = tiles[t].partial;
        } else if (end[i] != tiles[t].partial) {
            return (int64_t)t;
        }
        end[i] = tiles[t].partial + 1;
    }
    return -1;
}

// Shares (workgroups before the split at integrand boundaries) of a class of
// `cubes` cubes: `want` if positive, else one per `block` cubes but at most
// `per_slot` per workgroup slot of the device (`resident` slots); never more
// than `max_shares` or the cubes, never fewer than one.  0 if no workgroup
// of the class fits (resident < 1).
inline int class_shares(int64_t cubes, int block, int resident, int want, int64_t per_slot,
                        int64_t max_shares) {
    if (resident < 1) return 0;
    int64_t shares = want;
    if (shares <= 0) {
        shares = (cubes + block - 1) / block;
        if (shares > per_slot * resident) shares = per_slot * resident;
    }
    if (shares > max_shares) shares = max_shares;
    if (shares > cubes) shares = cubes;
    if (shares < 1) shares = 1;
    return (int)shares;
}

// Time in us that a SIMD takes for 64 cubes of p samples, one per lane
// (measured over the dimensions; a wave alone takes four times as long).
inline double cube_us(int dim, double p) { return 0.5 * p * (0.1 + 0.11 * dim); }

// The time of the histogram that a workgroup adds to the global bins at its
// end: adds to one address go one by one, 20 ns each, whichever workgroups
// they come from.
constexpr double kFlushUs = 0.02;

// Estimated time in us of a class's V-Sample split into `shares`: `items`
// integrands of `cubes` cubes and `samples` samples in all, the largest of
// `largest` cubes (0: not known), `resident` workgroups of `block` threads at
// once on `cus` CUs.  A thread takes its whole cubes of a tile, a SIMD its waves
// in turn, two at least in the time of two; the tiles take the chip's slots
// round by round, the last ones spread over the CUs.  Uneven progress costs an
// eighth of a single round (0.12) and less of more of them, each of which fills
// its tables again, 2 + 0.3 dim us, and 5 ns per tile.  A workgroup's adds to
// the global bins wait for those of the same integrand only, and in several
// rounds for the others' sampling: they count where they outweigh it.
//
// `alone` is the class's part of all the batch's samples: where others' tiles
// take over the slots that uneven progress leaves, it costs that much less (512
// integrands of 1e6 to 1e7 samples, some 60 classes: 36.0 ms for four iterations,
// 36.7 without this).
//
// Over 72 classes of one family (2-D to 8-D, 1 to 64 integrands, 1e6 to 1e9
// samples in all), each timed at 14 numbers of shares, the split chosen by this
// is 2% slower than the fastest in the geometric mean; taken without the uneven
// progress and with all adds one after the other, which kept the large ones at
// one round, 7%.
inline double tiles_us(int dim, int64_t items, int64_t cubes, int64_t samples, bool bins,
                       int block, int64_t resident, int cus, int64_t shares, int64_t largest = 0,
                       double alone = 1.0) {
    const double wave = cube_us(dim, (double)samples / (double)cubes);
    const int64_t tiles = shares + items - 1;
    int64_t each = (cubes + shares - 1) / shares;
    if (largest > 0) each = std::min(each, largest);
    each = (each + block - 1) / block;
    const int64_t per_cu = std::max<int64_t>(1, resident / cus);
    const auto waves = [&](int64_t blocks) { return std::max((double)blocks * block / 256.0, 2.0); };
    const int64_t last = tiles % resident;
    const double turns = (double)(tiles / resident) * waves(per_cu) +
                         (last ? waves((last + cus - 1) / cus) : 0.0);
    const double rounds = ceil((double)tiles / (double)resident);
    const double sampling = (double)each * turns * wave *
                            (1.0 + 0.12 * alone * std::min(1.0, (double)resident / (double)tiles));
    const double flush = bins ? kFlushUs * (double)tiles / (double)items : 0.0;
    return (2.0 + 0.3 * dim) * rounds + 0.005 * (double)tiles +
           (tiles <= resident ? sampling + flush : std::max(sampling, flush));
}

// Default shares of a class, at most `most`: the cheapest by tiles_us of the
// splits that give every thread 1 to 64 whole cubes in one round and of those
// that fill 1 .. 8 rounds, with the boundaries of integrands or without.  Small
// tiles balance the load, but every one of them fills its tables and adds its
// histogram.  By this rule, and with 8 shares per slot whatever the work: 48
// integrands of 1e5 to 1e7 samples in 2-D to 8-D 2.2 to 2.8 ms for four
// iterations (six draws) and 9 to 13; 512 of 1e6 to 1e7 35 to 36 and 54 to 56;
// eight of 5e7 of one family, three iterations, 2-D to 8-D, 2.7 to 6.3 and 2.9
// to 6.4.
inline int64_t default_shares(int dim, int64_t items, int64_t cubes, int64_t samples, bool bins,
                              int block, int64_t resident, int cus, int64_t most,
                              int64_t largest = 0, double alone = 1.0) {
    int64_t best = 1;
    double best_us = -1.0;
    const auto offer = [&](int64_t shares) {
        shares = std::max<int64_t>(1, std::min(shares, most));
        const double us =
            tiles_us(dim, items, cubes, samples, bins, block, resident, cus, shares, largest, alone);
        if (best_us < 0.0 || us < best_us) {
            best = shares;
            best_us = us;
        }
    };
    for (int64_t each = 1; each <= 64; ++each) {
        const int64_t shares = (cubes + each * block - 1) / (each * block);
        if (shares + items - 1 <= resident) offer(shares);
    }
    for (int64_t rounds = 1; rounds <= 8; ++rounds) {
        offer(rounds * resident - (items - 1));
        // where the integrands outnumber the slots, their boundaries make the
        // tiles whatever the shares, and the shares are to cut the largest
        offer(rounds * resident);
    }
    return best;
}

// Spreads classes of the given costs over at most `streams` branches, longest
// first onto the least loaded branch.  branch[k] receives class k's branch;
// returns the number of branches, min(streams, classes) but at least 1 (a
// branch never goes without work).
inline int assign_branches(const std::vector<double> &cost, int streams,
                           std::vector<int> &branch) {
    std::vector<std::pair<double, int>> order;
    for (int k = 0; k < (int)cost.size(); ++k) order.push_back({cost[k], k});
    std::sort(order.begin(), order.end(), [](const std::pair<double, int> &a,
                                             const std::pair<double, int> &b) {
        return a.first > b.first || (a.first == b.first && a.second < b.second);
    });
    const int branches = std::max(1, std::min(streams, (int)cost.size()));
    std::vector<double> load(branches, 0.0);
    branch.assign(cost.size(), 0);
    for (const auto &ck : order) {
        const int br = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        branch[ck.second] = br;
        load[br] += ck.first;
    }
    return branches;
}

}  // namespace mcubes
