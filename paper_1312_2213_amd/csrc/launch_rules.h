// launch_rules.h -- how work is cut and which kernels take it, as plain
// arithmetic with no HIP dependency: the kernels and the runtime include it,
// and a check program builds it on its own (with sanitizers).
#pragma once

#include <math.h>
#include <stdint.h>

namespace muca {

// Calls f(done, n) for consecutive segments of n <= at_most of `total` sweeps,
// done sweeps behind each.  The count is unsigned: total + at_most may lie
// beyond 2^31, not beyond 2^32.
template <class F>
__attribute__((always_inline)) constexpr void for_segments(int32_t total, int32_t at_most, F f)
{
    for (uint32_t done = 0; done < (uint32_t)total; done += (uint32_t)at_most) {
        const uint32_t left = (uint32_t)total - done;
        f((int32_t)done, (int32_t)(left < (uint32_t)at_most ? left : (uint32_t)at_most));
    }
}

// ---------------------------------------------------------------------------
// One wavefront per chain, or 1 to 4 lanes per chain
// ---------------------------------------------------------------------------
// How well the log weights of a run are known: the mean, over the links
// between bins that its iterations have measured, of the statistical error
// P^-1/2 of a link's ln ratio (P, the link's accumulated statistics, is that
// ratio's inverse variance), at most 1 each.  0 for weights without
// measurements: flat ones, or a caller's.  At most 1024 links, evenly spaced,
// are looked at (all 8193 of Potts L = 64: 14 to 34 us, these 2 to 4).
inline double weights_noise(int n, const double *P)
{
    double sum = 0.0;
    int links = 0;
    for (int b = 0, step = (n + 1023) / 1024; b < n; b += step)
        if (P[b] > 0.0) {
            sum += P[b] > 1.0 ? 1.0 / sqrt(P[b]) : 1.0;
            ++links;
        }
    return links ? sum / links : 0.0;
}

// A tile's passes grow with the noise of the weights (its thresholds then
// differ from bin to bin), the time of 1 to 4 lanes per chain does not: the
// two meet at fewer chains during the first iterations.  The classes of noise
// by which the lines below are drawn: 0 settled (from the sixth to tenth
// iteration of some ten to forty sweeps, the second of a few hundred), 1 in
// between, 2 the first iterations.  Thresholds of multimagnetic runs are set
// by beta as much as by the weights: their passes hardly change.
enum { kSettled = 0, kBetween = 1, kRough = 2 };
inline int weights_class(int model, double noise) // MUCA_ISING, MUCA_POTTS, MUCA_MUMA
{
    if (model == 0)
        return noise < 0.05 ? kSettled : noise < 0.075 ? kBetween : kRough;
    return model == 1 && noise >= 0.09 ? kRough : kSettled;
}

// Most chains of a run that takes the one-wavefront-per-chain kernel by
// default.  Its time goes by rounds of 4096 chains, sixteen on each of 256
// CUs: a table of 82 KB or more leaves room for one workgroup per CU, and so
// do the 100 scalar registers of 1024 threads.  That of 1 to 4 lanes per
// chain hardly changes up to 16384 chains, where four lanes give every SIMD a
// wavefront.  So the lines lie at ends of rounds, or where a round begun
// costs less than a full one.  Measured, time of the best of 1, 2 and 4 lanes
// over that of one wavefront per chain, by the chains of a run (10 to 40
// sweeps per iteration):
//         second iteration           settled weights
//           4096  4160  8192         4160  6144  8192  8256 10240 12288
//   Ising
//     64    2.07  1.15  0.92         1.82  1.79  1.55  1.25  1.12  1.02
//     48    1.54  0.90  0.85         1.42  1.18  1.07  0.97  0.88  0.86
//     32    1.29  0.85  0.93         1.32  1.24  1.18  0.93  0.91  0.82
//     24    1.43  0.92  0.75         1.26  1.07  1.09  0.89  0.84  0.82
//     16    1.27  0.91  0.97         1.39  1.31  1.28  0.99  0.94  0.93
//     8     1.33  1.04  0.97         1.41  1.19  1.24  1.09  0.96  0.97
//   Potts
//     48    2.43  1.37  1.22         1.79  1.75  1.71  1.24  1.18  1.13
//     32    1.62  0.94  1.03         1.55  1.43  1.36  1.03  0.98  0.92
//     24    1.63  0.94  0.75         1.21  1.07  1.07  0.82  0.79  0.71
//     16    1.26  0.93  0.84         1.56  1.39  1.38  1.09  1.03  0.98
//     8     1.41  1.00  0.93         1.32  1.18  1.14  1.00  0.88  0.87
//   Ising in between, one iteration each: L = 64 1.07 to 1.12 at 6144 and
//     0.93 to 1.32 at 8192, L = 48 0.84 to 1.26 at 8192, L = 32 0.97 to 1.13
//     at 8192, L = 24 1.03 to 1.18 at 6144 and 0.79 to 0.95 at 8192, L = 16
//     1.08 to 1.18 at 8192
//   Potts L = 48, second iteration: 0.93 at 8256, 0.90 at 12288
//   MUMA, second iteration and settled: L = 64 (staged) 1.34 and 1.48 at
//     20480, L = 48 1.00 and 1.11 at 20480, L = 32 1.04 and 1.16 at 20480,
//     L = 24 1.01 and 1.10 at 16384, 0.91 and 0.97 at 16896, L = 16 1.15 and
//     1.06 at 14336, L = 8 1.65 and 1.17 at 12288
//   L = 4, launches of 10 and 100 sweeps, against four lanes: Ising at 4096
//     1.01 and 1.31, MUMA at 4096 1.21 and 1.93, Potts at 1536 1.00 and 1.39,
//     at 2048 0.90 and 1.39, at 4096 0.83 and 0.96
//   L = 64 with the table in global memory, whose latency few lanes per chain
//     hide worse, second iteration and settled: Ising 1.13 and 1.93 at 8192,
//     0.82 and 1.47 at 12288, 0.79 and 0.96 at 16384, Potts 1.21 and 1.70 at
//     12288, 0.91 and 1.29 at 16384, 0.95 and 1.42 at 24576, MUMA 1.31 and
//     1.35 at 40960
// No line of a lattice that has 16 lanes per chain by default (all but Potts
// of L = 4, 8 and 24) lies below the 4096 chains up to which it has them.
inline long tile_max_chains(int model, int L, bool staged, int weights)
{
    const int row = L >= 64 ? (staged ? 1 : 0) : L >= 48 ? 2 : L >= 32 ? 3 : L >= 24 ? 4 : L >= 16 ? 5 : L >= 8 ? 6 : 7;
    // [64 with the table in global memory, 64, 48, 32, 24, 16, 8, 4]
    constexpr int lines[3][3][8] = {
        {{12288, 10240, 8192, 8192, 8192, 8192, 8192, 4096},
         {8192, 6144, 8192, 8192, 6144, 8192, 8192, 4096},
         {8192, 4096, 4096, 4096, 4096, 4096, 4096, 4096}},
        {{24576, 12288, 12288, 8192, 6144, 8192, 8192, 1536},
         {24576, 12288, 12288, 8192, 6144, 8192, 8192, 1536},
         {12288, 12288, 8192, 4096, 4096, 4096, 4096, 1536}},
        {{40960, 20480, 20480, 20480, 16384, 14336, 12288, 4096},
         {40960, 20480, 20480, 20480, 16384, 14336, 12288, 4096},
         {40960, 20480, 20480, 20480, 16384, 14336, 12288, 4096}},
    };
    return lines[model][weights][row];
}

// Chains per workgroup of the one-wavefront-per-chain kernel, at most
// `most`: as many workgroups as there are CUs, down to one wavefront per SIMD.
inline int default_tile_chains(int most, long n_chains, int cus)
{
    int n = most < 16 ? most : 16;
    while (n > 4 && n_chains <= (long)cus * (n / 2))
        n /= 2;
    return n;
}

// ---------------------------------------------------------------------------
// What the autotuners time
// ---------------------------------------------------------------------------
// Lanes per chain and threads per block.  Sixteen lanes are a wavefront per
// chain: workgroups of 4, 8 and 16 chains, the ones that are taken by default
// (2048 chains of Potts q = 8, L = 48, settled weights: 41 cycles per site at
// 8, 54 and 70 at 16 and 4 with a staged table).
struct LaunchShape {
    int lanes, threads;
};
constexpr LaunchShape kTunedShapes[] = {{1, 64}, {1, 256}, {1, 512}, {2, 64},  {2, 256},  {2, 512},
                                        {4, 64}, {4, 256}, {4, 512}, {16, 64}, {16, 128}, {16, 256}};

// Revision of what they time, part of every key of MUCA_AUTOTUNE_CACHE: an
// entry is read only by a library whose kernels, candidates and probe weights
// are the ones that it was measured with.  Raise it when any of them changes.
// (1, without a mark in the key: 16 lanes were lanes of one wavefront shared
// by four chains; 2: item times on the run's own weights.)
constexpr int kTunedRevision = 3;

// Log weights on which candidates are timed: independent and uniform in
// (-0.15, 0.15).  On flat weights a tile takes the fewest passes it can, and
// one wavefront per chain would be preferred where it is the slower one as
// soon as the weights move.  Cycles per site, flat / these / a run's twelfth
// to thirtieth iteration of ten sweeps: Ising L = 64, 8192 chains 41.4 / 65.0
// / 71.8 to 66.6, Ising L = 32, 4096 chains 23.7 / 43.0 / 50.8 to 47.9, Potts
// L = 48, 4096 chains 43.0 / 57.5 / 54.9 to 53.6 (four lanes: 101, 107, 170,
// whatever the weights).
inline double probe_lnw(int bin)
{
    uint64_t z = ((uint64_t)bin + 1) * 0x9E3779B97F4A7C15ull; // splitmix64
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return 0.3 * ((double)(z >> 11) * 0x1p-53 - 0.5);
}

// ---------------------------------------------------------------------------
// Work items of a batched round
// ---------------------------------------------------------------------------
// Chains of one work item: 64 at four lanes per chain, 16, 8 or 4 at one
// wavefront per chain.
constexpr int kItemChains = 64, kTileItemChains = 16;

// Cycles per site of a full item alone on its CU, for runs whose item times
// were not measured: [Ising, Potts, MUMA][L = 64, 48, 32, 24, 16, 8][four
// lanes, a wavefront per chain].  Measured at 16384 and 4096 chains, one
// workgroup on every CU, settled weights (Potts L = 64: table in global
// memory).
inline double nominal_cycles(int model, int L, bool tiles)
{
    constexpr double cycles[3][6][2] = {
        {{100, 33}, {106, 42}, {108, 44}, {127, 48}, {128, 44}, {177, 50}},
        {{196, 57}, {178, 55}, {173, 60}, {188, 78}, {190, 65}, {225, 77}},
        {{151, 20}, {110, 26}, {111, 24}, {133, 31}, {120, 29}, {181, 36}},
    };
    return cycles[model][L >= 64 ? 0 : L >= 48 ? 1 : L >= 32 ? 2 : L >= 24 ? 3 : L >= 16 ? 4 : 5][tiles ? 1 : 0];
}

// What an item of a wavefront per chain takes of that time with weights of a
// class (see weights_class): second iteration over settled, Ising 1.3 (L =
// 64) to 1.8 (L = 24), Potts 1.2 (L = 16) to 1.7 (L = 32).
inline double tile_slowdown(int model, int weights)
{
    return weights == kRough ? (model == 0 ? 1.6 : 1.4) : weights == kBetween ? 1.25 : 1.0;
}

// Workgroups of 8 and 4 wavefronts leave the CU's issue slots to fewer of
// them: an item of 8 (4) chains takes this share of the time of one of 16
// (Potts L = 48: 42, 31 and 23 cycles per site; Ising L = 64: 23, 18 and 13).
inline double tile_share(int chains) { return chains == 16 ? 1.0 : chains == 8 ? 0.75 : 0.55; }

// Estimated length of a round on n_cus CUs.  side_by_side: the work that two
// items on one CU do in the time of one alone, 1 where a CU holds one item.
// They raise the throughput of rounds with more items than CUs; no item is
// shorter for it.
struct RoundLength {
    double longest = 0.0, shortest = 0.0, total = 0.0;
    long items = 0;
    void add(long k, double t)
    {
        longest = t > longest ? t : longest;
        shortest = items == 0 || t < shortest ? t : shortest;
        total += (double)k * t;
        items += k;
    }
    double estimate(int n_cus, double side_by_side) const
    {
        const long rounds = (items + n_cus - 1) / n_cus;
        double len = total / ((double)n_cus * side_by_side); // all items spread evenly
        if (items > n_cus) { // some CU takes at least `rounds` items
            const double busiest = (double)rounds * shortest / side_by_side;
            len = busiest > len ? busiest : len;
        }
        return longest > len ? longest : len;
    }
};

// One run of a round.  In: its chains and the time of a full item at [four
// lanes per chain, a wavefront per chain], < 0 where that kernel changed the
// run's results when it was measured, and the table placement that each time
// stands for (kept here for the caller).  Out: chains per item and an item's
// time.
struct RoundRun {
    long chains;
    double t[2];
    bool table_in_lds[2];
    int item_chains;
    double cost;
    long items(int per_item) const { return (chains + per_item - 1) / per_item; }
};

enum { kRoundFourLanes = 0, kRoundTiles = 1, kRoundTooManyItems = -1, kRoundNoKernel = -2 };

// The kernel of a round (one for all its runs: the one with the shorter
// estimate) and its items.  may4, may16: the caller's choice of kernels.  A
// kernel that any run rejected is out, and so is one whose items exceed
// max_items (counted in items of 64 or 16 chains); *n_items: the items of the
// kernel that comes closest to fitting.
inline int choose_round(RoundRun *runs, int n, bool may4, bool may16, int max_items, int n_cus, double side_by_side,
                        long *n_items)
{
    RoundLength len4, len16;
    for (int i = 0; i < n; ++i) {
        may4 = may4 && runs[i].t[0] >= 0.0;
        may16 = may16 && runs[i].t[1] >= 0.0;
        len4.add(runs[i].items(kItemChains), runs[i].t[0]);
        len16.add(runs[i].items(kTileItemChains), runs[i].t[1]);
    }
    if (!may4 && !may16)
        return kRoundNoKernel;
    *n_items = may4 ? len4.items : len16.items;
    may4 = may4 && len4.items <= max_items;
    may16 = may16 && len16.items <= max_items;
    if (!may4 && !may16)
        return kRoundTooManyItems;
    if (may16) {
        // no item longer than the longest run's in items of 16, 8 or 4
        // chains; every run takes its largest items within that
        auto chains_within = [&](int i, double limit) {
            int c = kTileItemChains;
            while (c > 4 && runs[i].t[1] * tile_share(c) > limit * 1.001)
                c /= 2;
            return c;
        };
        double best = -1.0, limit = len16.longest;
        for (int c = kTileItemChains; c >= 4; c /= 2) {
            RoundLength len;
            for (int i = 0; i < n; ++i) {
                const int k = chains_within(i, len16.longest * tile_share(c));
                len.add(runs[i].items(k), runs[i].t[1] * tile_share(k));
            }
            const double est = len.estimate(n_cus, 1.0);
            if (len.items <= max_items && (best < 0.0 || est < 0.999 * best))
                best = est, limit = len16.longest * tile_share(c);
        }
        for (int i = 0; i < n; ++i) {
            runs[i].item_chains = chains_within(i, limit);
            runs[i].cost = runs[i].t[1] * tile_share(runs[i].item_chains);
        }
        if (!may4 || len4.estimate(n_cus, side_by_side) >= best)
            return kRoundTiles;
    }
    for (int i = 0; i < n; ++i) {
        runs[i].item_chains = kItemChains;
        runs[i].cost = runs[i].t[0];
    }
    return kRoundFourLanes;
}

} // namespace muca
