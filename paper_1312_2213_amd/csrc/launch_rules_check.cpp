// launch_rules_check.cpp -- prints what the rules of launch_rules.h give for
// cases read from a text file, so that they can be built on their own with
// sanitizers and compared with an independent implementation.
//
// Input, whitespace-separated, one case after another:
//   segments <total> <at_most>
//   noise <n> P[n]
//   line <model> <L> <staged> <noise>
//   tile <most> <n_chains> <cus>
//   shapes
//   probe <bins>
//   round <may4> <may16> <max_items> <n_cus> <side_by_side> <n> (<chains> <t4> <t16>)[n]
// Output: one line per case:
//   segments: number of segments, their sum, shortest, longest, and the
//     sweeps before the last one (it stops at 10^7 segments)
//   noise: weights_noise
//   line: weights_class and tile_max_chains
//   tile: default_tile_chains
//   shapes: lanes and threads of every entry of kTunedShapes
//   probe: probe_lnw of every bin
//   round: choose_round, then chains per item and item time of every run
#include <algorithm>
#include <cinttypes>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "launch_rules.h"

namespace {

FILE *in = nullptr;

[[noreturn]] void fail(const char *what)
{
    std::fprintf(stderr, "launch_rules_check: bad input (%s)\n", what);
    std::exit(2);
}

long long get_int()
{
    long long v;
    if (std::fscanf(in, "%lld", &v) != 1)
        fail("integer");
    return v;
}

double get_double()
{
    char tok[64];
    if (std::fscanf(in, "%63s", tok) != 1)
        fail("double");
    return std::strtod(tok, nullptr);
}

} // namespace

int main(int argc, char **argv)
{
    if (argc != 2)
        fail("usage: launch_rules_check <cases file>");
    in = std::fopen(argv[1], "r");
    if (!in)
        fail("cannot open the cases file");
    char kind[32];
    while (std::fscanf(in, "%31s", kind) == 1) {
        if (!std::strcmp(kind, "segments")) {
            const int32_t total = (int32_t)get_int(), at_most = (int32_t)get_int();
            int64_t k = 0, sum = 0, shortest = INT64_MAX, longest = 0, before = 0;
            muca::for_segments(total, at_most, [&](int32_t done, int32_t n) {
                if (done != sum || ++k > 10000000) {
                    std::printf("segments do not end or do not follow each other\n");
                    std::exit(1);
                }
                before = done;
                sum += n;
                shortest = std::min<int64_t>(shortest, n);
                longest = std::max<int64_t>(longest, n);
            });
            std::printf("%" PRId64 " %" PRId64 " %" PRId64 " %" PRId64 " %" PRId64 "\n", k, sum, k ? shortest : 0,
                        longest, before);
        } else if (!std::strcmp(kind, "noise")) {
            const int n = (int)get_int();
            if (n < 0 || n > (1 << 20))
                fail("length");
            std::vector<double> P((size_t)n);
            for (double &p : P)
                p = get_double();
            std::printf("%.17g\n", muca::weights_noise(n, P.data()));
        } else if (!std::strcmp(kind, "line")) {
            const int model = (int)get_int(), L = (int)get_int();
            const bool staged = get_int() != 0;
            const int weights = muca::weights_class(model, get_double());
            std::printf("%d %ld\n", weights, muca::tile_max_chains(model, L, staged, weights));
        } else if (!std::strcmp(kind, "tile")) {
            const int most = (int)get_int();
            const long n = (long)get_int();
            std::printf("%d\n", muca::default_tile_chains(most, n, (int)get_int()));
        } else if (!std::strcmp(kind, "shapes")) {
            for (const muca::LaunchShape &s : muca::kTunedShapes)
                std::printf("%d %d ", s.lanes, s.threads);
            std::printf("\n");
        } else if (!std::strcmp(kind, "probe")) {
            const int n = (int)get_int();
            for (int b = 0; b < n; ++b)
                std::printf("%.17g ", muca::probe_lnw(b));
            std::printf("\n");
        } else if (!std::strcmp(kind, "round")) {
            const bool may4 = get_int() != 0, may16 = get_int() != 0;
            const int max_items = (int)get_int(), n_cus = (int)get_int();
            const double side = get_double();
            const int n = (int)get_int();
            if (n < 1 || n > 4096)
                fail("runs");
            std::vector<muca::RoundRun> r((size_t)n);
            for (muca::RoundRun &x : r) {
                x = muca::RoundRun{};
                x.chains = (long)get_int();
                x.t[0] = get_double();
                x.t[1] = get_double();
            }
            long items = 0;
            std::printf("%d", muca::choose_round(r.data(), n, may4, may16, max_items, n_cus, side, &items));
            for (const muca::RoundRun &x : r)
                std::printf(" %d %.17g", x.item_chains, x.cost);
            std::printf("\n");
        } else {
            fail(kind);
        }
    }
    std::fclose(in);
    return 0;
}
