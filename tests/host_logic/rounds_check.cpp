// Host-only check of how the 24-field kernel deals units to workgroups (csrc/rounds.hpp): every unit exactly once, and a compute unit that
// is held by somebody else costs little.  Built with g++ by tests/test_rounds.py.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "rounds.hpp"

using namespace octfd;

// Rounds that XCD `x` takes with `units` compute units: workgroups start in their order, each on the first compute unit that is free.
static int64_t busy(int64_t n_units, int x, int units)
{
    const int64_t rounds = rounds_of(n_units);
    const int parts = parts_of(rounds);
    std::vector<int64_t> until(units, 0);
    for (int i = x; i < parts * kRound; i += kSchedXcds) {
        const Rounds mine = rounds_of_part(i / kRound, parts, rounds);
        int64_t taken = 0;
        for (int64_t r = mine.first; r < mine.last && unit_of_round(r, i % kRound, n_units) >= 0; ++r) ++taken;
        *std::min_element(until.begin(), until.end()) += taken;
    }
    return *std::max_element(until.begin(), until.end());
}

int main()
{
    const int per_xcd = kRound / kSchedXcds;
    std::vector<int64_t> sizes;
    for (int64_t n = 1; n <= 3000; n += n % 256 < 8 || n % 256 > 248 ? 1 : 37) sizes.push_back(n);
    for (int64_t n : {10532, 16384, 51037, 131072, 524288}) sizes.push_back(n);
    for (const int64_t n : sizes) {
        const int64_t rounds = rounds_of(n);
        const int parts = parts_of(rounds);
        std::vector<int> times(n, 0);
        int64_t last = 0;
        for (int part = 0; part < parts; ++part) {
            const Rounds mine = rounds_of_part(part, parts, rounds);
            if (mine.first != last || mine.last <= mine.first) { std::printf("FAILED: rounds of part %d of %ld units\n", part, (long)n); return 1; }
            last = mine.last;
            for (int wg = 0; wg < kRound; ++wg) {
                bool ended = false;                  // a workgroup ends with the first round that has nothing for it
                for (int64_t r = mine.first; r < mine.last; ++r) {
                    const int64_t u = unit_of_round(r, wg, n);
                    if (u >= n || (ended && u >= 0)) { std::printf("FAILED: unit %ld of %ld\n", (long)u, (long)n); return 1; }
                    if (u < 0) ended = true;
                    else ++times[u];
                }
            }
        }
        if (last != rounds || std::count(times.begin(), times.end(), 1) != n) { std::printf("FAILED: units of %ld not taken once each\n", (long)n); return 1; }
        for (int x = 0; x < kSchedXcds; ++x) {
            const int64_t alone = busy(n, x, per_xcd), held = busy(n, x, per_xcd - 1);
            if (alone > rounds) { std::printf("FAILED: %ld units take %ld rounds\n", (long)n, (long)alone); return 1; }
            // one compute unit of 32 less is at least one round more, and at most an eighth of them with the round that is begun and not full
            if (rounds > 2 && held > rounds + 1 + rounds / 8) { std::printf("FAILED: %ld units take %ld rounds instead of %ld\n", (long)n, (long)held, (long)alone); return 1; }
        }
    }
    std::printf("units dealt\n");
    return 0;
}
