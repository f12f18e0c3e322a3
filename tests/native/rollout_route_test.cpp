// The rule for the worlds that a Classic rollout owes (csrc/rollout_route.hpp) against the sizes at which both
// sides were measured.
#include <cstdio>

#include "../../paper_2402_16801_amd/csrc/rollout_route.hpp"

struct Measured { bool perlin; long long n, steps; double launch_us, block_us; };

int main()
{
    const Measured rows[] = {
        { false, 1, 1, 13.5, 10.2 },    { false, 1, 8, 46.8, 44.5 },     { false, 1, 32, 162, 161 },      { false, 16, 1, 14.3, 11.5 },
        { false, 16, 8, 57.9, 56.2 },   { false, 16, 16, 107.3, 106.6 }, { false, 64, 1, 15.3, 13.1 },    { false, 64, 4, 34.7, 34.3 },
        { false, 256, 1, 17.2, 16.3 },  { false, 64, 8, 59.6, 61.1 },    { false, 16, 32, 206.4, 209.0 }, { false, 256, 4, 36.5, 38.2 },
        { false, 600, 2, 24.8, 25.6 },  { false, 1024, 1, 18.6, 18.9 },  { false, 4096, 1, 20.3, 21.5 },
        { true, 1, 1, 13.7, 10.3 },     { true, 1, 16, 86.8, 83.8 },     { true, 16, 4, 33.8, 31.9 },     { true, 16, 8, 59.4, 58.8 },
        { true, 64, 2, 22.9, 22.0 },    { true, 16, 16, 111.2, 112.4 },  { true, 64, 4, 36.0, 36.9 },     { true, 256, 2, 25.3, 26.8 },
        { true, 600, 1, 19.3, 20.6 },   { true, 4096, 1, 21.5, 25.4 },
    };
    int bad = 0;
    for (const Measured& m : rows)
        if ((cx::rollout_own_from(false, m.perlin, true, m.n, m.steps, 10000) == m.steps - 1) != (m.block_us < m.launch_us)) {
            std::printf("perlin %d, %lld environments, %lld steps: the slower side\n", (int)m.perlin, m.n, m.steps);
            ++bad;
        }
    // short episodes owe worlds sooner; many environments generate after every step only with four lanes each
    auto from = [](bool four_lanes, bool perlin, bool observed, long long n, long long steps, long long cap = 10000) {
        return cx::rollout_own_from(four_lanes, perlin, observed, n, steps, cap);
    };
    bad += from(false, false, true, 16, 8, 9) != 8 || from(true, false, true, 49151, 64) != 64 || from(true, false, true, 49152, 64) != cx::ONE_EACH_STEP ||
           from(true, true, true, 65536, 1) != cx::ONE_EACH_STEP || from(false, true, true, 65536, 64) != 64 ||
           from(true, false, false, 65536, 64) != 64 || from(true, true, false, 49152, 16) != 16 || from(false, false, false, 1, 1) != 0;
    if (bad == 0) std::printf("rollout_route_test: ok\n");
    return bad != 0;
}
