// The rule that gives floors to blocks or to single wavefronts (csrc/floor_route.hpp) against the sizes at
// which both were measured, and its estimate of the worlds a rollout owes.
#include <cstdio>

#include "../../paper_2402_16801_amd/csrc/floor_route.hpp"

using cf::FloorWork;

struct Measured { FloorWork work; bool perlin; long long floors; double blocks_us, wavefronts_us; };

int main()
{
    const Measured rows[] = {
        { FloorWork::RESET, false, 288, 7.1, 16.0 },   { FloorWork::RESET, false, 3600, 19.6, 22.3 },  { FloorWork::RESET, false, 4194, 21.7, 22.9 },
        { FloorWork::RESET, false, 4788, 23.8, 23.1 }, { FloorWork::RESET, false, 6138, 28.6, 24.5 },  { FloorWork::RESET, false, 7200, 32.3, 28.0 },
        { FloorWork::RESET, false, 73728, 263, 174 },
        { FloorWork::IMPORT, false, 288, 13.3, 23.1 }, { FloorWork::IMPORT, false, 4194, 33.6, 34.6 }, { FloorWork::IMPORT, false, 4797, 36.5, 35.6 },
        { FloorWork::IMPORT, false, 18000, 114, 87 },
        { FloorWork::RESET, true, 288, 11.8, 27.5 },   { FloorWork::RESET, true, 3600, 35.6, 38.0 },   { FloorWork::RESET, true, 4194, 39.7, 38.8 },
        { FloorWork::RESET, true, 6138, 53.3, 44.2 },  { FloorWork::RESET, true, 7200, 61.2, 65.6 },   { FloorWork::RESET, true, 9720, 78.6, 84.9 },
        { FloorWork::RESET, true, 11988, 94.3, 95.0 }, { FloorWork::RESET, true, 14400, 111, 104 },    { FloorWork::RESET, true, 73728, 525, 343 },
        { FloorWork::IMPORT, true, 288, 18.5, 34.9 },  { FloorWork::IMPORT, true, 2592, 39.6, 42.2 },  { FloorWork::IMPORT, true, 3600, 48.0, 46.0 },
        { FloorWork::IMPORT, true, 9720, 104, 97 },    { FloorWork::IMPORT, true, 18000, 191, 150 },
        { FloorWork::MUTATE, true, 288, 23.0, 29.6 },  { FloorWork::MUTATE, true, 1440, 31.3, 34.2 },  { FloorWork::MUTATE, true, 2052, 36.2, 34.8 },
        { FloorWork::MUTATE, true, 3069, 44.4, 35.3 }, { FloorWork::MUTATE, true, 18000, 158, 121 },
        { FloorWork::OWED, false, 819, 124, 132 },     { FloorWork::OWED, false, 1638, 139.5, 143.6 }, { FloorWork::OWED, false, 3276, 181.7, 179.4 },
        { FloorWork::OWED, false, 13107, 675, 643 },   { FloorWork::OWED, true, 819, 128, 142 },       { FloorWork::OWED, true, 1638, 147.5, 156.5 },
        { FloorWork::OWED, true, 3276, 197.3, 194.9 }, { FloorWork::OWED, true, 13107, 748, 703 },
    };
    int bad = 0;
    for (const Measured& m : rows)
        if (cf::floors_by_blocks(m.work, m.perlin, m.floors) != (m.blocks_us < m.wavefronts_us)) {
            std::printf("work %d, perlin %d, %lld floors: the slower form\n", (int)m.work, (int)m.perlin, m.floors);
            ++bad;
        }
    // Perlin imports by five and by six wavefronts per SIMD
    const struct { long long floors; double five_us, six_us; } rounds[] = { { 5040, 41.8, 44.3 }, { 5121, 41.9, 44.9 }, { 5148, 48.7, 45.1 }, { 5400, 49.5, 45.8 },
        { 6138, 55.8, 47.5 }, { 6300, 56.7, 57.2 }, { 18000, 123, 130 } };
    for (const auto& m : rounds)
        if (cf::one_tight_round(FloorWork::IMPORT, true, m.floors) != (m.six_us < m.five_us)) {
            std::printf("import of %lld floors: the slower bound\n", m.floors);
            ++bad;
        }
    bad += cf::one_tight_round(FloorWork::IMPORT, false, 5400) || cf::one_tight_round(FloorWork::RESET, true, 5400);
    bad += cf::worlds_owed(4096, 16, 100000) != 364 || cf::worlds_owed(4096, 500, 100000) != 4096 || cf::worlds_owed(343, 20, 13) != 343 ||
           cf::worlds_owed(343, 1, 13) != 26 || cf::worlds_owed(7, 1, 1) != 7;
    if (bad == 0) std::printf("floor_route_test: ok\n");
    return bad != 0;
}
