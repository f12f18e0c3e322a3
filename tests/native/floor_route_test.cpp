// The rule that gives floors to blocks or to single wavefronts (csrc/floor_route.hpp) against the sizes at
// which both were measured, and its estimate of the worlds a rollout owes.
#include <cstdio>

#include "../../paper_2402_16801_amd/csrc/floor_route.hpp"

using cf::FloorWork;

struct Measured { FloorWork work; bool perlin; long long floors; double blocks_us, wavefronts_us; };

int main()
{
    const Measured rows[] = {
        { FloorWork::RESET, false, 288, 6.4, 14.5 },    { FloorWork::RESET, false, 2700, 14.1, 18.1 },  { FloorWork::RESET, false, 4194, 19.0, 20.6 },
        { FloorWork::RESET, false, 4500, 19.9, 20.8 },  { FloorWork::RESET, false, 5130, 21.9, 21.3 },  { FloorWork::RESET, false, 6138, 25.0, 22.1 },
        { FloorWork::RESET, false, 8640, 32.8, 30.6 },  { FloorWork::RESET, false, 73728, 230, 144 },
        { FloorWork::IMPORT, false, 288, 12.6, 22.3 },  { FloorWork::IMPORT, false, 3600, 28.5, 32.7 }, { FloorWork::IMPORT, false, 4500, 33.1, 33.9 },
        { FloorWork::IMPORT, false, 4797, 34.65, 34.6 }, { FloorWork::IMPORT, false, 5121, 36.2, 34.9 }, { FloorWork::IMPORT, false, 18000, 112, 89 },
        { FloorWork::RESET, true, 288, 9.4, 21.7 },     { FloorWork::RESET, true, 1800, 19.5, 24.3 },   { FloorWork::RESET, true, 2340, 23.6, 25.5 },
        { FloorWork::RESET, true, 2700, 26.3, 25.7 },   { FloorWork::RESET, true, 3600, 32.6, 28.5 },   { FloorWork::RESET, true, 5130, 43.2, 35.1 },
        { FloorWork::RESET, true, 6138, 50.3, 41.0 },   { FloorWork::RESET, true, 8190, 64.5, 51.4 },   { FloorWork::RESET, true, 11988, 90.6, 62.7 },
        { FloorWork::RESET, true, 73728, 515, 237 },
        { FloorWork::IMPORT, true, 288, 16.0, 29.6 },   { FloorWork::IMPORT, true, 2070, 32.6, 37.2 },  { FloorWork::IMPORT, true, 2592, 38.1, 38.7 },
        { FloorWork::IMPORT, true, 2790, 40.1, 38.9 },  { FloorWork::IMPORT, true, 3600, 47.6, 40.3 },  { FloorWork::IMPORT, true, 18000, 203, 123 },
        { FloorWork::MUTATE, true, 288, 19.5, 23.1 },   { FloorWork::MUTATE, true, 720, 22.0, 23.8 },   { FloorWork::MUTATE, true, 1080, 24.1, 25.3 },
        { FloorWork::MUTATE, true, 1440, 27.5, 25.8 },  { FloorWork::MUTATE, true, 2052, 31.4, 26.2 },  { FloorWork::MUTATE, true, 18000, 152, 85 },
        { FloorWork::OWED, false, 819, 119.4, 127.7 },  { FloorWork::OWED, false, 2079, 151.0, 154.7 }, { FloorWork::OWED, false, 2880, 173.4, 175.9 },
        { FloorWork::OWED, false, 4095, 218.7, 216.7 }, { FloorWork::OWED, false, 13104, 661, 637 },    { FloorWork::OWED, true, 819, 124.7, 134.2 },
        { FloorWork::OWED, true, 2079, 160.8, 162.9 },  { FloorWork::OWED, true, 2880, 185.5, 184.0 },  { FloorWork::OWED, true, 4095, 233.9, 226.6 },
        { FloorWork::OWED, true, 13104, 724, 674 },
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
