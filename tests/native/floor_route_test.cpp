// The rule that gives floors to blocks or to single wavefronts (csrc/floor_route.hpp) against the sizes at
// which both were measured, and its estimate of the worlds a rollout owes.
#include <cstdio>

#include "../../paper_2402_16801_amd/csrc/floor_route.hpp"

using cf::FloorWork;

struct Measured { FloorWork work; bool perlin; long long floors; double blocks_us, wavefronts_us; };

int main()
{
    const Measured rows[] = {
        { FloorWork::RESET, false, 288, 6.07, 15.44 }, { FloorWork::RESET, false, 2700, 10.76, 16.34 }, { FloorWork::RESET, false, 3600, 13.33, 16.67 }, { FloorWork::RESET, false, 4500, 15.73, 16.77 },
        { FloorWork::RESET, false, 4680, 16.18, 16.8 }, { FloorWork::RESET, false, 4860, 16.5, 16.84 }, { FloorWork::RESET, false, 4950, 16.76, 16.89 }, { FloorWork::RESET, false, 5040, 17.04, 16.79 },
        { FloorWork::RESET, false, 5220, 17.43, 16.92 }, { FloorWork::RESET, false, 5400, 17.98, 16.91 }, { FloorWork::RESET, false, 6300, 20.22, 18.65 }, { FloorWork::RESET, false, 7200, 22.67, 20.17 },
        { FloorWork::RESET, false, 8298, 25.7, 22.26 }, { FloorWork::RESET, false, 9360, 28.28, 24.24 }, { FloorWork::RESET, false, 10800, 31.96, 26.19 }, { FloorWork::RESET, false, 11520, 33.81, 27.45 },
        { FloorWork::RESET, false, 18000, 50.3, 37.61 },
        { FloorWork::IMPORT, false, 288, 8.34, 18.55 }, { FloorWork::IMPORT, false, 1800, 10.52, 20.42 }, { FloorWork::IMPORT, false, 3600, 17.3, 22.8 }, { FloorWork::IMPORT, false, 4797, 21.48, 24.85 },
        { FloorWork::IMPORT, false, 5400, 23.51, 25.52 }, { FloorWork::IMPORT, false, 5850, 24.83, 26.09 }, { FloorWork::IMPORT, false, 6300, 26.43, 26.47 }, { FloorWork::IMPORT, false, 6480, 27.02, 26.49 },
        { FloorWork::IMPORT, false, 6660, 27.63, 26.73 }, { FloorWork::IMPORT, false, 7200, 29.57, 28.24 }, { FloorWork::IMPORT, false, 9000, 35.87, 33.91 }, { FloorWork::IMPORT, false, 18000, 82.05, 59.58 },
        { FloorWork::RESET, true, 288, 7.98, 20.67 }, { FloorWork::RESET, true, 2700, 14.17, 21.53 }, { FloorWork::RESET, true, 3600, 17.03, 21.7 }, { FloorWork::RESET, true, 4500, 20.43, 21.82 },
        { FloorWork::RESET, true, 4680, 20.97, 21.76 }, { FloorWork::RESET, true, 4860, 21.56, 21.77 }, { FloorWork::RESET, true, 4950, 21.96, 21.8 }, { FloorWork::RESET, true, 5040, 22.31, 21.81 },
        { FloorWork::RESET, true, 5400, 23.5, 21.93 }, { FloorWork::RESET, true, 6300, 26.77, 24.4 }, { FloorWork::RESET, true, 7200, 29.98, 26.46 }, { FloorWork::RESET, true, 9360, 37.15, 30.38 },
        { FloorWork::RESET, true, 12240, 47.24, 35.11 }, { FloorWork::RESET, true, 18000, 67.63, 47.81 },
        { FloorWork::IMPORT, true, 288, 10.03, 23.82 }, { FloorWork::IMPORT, true, 2592, 16.08, 26.69 }, { FloorWork::IMPORT, true, 3600, 20.34, 28.27 }, { FloorWork::IMPORT, true, 4500, 24.09, 29.83 },
        { FloorWork::IMPORT, true, 4797, 25.58, 30.39 }, { FloorWork::IMPORT, true, 5400, 28.28, 31.12 }, { FloorWork::IMPORT, true, 5850, 30.03, 31.59 }, { FloorWork::IMPORT, true, 6300, 31.98, 32.84 },
        { FloorWork::IMPORT, true, 6480, 32.94, 31.67 }, { FloorWork::IMPORT, true, 6660, 33.67, 31.52 }, { FloorWork::IMPORT, true, 7200, 36.38, 34.43 }, { FloorWork::IMPORT, true, 9000, 43.92, 39.17 },
        { FloorWork::IMPORT, true, 18000, 101.01, 78.86 },
        { FloorWork::MUTATE, true, 288, 18.77, 22.57 }, { FloorWork::MUTATE, true, 999, 22.86, 23.51 }, { FloorWork::MUTATE, true, 1080, 22.1, 23.14 }, { FloorWork::MUTATE, true, 1350, 22.85, 23.4 },
        { FloorWork::MUTATE, true, 1620, 22.84, 23.45 }, { FloorWork::MUTATE, true, 1800, 22.4, 23.37 }, { FloorWork::MUTATE, true, 1935, 22.89, 23.82 }, { FloorWork::MUTATE, true, 2070, 23.97, 23.68 },
        { FloorWork::MUTATE, true, 2250, 24.74, 23.82 }, { FloorWork::MUTATE, true, 2700, 26.35, 23.83 }, { FloorWork::MUTATE, true, 3600, 29.72, 23.97 }, { FloorWork::MUTATE, true, 9000, 49.46, 30.94 },
        { FloorWork::OWED, false, 819, 91.67, 101.72 }, { FloorWork::OWED, false, 2880, 135.1, 139.06 }, { FloorWork::OWED, false, 3276, 137.87, 140.15 }, { FloorWork::OWED, false, 3681, 154.66, 155.04 },
        { FloorWork::OWED, false, 4500, 185.3, 186.13 }, { FloorWork::OWED, false, 4914, 198.49, 200.96 }, { FloorWork::OWED, false, 5526, 222.13, 222.87 }, { FloorWork::OWED, false, 6138, 247.17, 246.42 },
        { FloorWork::OWED, false, 6750, 269.62, 268.78 }, { FloorWork::OWED, false, 7371, 295.67, 290.76 }, { FloorWork::OWED, false, 8190, 326.02, 319.1 },
        { FloorWork::OWED, true, 819, 93.35, 106.73 }, { FloorWork::OWED, true, 2880, 139.88, 145.49 }, { FloorWork::OWED, true, 3276, 143.87, 147.5 }, { FloorWork::OWED, true, 3681, 160.59, 162.37 },
        { FloorWork::OWED, true, 4500, 193.1, 194.3 }, { FloorWork::OWED, true, 4914, 210.55, 211.62 }, { FloorWork::OWED, true, 5526, 233.07, 233.42 }, { FloorWork::OWED, true, 6138, 260.51, 258.96 },
        { FloorWork::OWED, true, 6750, 284.56, 278.93 }, { FloorWork::OWED, true, 7371, 312.91, 305.74 }, { FloorWork::OWED, true, 8190, 348.33, 339.51 },
    };
    int bad = 0;
    for (const Measured& m : rows)
        if (cf::floors_by_blocks(m.work, m.perlin, m.floors) != (m.blocks_us < m.wavefronts_us)) {
            std::printf("work %d, perlin %d, %lld floors: the slower form\n", (int)m.work, (int)m.perlin, m.floors);
            ++bad;
        }
    bad += cf::worlds_owed(4096, 16, 100000) != 364 || cf::worlds_owed(4096, 500, 100000) != 4096 || cf::worlds_owed(343, 20, 13) != 343 ||
           cf::worlds_owed(343, 1, 13) != 26 || cf::worlds_owed(7, 1, 1) != 7;
    if (bad == 0) std::printf("floor_route_test: ok\n");
    return bad != 0;
}
