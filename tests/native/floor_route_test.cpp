// The rule that gives floors to blocks or to single wavefronts (csrc/floor_route.hpp) against the sizes at
// which both were measured, and its estimate of the worlds a rollout owes.
#include <cstdio>

#include "../../paper_2402_16801_amd/csrc/floor_route.hpp"

using cf::FloorWork;

struct Measured { FloorWork work; bool perlin; long long floors; double blocks_us, wavefronts_us; };

int main()
{
    const Measured rows[] = {
        { FloorWork::RESET, false, 288, 6.03, 15.29 }, { FloorWork::RESET, false, 2700, 13.16, 18.58 }, { FloorWork::RESET, false, 4500, 18.19, 21.18 }, { FloorWork::RESET, false, 5400, 20.66, 22.41 },
        { FloorWork::RESET, false, 7686, 26.88, 26.15 }, { FloorWork::RESET, false, 7992, 27.66, 26.21 }, { FloorWork::RESET, false, 8190, 28.19, 26.26 }, { FloorWork::RESET, false, 8298, 28.5, 29.58 },
        { FloorWork::RESET, false, 9000, 30.27, 31.63 }, { FloorWork::RESET, false, 10188, 33.29, 33.74 }, { FloorWork::RESET, false, 10800, 35.03, 35.82 }, { FloorWork::RESET, false, 11394, 36.62, 36.2 },
        { FloorWork::RESET, false, 13500, 41.89, 40.37 }, { FloorWork::RESET, false, 36000, 100.56, 77.32 }, { FloorWork::RESET, false, 73728, 199.09, 138.92 },
        { FloorWork::IMPORT, false, 288, 12.53, 22.83 }, { FloorWork::IMPORT, false, 3600, 28.16, 32.52 }, { FloorWork::IMPORT, false, 4797, 33.87, 34.77 }, { FloorWork::IMPORT, false, 5049, 34.99, 35.08 },
        { FloorWork::IMPORT, false, 5193, 35.6, 35.93 }, { FloorWork::IMPORT, false, 5400, 36.44, 36.07 }, { FloorWork::IMPORT, false, 5697, 37.76, 36.69 }, { FloorWork::IMPORT, false, 9000, 52.62, 46.41 },
        { FloorWork::IMPORT, false, 18000, 107.84, 77.92 },
        { FloorWork::RESET, true, 288, 7.91, 20.47 }, { FloorWork::RESET, true, 2700, 17.03, 23.53 }, { FloorWork::RESET, true, 4500, 23.38, 26.34 }, { FloorWork::RESET, true, 5400, 26.67, 27.6 },
        { FloorWork::RESET, true, 5688, 27.7, 27.61 }, { FloorWork::RESET, true, 5886, 28.43, 27.71 }, { FloorWork::RESET, true, 6084, 29.09, 27.85 }, { FloorWork::RESET, true, 6192, 29.46, 32.9 },
        { FloorWork::RESET, true, 9000, 39.22, 42.96 }, { FloorWork::RESET, true, 10800, 45.44, 47.53 }, { FloorWork::RESET, true, 11700, 48.83, 49.57 }, { FloorWork::RESET, true, 12186, 50.54, 50.35 },
        { FloorWork::RESET, true, 12996, 53.34, 52.64 }, { FloorWork::RESET, true, 18000, 70.47, 63.75 }, { FloorWork::RESET, true, 73728, 264.66, 185.82 },
        { FloorWork::IMPORT, true, 288, 14.51, 28.03 }, { FloorWork::IMPORT, true, 2592, 27.06, 35.52 }, { FloorWork::IMPORT, true, 3600, 32.92, 37.9 }, { FloorWork::IMPORT, true, 4500, 38.06, 39.47 },
        { FloorWork::IMPORT, true, 4950, 40.41, 40.13 }, { FloorWork::IMPORT, true, 5850, 45.34, 42.07 }, { FloorWork::IMPORT, true, 6192, 47.26, 46.84 },
        { FloorWork::IMPORT, true, 9000, 62.47, 58.28 }, { FloorWork::IMPORT, true, 18000, 128.24, 97.56 },
        { FloorWork::MUTATE, true, 288, 18.66, 22.11 }, { FloorWork::MUTATE, true, 720, 21.73, 22.78 }, { FloorWork::MUTATE, true, 1080, 22.7, 23.88 }, { FloorWork::MUTATE, true, 1440, 23.9, 24.31 },
        { FloorWork::MUTATE, true, 1548, 24.09, 24.38 }, { FloorWork::MUTATE, true, 1620, 24.4, 24.46 }, { FloorWork::MUTATE, true, 1800, 24.84, 24.48 }, { FloorWork::MUTATE, true, 2160, 26.38, 25.03 },
        { FloorWork::MUTATE, true, 3600, 32.18, 27.92 }, { FloorWork::MUTATE, true, 18000, 88.28, 68.55 },
        { FloorWork::OWED, false, 819, 117.9, 127.7 }, { FloorWork::OWED, false, 2079, 149.0, 155.0 }, { FloorWork::OWED, false, 2880, 172.3, 177.4 }, { FloorWork::OWED, false, 4095, 217.3, 218.5 },
        { FloorWork::OWED, false, 4914, 257.2, 257.5 }, { FloorWork::OWED, false, 5526, 287.8, 286.1 }, { FloorWork::OWED, false, 6138, 317.1, 314.6 }, { FloorWork::OWED, false, 8190, 418.3, 412.6 },
        { FloorWork::OWED, true, 819, 120.1, 132.6 }, { FloorWork::OWED, true, 2079, 153.2, 160.0 }, { FloorWork::OWED, true, 2880, 178.1, 182.4 }, { FloorWork::OWED, true, 4095, 224.38, 224.43 },
        { FloorWork::OWED, true, 4914, 265.9, 264.0 }, { FloorWork::OWED, true, 5526, 297.3, 292.9 }, { FloorWork::OWED, true, 8190, 439.6, 426.4 },
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
