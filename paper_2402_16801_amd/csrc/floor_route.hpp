// Whether floors are generated by blocks of five wavefronts or by single wavefronts (full game).
//
// A block makes one pass over the 288 runs of a floor, a single wavefront five; but no wavefront of
// a block works while the first one lays the floor out.  A few floors last as long as one of them, so
// blocks are ahead; thousands are a matter of throughput, and single wavefronts are ahead.  The lines lie between measured sizes (us, blocks / single
// wavefronts; floors in the order of floor_grid, overworlds first):
//   reset, value noise      288  6.1 / 15.4   3,600 13.3 / 16.7   4,500 15.7 / 16.8   4,950 16.8 / 16.9   5,040 17.0 / 16.8   5,400 18.0 / 16.9   7,200 22.7 / 20.2   8,298 25.7 / 22.3   10,800 32.0 / 26.2   18,000 50.3 / 37.6
//     (calls with their observation of 4,770 20.3 / 20.7, of 5,040 20.9 / 20.8)
//   import, value noise     288  8.3 / 18.6   3,600 17.3 / 22.8   4,797 21.5 / 24.9   5,850 24.8 / 26.1   6,300 26.4 / 26.5   6,480 27.0 / 26.5   7,200 29.6 / 28.2   9,000 35.9 / 33.9   18,000 82.1 / 59.6
//     (behind a step 6,300 37.3 / 38.1, 6,750 39.0 / 38.7; level turns over 700 47.3 / 48.1, 800 51.9 / 53.1, 900 56.8 / 58.0)
//   reset, Perlin noise     288  8.0 / 20.7   3,600 17.0 / 21.7   4,500 20.4 / 21.8   4,860 21.6 / 21.8   4,950 22.0 / 21.8   5,400 23.5 / 21.9   7,200 30.0 / 26.5   9,360 37.2 / 30.4   12,240 47.2 / 35.1   18,000 67.6 / 47.8
//     (calls with their observation of 4,770 25.2 / 25.8, of 5,040 26.3 / 25.9)
//   import, Perlin noise    288 10.0 / 23.8   3,600 20.3 / 28.3   4,797 25.6 / 30.4   5,850 30.0 / 31.6   6,300 32.0 / 32.8   6,480 32.9 / 31.7   7,200 36.4 / 34.4   9,000 43.9 / 39.2   18,000 101 / 78.9
//     (level turns over 700 75.7 / 77.5, 750 79.1 / 76.1)
//   noise mutation          288 18.8 / 22.6   1,080 22.1 / 23.1   1,620 22.8 / 23.5   1,935 22.9 / 23.8   2,070 24.0 / 23.7   2,700 26.4 / 23.8   3,600 29.7 / 24.0   9,000 49.5 / 30.9
//   owed by a rollout       us of a whole rollout with its two launches for owed worlds in the one or the other form, environments x steps (floors owed):
//                           1,024 x 16 (819) 91.7 / 101.7   3,600 x 16 (2,880) 135.1 / 139.1   4,096 x 24 (4,914) 198.5 / 201.0   4,096 x 27 (5,526) 222.1 / 222.9   4,096 x 30 (6,138) 247.2 / 246.4   4,096 x 40 (8,190) 326 / 319
//                           Perlin noise: 93.4 / 106.7   139.9 / 145.5   210.6 / 211.6   233.1 / 233.4   260.5 / 259.0   348 / 340
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

namespace cf {

enum class FloorWork { RESET, IMPORT, MUTATE, OWED };

// Wavefronts per SIMD that the generating kernels are bounded to.  With Perlin noise six (five: resets of 4,096 environments 230 us, 218 with
// six; level turns over 256, 1,000 and 2,000 levels 69.7, 141 and 217 us, 65.7, 138 and 213 with six), which spill no vector register.
constexpr int VALUE_WAVES = 8, PERLIN_WAVES = 6;

inline bool floors_by_blocks(FloorWork work, bool perlin, long long floors)
{
    switch (work) {
    case FloorWork::RESET: return floors <= (perlin ? 4900 : 5000);
    case FloorWork::IMPORT: return floors <= 6400;
    case FloorWork::MUTATE: return floors <= 2000;     // Perlin worlds only
    default: return floors <= 5800;
    }
}

// Worlds that n environments owe after `steps` steps, for the rule above (what is generated is what is on the
// lists): one for each that has finished an episode, and episodes last about 180 steps unless the cap ends them.
inline long long worlds_owed(long long n, long long steps, long long max_episode_steps)
{
    const long long length = max_episode_steps < 180 ? max_episode_steps : 180;
    return steps >= length ? n : n * steps / length;
}

}  // namespace cf
