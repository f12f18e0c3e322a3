// Whether floors are generated by blocks of five wavefronts or by single wavefronts (full game).
//
// A block makes one pass over the 288 runs of a floor, a single wavefront five; but no wavefront of
// a block works while the first one lays the floor out.  A few floors last as long as one of them, so
// blocks are ahead; thousands are a matter of throughput, and single wavefronts are ahead.  In between single wavefronts of a
// reset catch up where they fill the chip exactly once (6,144 of Perlin noise, 8,192 of value noise run at the same time), and
// fall back with the next round.  The lines lie between measured sizes (us, blocks / single wavefronts):
//   reset, value noise      288  6.0 / 15.3   4,500 18.2 / 21.2   7,200 25.5 / 25.5   7,686 26.9 / 26.2   8,190 28.2 / 26.3   8,298 28.5 / 29.6   10,800 35.0 / 35.8   11,394 36.6 / 36.2   16,200 49.0 / 45.1   73,728 199 / 139
//     (over maps that are not in the cache: calls with their observation of 6,300 40.5 / 41.4, of 7,056 43.0 / 42.0)
//   import, value noise     288 12.5 / 22.8   3,600 28.2 / 32.5   4,797 33.9 / 34.8   5,193 35.6 / 35.9   5,400 36.4 / 36.1   6,003 39.2 / 37.1   9,000 52.6 / 46.4   18,000 108 / 78
//   reset, Perlin noise     288  7.9 / 20.5   2,700 17.0 / 23.5   5,400 26.7 / 27.6   5,688 27.7 / 27.6   6,084 29.1 / 27.9   6,192 29.5 / 32.9   9,000 39.2 / 43.0   11,700 48.8 / 49.6   12,186 50.5 / 50.4   14,400 58.0 / 55.9   73,728 265 / 186
//   import, Perlin noise    288 14.5 / 28.0   2,592 27.1 / 35.5   4,500 38.1 / 39.5   4,950 40.4 / 40.1   6,093 46.7 / 42.6   6,192 47.3 / 46.8   9,000 62.5 / 58.3   18,000 128 / 98
//     (with other kernels in between blocks fall behind earlier: level turns over 400 76.9 / 80.8, 500 88.4 / 88.2, 540 93.9 / 90.6)
//   noise mutation          288 18.7 / 22.1   1,080 22.7 / 23.9   1,548 24.1 / 24.4   1,620 24.4 / 24.5   1,800 24.8 / 24.5   2,700 28.5 / 25.7   18,000 88.3 / 68.6
//   owed by a rollout       us of a whole rollout with its two launches for owed worlds in the one or the other form, environments x steps (floors owed):
//                           1,024 x 16 (819) 118 / 128   3,600 x 16 (2,880) 172 / 177   4,096 x 20 (4,095) 217.3 / 218.5   4,096 x 24 (4,914) 257.2 / 257.5   4,096 x 27 (5,526) 287.8 / 286.1   4,096 x 40 (8,190) 418 / 413
//                           Perlin noise: 120 / 133   178 / 182   224.4 / 224.4   265.9 / 264.0   297 / 293   440 / 426
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

namespace cf {

enum class FloorWork { RESET, IMPORT, MUTATE, OWED };

// Wavefronts per SIMD that the generating kernels are bounded to.  With Perlin noise six (five: resets of 4,096 environments 230 us, 218 with
// six; level turns over 256, 1,000 and 2,000 levels 69.7, 141 and 217 us, 65.7, 138 and 213 with six), which spill no vector register.
constexpr long long SIMDS = 1024;
constexpr int VALUE_WAVES = 8, PERLIN_WAVES = 6;

inline bool floors_by_blocks(FloorWork work, bool perlin, long long floors)
{
    const bool one_round = floors <= SIMDS * (perlin ? PERLIN_WAVES : VALUE_WAVES);
    switch (work) {
    case FloorWork::RESET: return floors <= (one_round ? (perlin ? 5650 : 6300) : (perlin ? 12100 : 11200));
    case FloorWork::IMPORT: return floors <= (perlin ? 4600 : 5300);
    case FloorWork::MUTATE: return floors <= 1650;     // Perlin worlds only
    default: return floors <= (perlin ? 4100 : 5000);
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
