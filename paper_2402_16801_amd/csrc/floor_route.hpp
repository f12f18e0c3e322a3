// Whether floors are generated by blocks of five wavefronts or by single wavefronts (full game).
//
// A block makes one pass over the 288 runs of a floor, a single wavefront five; but no wavefront of
// a block works while the first one lays the floor out.  A few floors last as long as one of them, so
// blocks are ahead; thousands are a matter of throughput, and single wavefronts are ahead.  The lines
// lie between measured sizes (us, blocks / single wavefronts):
//   reset, value noise      288  6.4 / 14.5   2,700 14.1 / 18.1   4,194 19.0 / 20.6   4,500 19.9 / 20.8   5,130 21.9 / 21.3   6,138 25.0 / 22.1   73,728 230 / 144
//   import, value noise     288 12.6 / 22.3   3,600 28.5 / 32.7   4,500 33.1 / 33.9   4,797 34.7 / 34.6   5,121 36.2 / 34.9   18,000 112 / 89
//   reset, Perlin noise     288  9.4 / 21.7   1,800 19.5 / 24.3   2,340 23.6 / 25.5   2,700 26.3 / 25.7   3,600 32.6 / 28.5
//     (5,120 single wavefronts ran at once then)
//     4,788 40.8 / 29.2   5,130 43.2 / 35.1   6,138 50.3 / 41.0   11,988 90.6 / 62.7   73,728 515 / 237
//   import, Perlin noise    288 16.0 / 29.6   2,070 32.6 / 37.2   2,592 38.1 / 38.7   2,790 40.1 / 38.9   3,600 47.6 / 40.3   18,000 203 / 123
//   noise mutation          288 19.5 / 23.1   720 22.0 / 23.8   1,080 24.1 / 25.3   1,440 27.5 / 25.8   2,052 31.4 / 26.2   18,000 152 / 85
//   owed by a rollout       us of a whole rollout with its two launches for owed worlds in the one or the other form, environments x steps (floors owed):
//                           1,024 x 16 (819) 119 / 128   2,600 x 16 (2,079) 151 / 155   3,600 x 16 (2,880) 173.4 / 175.9   4,096 x 20 (4,095) 218.7 / 216.7   4,096 x 64 (13,104) 661 / 637
//                           Perlin noise: 125 / 134   160.8 / 162.9   185.5 / 184.0   234 / 227   724 / 674
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

namespace cf {

enum class FloorWork { RESET, IMPORT, MUTATE, OWED };

// Wavefronts per SIMD that the generating kernels are bounded to.  With Perlin noise six, which spill nothing (five:
// resets of 4,096 environments 230 us, 218 with six; level turns over 256, 1,000 and 2,000 levels 69.7, 141 and 217 us, 65.7, 138 and 213 with six).
constexpr long long SIMDS = 1024;
constexpr int VALUE_WAVES = 8, PERLIN_WAVES = 6;

// Imports of Perlin worlds by single wavefronts that six to a SIMD take in one round and five in two, by five / six per SIMD, us,
// when six spilled registers:
//   5,121 floors 41.9 / 44.9   5,148 48.7 / 45.1   5,400 49.5 / 45.8   5,580 51.3 / 46.1   6,138 55.8 / 47.5   6,300 56.7 / 57.2
// A few wavefronts beyond a round do not make a second one: they run beside the last of the first.  No call asks this
// since every import runs six to a SIMD; what it knows about rounds is kept with its test.
inline bool one_tight_round(FloorWork work, bool perlin, long long floors)
{
    constexpr long long FEW = 8;
    return work == FloorWork::IMPORT && perlin && floors > SIMDS * (PERLIN_WAVES - 1) + FEW && floors <= SIMDS * PERLIN_WAVES + FEW;
}

inline bool floors_by_blocks(FloorWork work, bool perlin, long long floors)
{
    switch (work) {
    case FloorWork::RESET:
    case FloorWork::IMPORT: return floors <= (perlin ? 2600 : 4650);
    case FloorWork::MUTATE: return floors <= 1250;     // Perlin worlds only
    default: return floors <= (perlin ? 2600 : 3200);
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
