// Whether floors are generated by blocks of five wavefronts or by single wavefronts (full game).
//
// A block makes one pass over the 288 runs of a floor, a single wavefront five; but no wavefront of
// a block works while the first one lays the floor out.  A few floors last as long as one of them, so
// blocks are ahead; thousands are a matter of throughput, and single wavefronts are ahead.  The lines
// lie between measured sizes (us, blocks / single wavefronts):
//   reset, value noise      288  7.1 / 16.0   3,600 19.6 / 22.3   4,194 21.7 / 22.9   4,788 23.8 / 23.1   6,138 28.6 / 24.5   73,728 263 / 174
//   import, value noise     288 13.3 / 23.1   3,600 30.8 / 33.6   4,194 33.6 / 34.6   4,797 36.5 / 35.6   6,138 43.6 / 38.0   18,000 114 / 87
//   reset, Perlin noise     288 11.8 / 27.5   3,600 35.6 / 38.0   4,194 39.7 / 38.8   6,138 53.3 / 44.2
//     6,144 single wavefronts run at once (six on each of 1,024 SIMDs); a second round costs as much as
//     the first until it is nearly full:  7,200 61.2 / 65.6   9,720 78.6 / 84.9   11,988 94.3 / 95.0   14,400 111 / 104   73,728 525 / 343
//   import, Perlin noise    288 18.5 / 34.9   2,592 39.6 / 42.2   3,069 43.2 / 43.1   3,600 48.0 / 46.0   9,720 104 / 97   18,000 191 / 150
//   noise mutation          288 23.0 / 29.6   1,440 31.3 / 34.2   2,052 36.2 / 34.8   3,069 44.4 / 35.3   9,720  95 / 88   18,000 158 / 121
//   owed by a rollout       us of a whole rollout with its two launches for owed worlds in the one or the other form, environments x steps (floors owed):
//                           1,024 x 16 (819) 124 / 132   2,048 x 16 (1,638) 139.5 / 143.6   4,096 x 16 (3,276) 181.7 / 179.4   4,096 x 64 (13,107) 675 / 643
//                           Perlin noise: 128 / 142   147.5 / 156.5   197.3 / 194.9   748 / 703
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

namespace cf {

enum class FloorWork { RESET, IMPORT, MUTATE, OWED };

// Wavefronts per SIMD that the generating kernels are bounded to.  With Perlin noise five cost no spilled registers;
// six do, and are 3 to 8 % slower, but take 5,121 to 6,144 single wavefronts in one round.
constexpr long long SIMDS = 1024;
constexpr int VALUE_WAVES = 8, PERLIN_WAVES = 5, PERLIN_WAVES_TIGHT = 6;

// Imports of Perlin worlds by single wavefronts whose second round would be short: five / six per SIMD, us:
//   5,121 floors 41.9 / 44.9   5,148 48.7 / 45.1   5,400 49.5 / 45.8   5,580 51.3 / 46.1   6,138 55.8 / 47.5   6,300 56.7 / 57.2
// A few wavefronts beyond a round do not make a second one: they run beside the last of the first.
inline bool one_tight_round(FloorWork work, bool perlin, long long floors)
{
    constexpr long long FEW = 8;
    return work == FloorWork::IMPORT && perlin && floors > SIMDS * PERLIN_WAVES + FEW && floors <= SIMDS * PERLIN_WAVES_TIGHT + FEW;
}

inline bool floors_by_blocks(FloorWork work, bool perlin, long long floors)
{
    switch (work) {
    case FloorWork::RESET: return perlin ? floors <= 4000 || (floors > 6144 && floors <= 12000) : floors <= 4500;
    case FloorWork::IMPORT: return floors <= (perlin ? 3072 : 4500);
    case FloorWork::MUTATE: return floors <= 1850;     // Perlin worlds only
    default: return floors <= 3072;
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
