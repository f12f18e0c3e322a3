// Who generates the worlds that a Classic rollout owes (see k_rollout in craftax.hip).
//
// A launch of regeneration blocks behind the rollout generates all of them with the whole chip.  That launch
// costs about 3 us even if it finds nothing, and a block of the rollout that stops for a world of its own stops
// for 5 to 8 us:
//  - a rollout that owes hardly any world has no such launch, and its blocks generate after their last step what
//    their environments are owed.  Measured, the launch behind it against none (us, environments x steps):
//      value noise   1 x 1 13.5 / 10.2   1 x 32 162 / 161   16 x 8 57.9 / 56.2   16 x 16 107.3 / 106.6   64 x 4 34.7 / 34.3
//                    256 x 1 17.2 / 16.3   64 x 8 59.6 / 61.1   256 x 4 36.5 / 38.2   1,024 x 1 18.6 / 18.9
//      Perlin noise  1 x 1 13.7 / 10.3   16 x 4 33.8 / 31.9   16 x 8 59.4 / 58.8   64 x 2 22.9 / 22.0
//                    16 x 16 111.2 / 112.4   64 x 4 36.0 / 36.9   256 x 2 25.3 / 26.8   1,024 x 1 19.6 / 21.6
//    (environments times steps over the 180 steps that an episode lasts: the worlds owed);
//  - where four lanes per environment nearly fill the chip a block generates a world after every step, because
//    the other blocks' memory traffic then covers for it (64 steps, value noise / Perlin noise, none against one:
//    32,768 environments 1,065 / 1,157 against 1,125 / 1,219, 49,152: 1,424 / 1,561 against 1,428 / 1,540, 65,536:
//    1,825 / 2,004 against 1,776 / 1,895).  Not in a rollout that writes no observation, where there is no such
//    traffic (65,536 x 64 none 969 / 1,145, all that are owed after a step 1,055 / 1,254; 49,152 805 / 938 against
//    896 / 1,054).  Not all that are owed either: with episodes of 20 steps they come together, and the launch
//    behind the rollout has the whole chip for what is left (65,536 x 32 1,607 / 2,143 with one, 1,662 / 2,243 with all).
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

#include "floor_route.hpp"

namespace cx {

constexpr long long OWN_WORLDS_FROM = 49152;

// Who generates: the launch behind the rollout (= steps), that launch and after every step a block one world
// (ONE_EACH_STEP), or the blocks after the last step, all that are owed (= steps - 1; no launch behind the rollout).
// As the number of the first step (from 0) after which a block generates worlds.
// four_lanes: four lanes per environment, else sixteen; observed: the rollout writes observations.
constexpr long long ONE_EACH_STEP = -1;
inline long long rollout_own_from(bool four_lanes, bool perlin, bool observed, long long n, long long steps, long long max_episode_steps)
{
    if (cf::worlds_owed(n, steps, max_episode_steps) < (perlin ? 1 : 2)) return steps - 1;
    return four_lanes && observed && n >= OWN_WORLDS_FROM ? ONE_EACH_STEP : steps;
}

}  // namespace cx
