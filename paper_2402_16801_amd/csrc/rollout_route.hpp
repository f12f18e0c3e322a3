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
//  - where four lanes per environment nearly fill the chip a block generates its worlds after every step, because
//    the other blocks' memory traffic then covers for it (64 steps, value noise / Perlin noise, none against one after
//    a step: 32,768 environments 1,065 / 1,157 against 1,125 / 1,219, 49,152: 1,424 / 1,561 against 1,428 / 1,540,
//    65,536: 1,825 / 2,004 against 1,776 / 1,895; one and a launch against all that are owed: 49,152 1,421 / 1,534
//    against 1,410 / 1,525, 65,536 1,769 / 1,889 against 1,761 / 1,877).  Not in a rollout of one step (65,536: 59.3 / 64.7
//    with the launch, 59.5 / 67.3 without) or, with Perlin noise, two (49,152: 82.5 / 83.5), and not in one that writes
//    no observation, where there is no such traffic (65,536 x 64 with the launch 969 / 1,145, without 1,055 / 1,254;
//    49,152 805 / 938 against 896 / 1,054).
// Plain C++ so that the rule itself can be tested without a GPU.
#pragma once

#include "floor_route.hpp"

namespace cx {

constexpr long long OWN_WORLDS_FROM = 49152;

// The step (from 0) from which on a block generates the worlds that its environments are owed, all that there
// are after each step, so that nothing is owed at the end and no launch follows; `steps`: never.
// four_lanes: four lanes per environment, else sixteen; observed: the rollout writes observations.
inline long long rollout_own_from(bool four_lanes, bool perlin, bool observed, long long n, long long steps, long long max_episode_steps)
{
    if (cf::worlds_owed(n, steps, max_episode_steps) < (perlin ? 1 : 2)) return steps - 1;
    return four_lanes && observed && n >= OWN_WORLDS_FROM && steps > (perlin ? 2 : 1) ? 0 : steps;
}

}  // namespace cx
