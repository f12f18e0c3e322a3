// Which regeneration units a block of a step launch takes when the step blocks share that work
// (four lanes per environment; see regeneration_share in craftax.hip).  A sub-list of `count`
// entries is 2 * count units (unit u = half u & 1 of entry u >> 1).  Its per_sub regeneration
// blocks take the head, one or two rounds of per_sub units (head_rounds); the tail is dealt out in turn to the
// nq step blocks that append to the sub-list and, behind them, to the regeneration blocks again.
// Plain integer arithmetic, usable on the host, so that "every unit is taken exactly once, by a
// block that exists" can be checked without a GPU.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define CX_UNITS_FN __host__ __device__ inline
#else
#define CX_UNITS_FN inline
#endif

namespace cx {

// Rounds that the regeneration blocks take before the step blocks share the rest.  Two while the chip holds all
// blocks of the launch at once: a second unit then costs a regeneration block nothing, and the step blocks keep
// their time.  One where the step blocks leave room for a part of them only: the others start when a step block
// ends, and their units come on top.  (Larger batches end in the order of their blocks anyway.)  resident: blocks
// of the kernel that the chip holds.  Step in us with one round / two, skewed actions, on states in turn and on one:
//   value noise (1,280 resident)   24,576 22.1 / 21.3   19.9 / 18.9   49,152 32.2 / 31.8   27.0 / 25.6   65,536 43.1 / 42.4   31.9 / 31.2
//     67,584 48.9 / 49.8   33.7 / 33.8   73,728 54.6 / 55.6   35.6 / 36.0   81,920 56.3 / 56.7   38.3 / 40.1   131,072 102.4 / 99.6   95.3 / 93.4
//   Perlin noise (1,280 resident)  57,344 45.6 / 41.9   30.1 / 29.0   61,440 44.7 / 41.6   31.4 / 30.0   65,536 45.6 / 43.3   33.1 / 31.5
//     67,584 50.8 / 49.7   34.8 / 34.9   73,728 57.2 / 56.4   36.8 / 37.6   81,920 57.5 / 57.2   40.7 / 43.0
CX_UNITS_FN uint32_t head_rounds(uint32_t step_blocks, uint32_t regen_blocks, uint32_t resident)
{
    return step_blocks <= resident && step_blocks + regen_blocks > resident ? 1u : 2u;
}

struct UnitWalk {
    uint32_t u;         // the unit to generate now; the walk is over once u >= 2 * count
    uint32_t round;     // units taken so far + 1
};

// helper: step block number `index` among the nq that append to this sub-list; else regeneration
// block number `index` among the sub-list's per_sub.  rounds: head_rounds of the launch.
CX_UNITS_FN UnitWalk first_unit(bool helper, uint32_t index, uint32_t per_sub, uint32_t rounds)
{
    return UnitWalk{ helper ? rounds * per_sub + index : index, 1u };
}
CX_UNITS_FN UnitWalk next_unit(UnitWalk w, bool helper, uint32_t index, uint32_t per_sub, uint32_t nq, uint32_t rounds)
{
    const uint32_t head = rounds * per_sub, workers = nq + per_sub;
    if (helper) w.u += workers;
    else w.u = w.round < rounds ? w.u + per_sub : (w.round == rounds ? head + nq + index : w.u + workers);
    ++w.round;
    return w;
}
// the first unit of step block `index`'s share: it has work if this is below 2 * count
CX_UNITS_FN uint32_t first_helper_unit(uint32_t index, uint32_t per_sub, uint32_t rounds) { return rounds * per_sub + index; }

}  // namespace cx
