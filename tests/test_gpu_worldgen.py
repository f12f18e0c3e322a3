"""Generated worlds, cell by cell, against the oracle: both variants and both noises over seeds from the
whole 64-bit range.  The comparison is exact: the generators evaluate integer fields in 32-bit floating
point rounded down, where floors and comparisons are those of the integers."""
import numpy as np
import pytest

from oracle import pyoracle as po
from paper_2402_16801_amd import binding as cx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("perlin", [False, True])
@pytest.mark.parametrize("full,n", [(False, 1), (False, 700), (True, 1), (True, 60), (True, 900)])
def test_worlds_match_oracle(full, n, perlin):
    # 900 full-game environments are 16,200 floors, beyond where single wavefronts take over from blocks
    noise = cx.WORLDGEN_PERLIN if perlin else cx.WORLDGEN_VALUE
    cfg = cx.default_config(cx.VARIANT_CRAFTAX if full else cx.VARIANT_CLASSIC, worldgen=noise)
    ocfg = po.full_default_config(worldgen=noise) if full else po.default_config(worldgen=noise)
    rng = np.random.RandomState(1234 + n + perlin)
    seeds = (rng.randint(0, 2 ** 32, n, dtype=np.uint64) << np.uint64(32)) | rng.randint(0, 2 ** 32, n, dtype=np.uint64)
    seeds[0] = np.uint64(2 ** 64 - 1)
    if n > 1:
        seeds[1] = 0
    sim = cx.Craftax(n, cfg)
    orc = po.FullOracle(n, ocfg) if full else po.Oracle(n, ocfg, po.OBS_SYM_U8_F32)
    got, want = sim.reset(seeds).cpu().numpy(), orc.reset(seeds)
    assert np.array_equal(got, want)
    assert sim.export_envs().tobytes() == orc.envs.tobytes()


@pytest.mark.parametrize("perlin", [False, True])
@pytest.mark.parametrize("n", [17, 49152])
def test_classic_rollout_owes_worlds(n, perlin):
    """A rollout in which episodes end once, twice and more often (a cap of 9 in 31 steps), below and at the
    size from which its blocks generate worlds themselves: afterwards every spare world is in place, so
    that steps go on exactly as in a batch that was stepped from the start."""
    import torch
    noise = cx.WORLDGEN_PERLIN if perlin else cx.WORLDGEN_VALUE
    steps, after = 31, 12
    cfg = cx.default_config(worldgen=noise, max_episode_steps=9)
    seeds = np.arange(n, dtype=np.uint64) + np.uint64(77)
    rolled, stepped = cx.Craftax(n, cfg), cx.Craftax(n, cfg)
    rolled.reset(seeds)
    stepped.reset(seeds)
    acts = torch.empty((steps + after, n), dtype=torch.int32, device=rolled.device)
    cx.craftax_synth_actions(acts, n, 0, steps + after, 3, 1, rolled.stream)
    rew = torch.zeros((steps, n), dtype=torch.float32, device=rolled.device)
    done = torch.zeros((steps, n), dtype=torch.uint8, device=rolled.device)
    cx.craftax_rollout(rolled.state, acts[:steps].contiguous(), steps, rolled.obs, rew, done, n, rolled.stream)
    for s in range(steps):
        obs, r, d = stepped.step(acts[s])
        assert torch.equal(r, rew[s]) and torch.equal(d, done[s]), s
    assert torch.equal(obs, rolled.obs)
    for s in range(steps, steps + after):
        a, b = rolled.step(acts[s]), stepped.step(acts[s])
        assert all(torch.equal(x, y) for x, y in zip(a, b)), s
    assert rolled.export_envs().tobytes() == stepped.export_envs().tobytes()


@pytest.mark.parametrize("perlin", [False, True])
@pytest.mark.parametrize("n,pre,steps,cap", [(1, 0, 31, 2), (16, 98, 3, 100), (40, 58, 2, 60), (64, 170, 2, 171)])
def test_classic_rollout_whose_blocks_generate_what_they_owe(n, pre, steps, cap, perlin):
    """Rollouts short enough to have no launch behind them: one environment whose episodes end again and again, and
    batches in which all episodes end together, so that a block generates a world for each of them after the last step."""
    import torch
    after = 2 * cap if cap < 10 else 6
    cfg = cx.default_config(worldgen=cx.WORLDGEN_PERLIN if perlin else cx.WORLDGEN_VALUE, max_episode_steps=cap)
    rolled, stepped = cx.Craftax(n, cfg), cx.Craftax(n, cfg)
    acts = torch.empty((pre + steps + after, n), dtype=torch.int32, device=rolled.device)
    cx.craftax_synth_actions(acts, n, 0, pre + steps + after, 5, 1, rolled.stream)
    for sim in (rolled, stepped):
        sim.reset(np.arange(n, dtype=np.uint64) + np.uint64(31))
        for s in range(pre):
            sim.step(acts[s])
    rew = torch.zeros((steps, n), dtype=torch.float32, device=rolled.device)
    done = torch.zeros((steps, n), dtype=torch.uint8, device=rolled.device)
    cx.craftax_rollout(rolled.state, acts[pre:pre + steps].contiguous(), steps, rolled.obs, rew, done, n, rolled.stream)
    for s in range(steps):
        obs, r, d = stepped.step(acts[pre + s])
        assert torch.equal(r, rew[s]) and torch.equal(d, done[s]), s
    assert int(done.sum()) > n // 3 and torch.equal(obs, rolled.obs)
    for s in range(pre + steps, pre + steps + after):
        a, b = rolled.step(acts[s]), stepped.step(acts[s])
        assert all(torch.equal(x, y) for x, y in zip(a, b)), s
    assert rolled.export_envs().tobytes() == stepped.export_envs().tobytes()


@pytest.mark.parametrize("n,perlin", [(250, True), (569, True), (570, True), (683, True), (684, True), (570, False)])
def test_full_import_generates_the_worlds_a_reset_would(n, perlin):
    """Imported levels have the spare worlds of the states they were exported from, whichever form of the generator takes the
    floors: blocks, single wavefronts, and around the number of Perlin floors (6,144) that single wavefronts take in one round."""
    import torch
    cfg = cx.default_config(cx.VARIANT_CRAFTAX, worldgen=cx.WORLDGEN_PERLIN if perlin else cx.WORLDGEN_VALUE, max_episode_steps=3)
    seeds = np.arange(n, dtype=np.uint64) + np.uint64(900)
    first, second = cx.Craftax(n, cfg), cx.Craftax(n, cfg)
    first.reset(seeds)
    second.reset(seeds + np.uint64(50000))
    second.import_envs(first.export_envs())
    acts = torch.empty((7, n), dtype=torch.int32, device=first.device)
    cx.craftax_synth_actions(acts, n, 0, 7, 3, 2, first.stream)
    for s in range(7):
        a, b = first.step(acts[s]), second.step(acts[s])
        assert all(torch.equal(x, y) for x, y in zip(a, b)), s
    assert first.export_envs().tobytes() == second.export_envs().tobytes()


@pytest.mark.parametrize("perlin", [False, True])
@pytest.mark.parametrize("n", [24577, 49151, 57345, 70001])
def test_classic_four_lanes_at_every_split_of_the_regeneration(n, perlin):
    """Four lanes per environment: rollouts that leave their worlds to a launch (up to 49,151 environments) and that generate
    them after every step, against steps whose regeneration blocks take two rounds of units, or one (70,001: the chip holds
    the step blocks and a part of the regeneration blocks)."""
    test_classic_rollout_owes_worlds(n, perlin)


def test_classic_rollout_without_observations_at_the_largest_batch():
    """Without observations the worlds of a large batch are left to the launch behind the rollout: afterwards the state is
    the one of a rollout that writes them, whose blocks generate after every step."""
    import torch
    n, steps = 49152, 21
    cfg = cx.default_config(max_episode_steps=9)
    seeds = np.arange(n, dtype=np.uint64) + np.uint64(5)
    seen, unseen = cx.Craftax(n, cfg), cx.Craftax(n, cfg)
    acts = torch.empty((steps, n), dtype=torch.int32, device=seen.device)
    cx.craftax_synth_actions(acts, n, 0, steps, 3, 1, seen.stream)
    out = []
    for sim, obs in ((seen, seen.obs), (unseen, None)):
        sim.reset(seeds)
        rew = torch.zeros((steps, n), dtype=torch.float32, device=sim.device)
        done = torch.zeros((steps, n), dtype=torch.uint8, device=sim.device)
        cx.craftax_rollout(sim.state, acts, steps, obs, rew, done, n, sim.stream)
        out.append((rew, done))
    assert all(torch.equal(a, b) for a, b in zip(*out))
    for s in range(steps):
        a, b = seen.step(acts[s]), unseen.step(acts[s])
        assert all(torch.equal(x, y) for x, y in zip(a, b)), s
    assert seen.export_envs().tobytes() == unseen.export_envs().tobytes()
