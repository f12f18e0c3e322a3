"""How observations reach memory depends on the batch: pictures are drawn by the launch that steps, and stores are
left in the L2, written through or streamed.  Every route against the kernel that only observes (which the parity
tests compare with the oracle), and the rules against a run without observations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2402_16801_amd import binding as cx, synth  # noqa: E402


def _run(n, steps, variant, **kw):
    cfg = cx.default_config(variant, **kw)
    sim, blind = cx.Craftax(n, cfg), cx.Craftax(n, cfg)
    seeds = synth.seeds_for(n)
    sim.reset(seeds)
    blind.reset(seeds)
    sim.obs.fill_(0x5A if sim.obs.dtype == torch.uint8 else 7.0)
    seen = torch.empty_like(sim.obs)
    actions = torch.empty((steps, n), dtype=torch.int32, device=sim.device)
    cx.craftax_synth_actions(actions, n, 0, steps, 3, 1 + 2 * (variant == cx.VARIANT_CRAFTAX), sim.stream)
    reward, done = torch.empty(n, device=sim.device), torch.empty(n, dtype=torch.uint8, device=sim.device)
    ended = 0
    for t in range(steps):
        obs, r, d = sim.step(actions[t])
        cx.craftax_observe(sim.state, seen, n, sim.stream)
        assert torch.equal(obs.view(torch.uint8), seen.view(torch.uint8)), f"observation at step {t}"
        cx.craftax_step(blind.state, actions[t], None, reward, done, n, sim.stream)
        assert torch.equal(r, reward) and torch.equal(d, done), f"reward or done at step {t}"
        ended += int(d.sum())
        if t == steps // 2:                                    # an edit: the next step serves episodes without a spare world
            for s in (sim, blind):
                cx.craftax_mutate_swap(s.state, 0, n, 7, 0, False, None, s.stream)
    assert sim.export_envs().tobytes() == blind.export_envs().tobytes()
    return ended


# streamed, written through from 32 MiB on (705 pictures), by every fourth block from 85 MiB on (1,872), streamed again
@pytest.mark.parametrize("n", [1, 17, 704, 705, 1871, 1872, 5700])
def test_classic_pictures_of_a_step(n):
    assert _run(n, 14, cx.VARIANT_CLASSIC, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=5) > 0


def test_classic_pictures_of_a_perlin_step_with_four_lanes():
    assert _run(33, 12, cx.VARIANT_CLASSIC, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=4, worldgen=cx.WORLDGEN_PERLIN, group_lanes=4) > 0


@pytest.mark.parametrize("mode", [cx.OBS_SYM_U8_I8, cx.OBS_SYM_U8_F32])
@pytest.mark.parametrize("n", [3, 1499, 1500, 1501, 12289, 24577])
def test_classic_byte_observations_of_a_step(n, mode):
    assert _run(n, 10, cx.VARIANT_CLASSIC, obs_mode=mode, max_episode_steps=4) > 0


# written through up to 85 MiB in all (16,529 environments), left in the L2 beyond
@pytest.mark.parametrize("n,lanes", [(1, 0), (5, 0), (66, 0), (700, 0), (12289, 0), (16529, 0), (16530, 0), (16531, 0), (24577, 0), (131, 4), (37, 8), (16529, 16), (16530, 16),
                                     (16531, 16)])
def test_classic_float_observations_of_a_step(n, lanes):
    assert _run(n, 10, cx.VARIANT_CLASSIC, obs_mode=cx.OBS_SYM_F32, max_episode_steps=4, group_lanes=lanes) > 0


# a turn of stores begins on a cache line wherever the buffer does, and writes nothing beside the observations
@pytest.mark.parametrize("lanes", [4, 8, 16])
@pytest.mark.parametrize("n,shift", [(1, 0), (3, 16), (17, 48), (67, 80), (130, 112)])
def test_classic_float_observations_in_a_buffer_off_the_cache_lines(n, shift, lanes):
    sim = cx.Craftax(n, cx.default_config(obs_mode=cx.OBS_SYM_F32, max_episode_steps=6, group_lanes=lanes))
    sim.reset(synth.seeds_for(n))
    size, guard = sim.obs.numel(), 4096
    room = torch.empty(size + 2 * guard, dtype=torch.uint8, device=sim.device)
    assert room.data_ptr() % 128 == 0
    steps, lo = 9, guard + shift
    actions = torch.empty((steps, n), dtype=torch.int32, device=sim.device)
    cx.craftax_synth_actions(actions, n, 0, steps, 3, 1, sim.stream)
    reward, done = torch.empty((steps, n), device=sim.device), torch.empty((steps, n), dtype=torch.uint8, device=sim.device)

    def check(step):
        room.fill_(0x5A)
        step(room[lo:lo + size])
        cx.craftax_observe(sim.state, sim.obs, n, sim.stream)
        assert torch.equal(room[lo:lo + size], sim.obs.view(-1)), "observation"
        assert bool((room[:lo] == 0x5A).all()) and bool((room[lo + size:] == 0x5A).all()), "bytes beside the observations"

    for t in range(steps):
        check(lambda obs: cx.craftax_step(sim.state, actions[t], obs, reward[t], done[t], n, sim.stream))
    check(lambda obs: cx.craftax_rollout(sim.state, actions, steps, obs, reward, done, n, sim.stream))


# floats left in the L2 (up to 31 environments), written through (up to 85 MiB in all, 2,688 environments), left in the L2 (up to 240 MiB,
# 7,591), then written through by every fourth block where they start within the first 256 MiB (up to environment 8,097, in step
# and observing blocks whose number divides by four) and streamed beyond; bytes streamed
@pytest.mark.parametrize("n,mode", [(1, cx.OBS_SYM_F32), (5, cx.OBS_SYM_F32), (31, cx.OBS_SYM_F32), (32, cx.OBS_SYM_F32), (2688, cx.OBS_SYM_F32), (2689, cx.OBS_SYM_F32), (7591, cx.OBS_SYM_F32), (7592, cx.OBS_SYM_F32), (8101, cx.OBS_SYM_F32),
                                    (5, cx.OBS_SYM_U8_F32)])
def test_craftax_observations_of_a_step(n, mode):
    assert _run(n, 8, cx.VARIANT_CRAFTAX, obs_mode=mode, max_episode_steps=3) > 0


@pytest.mark.parametrize("n", [33, 2700, 7600])
def test_craftax_floats_of_a_perlin_step(n):
    assert _run(n, 6, cx.VARIANT_CRAFTAX, obs_mode=cx.OBS_SYM_F32, max_episode_steps=3, worldgen=cx.WORLDGEN_PERLIN) > 0


# as for Classic: streamed, written through from 32 MiB on (196 pictures), by every fourth block from 85 MiB on (520); beyond the first
# 256 MiB all are streamed, of 1,565 pictures the last one, whose block would write through
@pytest.mark.parametrize("n", [1, 3, 195, 196, 519, 520, 1564, 1565])
def test_craftax_pictures_of_a_step(n):
    assert _run(n, 8, cx.VARIANT_CRAFTAX, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=3) > 0


# beyond 8,192 environments the window of a spare world's start is fetched only when an episode ends
@pytest.mark.parametrize("worldgen", [cx.WORLDGEN_VALUE, cx.WORLDGEN_PERLIN])
def test_craftax_pictures_of_a_step_of_a_large_batch(worldgen):
    assert _run(8193, 5, cx.VARIANT_CRAFTAX, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=2, worldgen=worldgen) > 0


def test_craftax_pictures_of_a_perlin_step_with_sixteen_lanes():
    assert _run(9, 8, cx.VARIANT_CRAFTAX, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=3, worldgen=cx.WORLDGEN_PERLIN, group_lanes=16) > 0


@pytest.mark.parametrize("variant,n", [("classic", 1500), ("craftax", 700)])
def test_pictures_of_a_captured_step_that_ends_an_episode_without_a_spare_world(variant, n):
    """A graph captured while no edit was pending launches no kernel behind the step.  All episodes start anew in one replay;
    swaps then put lava beside the start of some, which the next replay walks into: their next world is not ready, the
    state in memory stays as it is, and that is what the picture has to show."""
    full, cap = variant == "craftax", 5
    sim = cx.Craftax(n, cx.default_config(cx.VARIANT_CRAFTAX if full else cx.VARIANT_CLASSIC, obs_mode=cx.OBS_PIXELS_F32, max_episode_steps=cap))
    sim.reset(synth.seeds_for(n, 900))
    actions = torch.zeros(n, dtype=torch.int32, device=sim.device)
    seen = torch.empty_like(sim.obs)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            cx.craftax_step(sim.state, actions, sim.obs, sim.reward, sim.done, n, torch.cuda.current_stream())
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()

    def replay(what):
        graph.replay()
        torch.cuda.synchronize()
        cx.craftax_observe(sim.state, seen, n, sim.stream)
        assert torch.equal(sim.obs.view(torch.uint8), seen.view(torch.uint8)), what
        return sim.done.cpu().numpy().astype(bool)

    for t in range(cap):
        ended = replay(f"observation at step {t}")
    assert ended.all()
    lava, c = 14, 24 if full else 32
    for round_ in range(400):
        cx.craftax_mutate_swap(sim.state, 0, n, 11, round_, False, None, sim.stream)
        if round_ % 20 == 19:
            d = sim.export_envs().view(sim.dump_dtype).reshape(-1)
            m = d["block"][:, 0] if full else d["map"].reshape(n, 64, 64)
            near = np.stack([m[:, c, c - 1], m[:, c, c + 1], m[:, c - 1, c], m[:, c + 1, c]], 1) == lava     # LEFT, RIGHT, UP, DOWN
            doomed = near.any(axis=1)
            if doomed.sum() >= 3:
                break
    assert doomed.any(), "no swap put lava next to a start: raise n or the number of rounds"
    actions.copy_(torch.as_tensor(np.where(doomed, 1 + near.argmax(axis=1), 0).astype(np.int32)))
    before = sim.export_envs()
    assert np.array_equal(replay("observation of the step into the lava"), doomed)
    assert np.array_equal(sim.export_envs()[doomed], before[doomed]), "nothing behind the step: the ended episodes stay in memory"
    actions.zero_()
    obs, _, _ = sim.step(actions)                               # the edit is still pending: this one serves them
    cx.craftax_observe(sim.state, seen, n, sim.stream)
    assert torch.equal(obs.view(torch.uint8), seen.view(torch.uint8))
    sim.close()
