"""The routes that set_state and fork choose between, and every state call inside
a captured graph: the same states, flags and images by each."""
import numpy as np
import pytest

from paper_2606_19641_amd import scenegen as g

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_19641_amd import gp
    gp.lib()


def _scenes():
    scenes = [g.crowded_scene(51 + k, n_agents=5 + 20 * k, n_roads=50, radius=20.0) for k in range(3)]
    for s in scenes:
        s.road_color[:] = 1
    scenes[1].signal_xyzr = np.array([[6.0, 1.0, 3.0, 0.5], [8.0, -3.0, 4.0, 0.3]], np.float32)
    scenes[1].signal_color = np.array([6, 7], np.uint8)
    return scenes


def _same(a, b):
    return torch.equal(a.get_state().view(torch.int32), b.get_state().view(torch.int32)) and torch.equal(
        a.get_actuators().view(torch.int32), b.get_actuators().view(torch.int32))


@pytest.mark.parametrize("src", ["device", "odd address", "pinned host"])
def test_set_state_from_any_memory(src):
    """One kernel for device memory at 4-byte alignment, the runtime's copy for the
    rest; a new episode either way (nobody halted, actuators at rest)."""
    from paper_2606_19641_amd import gp
    print(f"set_state from {src}", flush=True)
    scenes = _scenes()
    cam, pal = g.camera_for(32), g.default_palette()
    a, b = gp.Sim(scenes, cam, pal), gp.Sim(scenes, cam, pal)
    state = torch.from_numpy(np.concatenate([s.agent_state for s in scenes]) + np.float32(0.25)).contiguous()
    act = torch.from_numpy(g.batch_actions(3, 0, scenes)).cuda()
    jerk = torch.full((a.n_agents,), 3, dtype=torch.uint8, device="cuda")
    for s in (a, b):
        s.step_jerk(jerk)
        s.check_infractions()                        # some are halted now
    a.set_state(state.cuda())
    nbytes = 4 * state.numel()
    if src == "pinned host":
        buf = torch.empty(nbytes, dtype=torch.uint8, pin_memory=True)
    else:
        buf = torch.empty(nbytes + 64, dtype=torch.uint8, device="cuda")
        buf = buf[1:1 + nbytes] if src == "odd address" else buf[4:4 + nbytes]
    buf.copy_(state.view(torch.uint8).flatten())
    torch.cuda.synchronize()
    st = gp.lib().gp_sim_set_state(b._h, buf.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == gp.GP_OK, gp.lib().gp_last_error()
    torch.cuda.synchronize()
    assert _same(a, b)
    assert torch.equal(b.get_state().cpu(), state)
    for s in (a, b):
        s.step(act)
        s.step_jerk(jerk)
    assert _same(a, b) and torch.equal(a.render()[0], b.render()[0])


def test_state_calls_in_a_captured_graph():
    """set_state, fork, the stepping render, the jerk step and the infraction check
    recorded into one graph; replays with eager work between them give what the
    same calls give eagerly."""
    from paper_2606_19641_amd import gp
    scenes = _scenes()
    cam, pal = g.camera_for(48), g.default_palette()
    sims = [gp.Sim(scenes, cam, pal) for _ in range(4)]
    rgb = [s.new_rgb() for s in sims]
    n = sims[0].n_agents
    flags = [torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2)]
    src = sims[0].get_state()
    act = torch.zeros((n, 2), device="cuda")
    jerk = torch.zeros(n, dtype=torch.uint8, device="cuda")
    lights = torch.zeros(sims[0].n_signals, dtype=torch.uint8, device="cuda")

    def calls(a, b, img_a, img_b, fl):
        a.set_state(src)
        a.set_signal_colors(lights)
        for _ in range(2):
            a.step_render_graph(act, img_a)
        a.step_jerk(jerk)
        a.check_infractions(fl)
        b.fork_from(a)
        b.step_render_graph(act, img_b)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        calls(sims[0], sims[1], rgb[0], rgb[1], flags[0])        # warm up
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(sims[0], sims[1], rgb[0], rgb[1], flags[0])
    rng = np.random.default_rng(9)
    first = np.concatenate([s.agent_state for s in scenes])
    for k in range(4):
        print(f"replay {k}", flush=True)
        src.copy_(torch.from_numpy(first + rng.uniform(-1, 1, first.shape).astype(np.float32)))
        act.copy_(torch.from_numpy(rng.uniform(-2, 2, (n, 2)).astype(np.float32)))
        jerk.copy_(torch.from_numpy(rng.integers(0, 12, n).astype(np.uint8)))
        lights.copy_(torch.from_numpy(rng.integers(6, 9, lights.numel()).astype(np.uint8)))
        graph.replay()
        calls(sims[2], sims[3], rgb[2], rgb[3], flags[1])
        torch.cuda.synchronize()
        assert _same(sims[0], sims[2]) and _same(sims[1], sims[3]), k
        assert torch.equal(rgb[0], rgb[2]) and torch.equal(rgb[1], rgb[3]) and torch.equal(flags[0], flags[1]), k
        sims[0].step(act)                                         # eager work between the replays
        sims[1].render()
