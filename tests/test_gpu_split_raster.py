"""The wave-split rgb raster at the edges of its lists and sizes, against the
general kernel (same sim, depth and primitive ids asked for) and the oracle:
every comparison is bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2606_19641_amd import scenegen as g

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_19641_amd import gp
    gp.lib()


def _crowd(seed, n_agents, n_roads=40, radius=25.0):
    s = g.crowded_scene(seed, n_agents=n_agents, n_roads=n_roads, radius=radius)
    s.road_color[:] = 1
    return s


def _check(sim, scenes, cam, pal, picks, label):
    """rgb-only image = the oracle's on the picked (scene, agent, camera) views
    and the banded raster's on every view."""
    rgb, _, _ = sim.render()
    keep = sim.get_launch()
    sim.set_launch(raster=0)
    ref, _, _ = sim.render()
    sim.set_launch(**keep)
    torch.cuda.synchronize()
    bad = (rgb != ref).flatten(1).any(1).nonzero().flatten().tolist()
    assert not bad, (label, bad[:8])
    base = np.cumsum([0] + [s.n_agents for s in scenes])
    out = rgb.cpu().numpy()
    for si, a, k in picks:
        r = oracle.render_scene_view(scenes[si], cam, pal, a, k)
        assert np.array_equal(out[(base[si] + a) * len(cam.cam_dirs) + k], r.rgb), (label, si, a, k)


@pytest.mark.parametrize("n_agents", [1, 32, 33, 64, 65, 128, 200])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_box_list_sizes(n_agents, waves):
    """Scenes on both sides of the list capacities (64, 128, 256 faces), one
    crowded enough for views to overflow theirs, boxes across the near plane
    and seen from above."""
    print(f"box list: {n_agents} agents, {waves} wavefronts", flush=True)
    scenes = [_crowd(900 + n_agents, n_agents, radius=14.0), _crowd(950 + n_agents, min(n_agents, 5), radius=40.0)]
    cam = g.camera_for(64, cams=g.FRONT_AND_SIDES)
    pal = g.mixed_palette()
    from paper_2606_19641_amd import gp
    sim = gp.Sim(scenes, cam, pal)
    sim.set_launch(raster=1, view_waves=waves)
    picks = [(0, a, k) for a in range(0, n_agents, max(1, n_agents // 3)) for k in range(3)]
    _check(sim, scenes, cam, pal, picks, (n_agents, waves))


@pytest.mark.parametrize("size", [(16, 16), (17, 9), (31, 33), (48, 1), (63, 40), (65, 64), (210, 126), (337, 100),
                                  (434, 252), (250, 801)])
def test_widths_and_alignments(size):
    """Any width from 16 on (groups of 16 samples that overlap at the row end,
    coverage bits that run on from row to row), images whose size and address
    are no multiple of 16 bytes, every wavefront count, bytes around the image
    left alone."""
    print(f"split raster at {size}", flush=True)
    W, H = size
    scenes = [_crowd(60 + W, 9, n_roads=150), _crowd(61 + W, 3, n_roads=0)]
    cam = g.Camera(width=W, height=H, focal_px=W / 2.0, cam_dirs=g.FRONT_AND_SIDES)
    pal = g.mixed_palette()
    pal[0] = (9, 70, 201)                       # every channel of sky and road differs
    pal[1] = (150, 31, 4)
    from paper_2606_19641_amd import gp
    sim = gp.Sim(scenes, cam, pal)
    picks = [(0, a, k) for a in (0, 4, 8) for k in range(3)] + [(1, 1, 0)]
    for waves in (1, 2, 4):
        sim.set_launch(raster=1, view_waves=waves)
        _check(sim, scenes, cam, pal, picks, (size, waves))
    ref, _, _ = sim.render()
    for off in (4, 8, 12):
        buf = torch.full((ref.numel() + 64,), 77, dtype=torch.uint8, device="cuda")
        sim.render(rgb=buf[off:off + ref.numel()].view(ref.shape))
        torch.cuda.synchronize()
        assert torch.equal(buf[off:off + ref.numel()].view(ref.shape), ref), (size, off)
        assert bool((buf[:off] == 77).all()) and bool((buf[off + ref.numel():] == 77).all()), (size, off)


@pytest.mark.parametrize("scenes", [1, 3, 9])
def test_wavefronts_for_few_views(scenes):
    """Few views take up to 16 wavefronts each (small box units, many set-up jobs)."""
    sc = [_crowd(300 + k, 12 + 31 * (k % 2), n_roads=90 + 400 * (k % 3)) for k in range(scenes)]
    cam = g.camera_for(96)
    pal = g.mixed_palette()
    from paper_2606_19641_amd import gp
    sim = gp.Sim(sc, cam, pal)
    for waves in (1, 2, 4):
        sim.set_launch(raster=1, view_waves=waves)
        _check(sim, sc, cam, pal, [(0, a, 0) for a in range(4)], (scenes, waves))


def _street(seed, n_agents, n_static, n_signals, radius=20.0):
    """A crowd with obstacles and lights all around it, some of the lights close
    to the cameras and cut by the near plane, one colour of road."""
    s = _crowd(seed, n_agents, n_roads=60, radius=radius)
    rng = np.random.default_rng(seed)
    k = n_static
    s.static_xyp = np.stack([rng.uniform(-radius, radius, k), rng.uniform(-radius, radius, k),
                             rng.uniform(-3, 3, k)], 1).astype(np.float32)
    s.static_dims = np.stack([rng.uniform(1, 6, k), rng.uniform(0.5, 2, k), rng.uniform(0.5, 2, k)], 1).astype(np.float32)
    s.static_color = np.full(k, 4, np.uint8)
    q = n_signals
    s.signal_xyzr = np.stack([rng.uniform(-radius, radius, q), rng.uniform(-radius, radius, q), rng.uniform(0.5, 5, q),
                              rng.uniform(0.1, 1.5, q)], 1).astype(np.float32)
    s.signal_color = rng.integers(6, 9, q).astype(np.uint8)
    return s


@pytest.mark.parametrize("lit", [False, True])
@pytest.mark.parametrize("counts", [(4, 0, 1), (6, 3, 64), (5, 2, 65), (30, 20, 0), (90, 100, 130)])
def test_light_and_traffic_lights(counts, lit):
    """The instances with the directional light and traffic lights: up to one
    light unit and more, a list that overflows (boxes and lights streamed), the
    state colours changing; alone and in a batch with a plain sim."""
    print(f"appearance: {counts} lit {lit}", flush=True)
    from paper_2606_19641_amd import gp
    scenes = [_street(70 + sum(counts), *counts), _street(71, 3, 1, 2)]
    cam = g.camera_for(80, 64, g.FRONT_AND_SIDES)
    pal = g.mixed_palette()
    pal[6:9] = ((255, 32, 32), (255, 200, 0), (32, 224, 64))
    sims = [gp.Sim([s], cam, pal) for s in scenes] + [gp.Sim([_crowd(72, 6)], cam, pal)]
    both = gp.Sim(scenes, cam, pal)
    for s in sims[:2] + [both]:
        s.set_light((0.6, -0.48, 0.64, 0.25) if lit else None)
    n = counts[0]
    for waves in (1, 2, 4):
        for step in range(2):
            if step and both.n_signals:
                both.set_signal_colors(torch.from_numpy(np.roll(np.concatenate([s.signal_color for s in scenes]), 1)).cuda())
            both.set_launch(raster=1, view_waves=waves)
            rgb, _, _ = both.render()
            ref, _, _ = both.render(depth=True, primid=True)
            torch.cuda.synchronize()
            assert torch.equal(rgb, ref), (counts, lit, waves, step)
    # a batch: the plain sim and the two streets, each as alone
    acts = [np.zeros((s.n_agents, 2), np.float32) for s in sims]
    alone = []
    for s, a in zip(sims, acts):
        keep = s.get_state()
        s.step(torch.from_numpy(a).cuda())
        alone.append(s.render(depth=True, primid=True)[0])
        s.set_state(keep)
    nb = gp.batch_required_bytes(sims)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    st = torch.empty(nb, dtype=torch.uint8, pin_memory=True)
    out = [s.new_rgb() for s in sims]
    gp.batch_step_render(sims, acts, out, ws, st)
    torch.cuda.synchronize()
    for k in range(3):
        assert torch.equal(out[k], alone[k]), (counts, lit, "batch", k)
    assert n == sims[0].n_agents


@pytest.mark.parametrize("n_roads", [4090, 4112, 9000])
@pytest.mark.parametrize("waves", [1, 4])
def test_more_culling_bins_than_the_list_holds(n_roads, waves):
    """Views that keep about as many culling bins as their list holds (256) and
    more: the bins are then taken in segments."""
    print(f"bins: {n_roads} strips, {waves} wavefronts", flush=True)
    scenes = [_crowd(41, 6, n_roads=n_roads, radius=20.0), _crowd(42, 2, n_roads=30)]
    cam = g.camera_for(64, cams=g.FRONT_AND_SIDES)
    pal = g.mixed_palette()
    from paper_2606_19641_amd import gp
    sim = gp.Sim(scenes, cam, pal)
    sim.set_launch(raster=1, view_waves=waves)
    _check(sim, scenes, cam, pal, [(0, a, k) for a in (0, 5) for k in range(3)], (n_roads, waves))


@pytest.mark.parametrize("z_near", [0.01, 0.2])
def test_spans_beyond_the_fp64_range(z_near):
    """Strips and boxes that reach 2^25 subpixels and more (long ones cut by a
    close near plane, a long focal length): their spans are counted in int64."""
    print(f"int64 spans: near {z_near}", flush=True)
    rng = np.random.default_rng(5)
    s = _crowd(43, 7, n_roads=160, radius=6.0)
    a = rng.uniform(0, 2 * np.pi, 160)
    c = rng.uniform(-4, 4, (160, 2))
    u, v = np.stack([np.cos(a), np.sin(a)], 1) * 150.0, np.stack([-np.sin(a), np.cos(a)], 1) * rng.uniform(0.05, 3, (160, 1))
    s.road_xy[:] = np.stack([c - u - v, c + u - v, c + u + v, c - u + v], 1).astype(np.float32)
    s.agent_dims[:, 0] = 12.0
    cam = g.Camera(width=96, height=70, focal_px=900.0, z_near=z_near, cam_dirs=g.FRONT_AND_SIDES)
    pal = g.mixed_palette()
    from paper_2606_19641_amd import gp
    sim = gp.Sim([s], cam, pal)
    _check(sim, [s], cam, pal, [(0, a, k) for a in range(7) for k in range(3)], z_near)


@pytest.mark.parametrize("case", ["one agent", "small scenes", "several cameras", "lists overflow", "lit, lists overflow"])
def test_render_that_steps_the_agents(case):
    """step_render_graph and a batch, where the raster steps the agents itself,
    against a step and a render apart: images and states over several steps,
    some agents halted, scenes of one to more than 64 agents."""
    from paper_2606_19641_amd import gp
    print(f"stepping render: {case}", flush=True)
    scenes = {"one agent": lambda: [_crowd(1, 1)],
              "small scenes": lambda: [_crowd(10 + k, 1 + k) for k in range(40)],
              "several cameras": lambda: [_crowd(2, 63), _crowd(3, 64), _crowd(4, 65, radius=60.0), _crowd(5, 3)],
              "lists overflow": lambda: [_crowd(6, 200, radius=12.0), _crowd(7, 2)],
              "lit, lists overflow": lambda: [_street(8, 90, 100, 130), _street(9, 5, 2, 1)]}[case]()
    cam = g.camera_for(48, cams=g.FRONT_AND_SIDES if case != "one agent" else g.FRONT)
    pal = g.mixed_palette()
    pal[6:9] = ((255, 32, 32), (255, 200, 0), (32, 224, 64))
    a, b, c = (gp.Sim(scenes, cam, pal) for _ in range(3))
    for s in (a, b, c):
        s.set_launch(raster=1)
        if case.startswith("lit"):
            s.set_light((0.6, -0.48, 0.64, 0.25))
        if case in ("several cameras", "lists overflow"):
            s.check_infractions()                    # halts the agents that overlap others
    nb = gp.batch_required_bytes([c])
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    st = torch.empty(nb, dtype=torch.uint8, pin_memory=True)
    out, batch = b.new_rgb(), c.new_rgb()
    n = sum(s.n_agents for s in scenes)
    for k in range(4):
        act = g.batch_actions(77, k, scenes)
        dev = torch.from_numpy(act).cuda()
        a.step(dev)
        ref, _, _ = a.render()
        b.step_render_graph(dev, out)
        gp.batch_step_render([c], [act], [batch], ws, st)
        torch.cuda.synchronize()
        for s, img, how in ((b, out, "step_render_graph"), (c, batch, "batch")):
            assert torch.equal(img, ref), (case, k, how)
            assert torch.equal(s.get_state().view(torch.int32), a.get_state().view(torch.int32)), (case, k, how)
    assert n == a.n_agents
