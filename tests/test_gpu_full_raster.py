"""The general raster (depth, primitive ids, mixed road colours) where its work
division can go wrong: bands that cut the image, widths below a 16-sample
group, list capacities and overflow, strips of any shape, far-off maps; bit for
bit against the oracle and the banded kernels."""
import dataclasses

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


def _check(scenes, cam, picks, label, light=None):
    from paper_2606_19641_amd import gp
    pal = g.mixed_palette()
    pal[0], pal[1] = (9, 70, 201), (150, 31, 4)
    pal[6:9] = g.default_palette()[6:9]
    sim = gp.Sim(scenes, cam, pal)
    sim.set_light(light)
    only, _, _ = sim.render()
    rgb, d, p = sim.render(depth=True, primid=True)
    for sched in (0, 1):
        sim.set_launch(raster=0, sched=sched)
        ref = sim.render(depth=True, primid=True)
        torch.cuda.synchronize()
        assert torch.equal(rgb, ref[0]) and torch.equal(p, ref[2]), (label, "banded")
        assert torch.equal(d.view(torch.int32), ref[1].view(torch.int32)), (label, "banded depth")
    assert torch.equal(only, rgb), (label, "rgb only")
    n_cams = len(cam.cam_dirs)
    base = np.cumsum([0] + [s.n_agents for s in scenes])
    rgb, d, p = rgb.cpu().numpy(), d.cpu().numpy(), p.cpu().numpy()
    for si, a, k in picks:
        ref = oracle.render_scene_view(scenes[si], cam, pal, a, k, light=light)
        v = (base[si] + a) * n_cams + k
        assert np.array_equal(rgb[v], ref.rgb), (label, si, a, k)
        assert np.array_equal(p[v], ref.primid), (label, si, a, k)
        assert np.array_equal(d[v].view(np.uint32), ref.depth.view(np.uint32)), (label, si, a, k)


def _one_colour(s):
    s.road_color[:] = 1
    return s


@pytest.mark.parametrize("n_agents", [1, 43, 44, 86, 170, 300])
@pytest.mark.parametrize("lit", [None, (0.6, -0.48, 0.64, 0.25)])
def test_list_capacities_and_overflow(n_agents, lit):
    print(f"general raster list: {n_agents} agents, light {lit}", flush=True)
    s = g.crowded_scene(500 + n_agents, n_agents=n_agents, n_roads=50, radius=10.0)
    rng = np.random.default_rng(n_agents)
    q = 70 if n_agents == 300 else 3
    s.signal_xyzr = np.stack([rng.uniform(-12, 12, q), rng.uniform(-12, 12, q), rng.uniform(0.5, 4, q),
                              rng.uniform(0.1, 1.2, q)], 1).astype(np.float32)
    s.signal_color = rng.integers(6, 9, q).astype(np.uint8)
    cam = g.camera_for(48, cams=g.FRONT_AND_SIDES)
    _check([s], cam, [(0, a, k) for a in range(0, n_agents, max(1, n_agents // 2)) for k in range(3)], n_agents, lit)


@pytest.mark.parametrize("size", [(1, 1), (5, 40), (15, 17), (16, 16), (17, 30), (210, 126), (333, 41), (64, 700)])
def test_sizes_and_bands(size):
    print(f"general raster size {size}", flush=True)
    scenes = [_one_colour(g.crowded_scene(77 + size[0], n_agents=7, n_roads=120, radius=15.0)),
              g.crowded_scene(78, n_agents=2, n_roads=1500, radius=30.0)]
    cam = g.Camera(width=size[0], height=size[1], focal_px=max(size[0] / 2.0, 4.0), cam_dirs=g.FRONT_AND_SIDES)
    for some in (scenes[:1], scenes):            # one road colour, mixed ones (and more strips than the ring holds)
        _check(some, cam, [(0, a, k) for a in (0, 3, 6) for k in range(3)], (size, len(some)))


@pytest.mark.parametrize("shift", [0.0, 500.0, 20000.0])
@pytest.mark.parametrize("colours", [1, 2])
def test_odd_strips_and_far_maps(shift, colours):
    """Strips of any shape (self-crossing, needle-thin, clockwise, huge, with
    corners on one row) under and around the camera: quads, fan triangles and
    the clipper, through the rgb-only rasters (one colour) and the general one."""
    print(f"odd strips at {shift}, {colours} colours", flush=True)
    rng = np.random.default_rng(11)
    s = g.crowded_scene(12, n_agents=6, n_roads=8, radius=8.0)
    n = 400
    c = rng.uniform(-40, 40, (n, 1, 2))
    q = c + rng.uniform(-6, 6, (n, 4, 2)) * rng.choice([0.02, 0.3, 1.0, 6.0, 200.0], (n, 1, 1))
    q[:40, 2] = q[:40, 0] + (q[:40, 1] - q[:40, 0]) * 3.0          # degenerate and crossing quads
    q[40:90, 1, 0] = q[40:90, 0, 0]                                # edges along the axes
    q[40:90, 3, 0] = q[40:90, 2, 0]
    roads = np.concatenate([s.road_xy.astype(np.float64), q])
    s = dataclasses.replace(s, road_xy=(roads + shift).astype(np.float32),
                            road_color=(1 + (np.arange(len(roads)) % colours) * 4).astype(np.uint8),
                            agent_state=(s.agent_state + np.array([shift, shift, 0, 0])).astype(np.float32))
    cam = g.camera_for(72, 56, g.STUDENT_RIG)
    _check([s], cam, [(0, a, k) for a in range(6) for k in range(4)], shift)


def _check_split(scenes, cam, picks, label, light=None):
    """The general raster asked for by name, against the banded kernels on every
    view and the oracle on the picked ones."""
    from paper_2606_19641_amd import gp
    pal = g.mixed_palette()
    pal[0], pal[1] = (9, 70, 201), (150, 31, 4)
    pal[6:9] = g.default_palette()[6:9]
    sim = gp.Sim(scenes, cam, pal)
    sim.set_light(light)
    sim.set_launch(raster=1)
    only, _, _ = sim.render()
    rgb, d, p = sim.render(depth=True, primid=True)
    sim.set_launch(raster=0)
    ref = sim.render(depth=True, primid=True)
    torch.cuda.synchronize()
    assert torch.equal(only, rgb), (label, "rgb only")
    assert torch.equal(rgb, ref[0]) and torch.equal(p, ref[2]), (label, "banded")
    assert torch.equal(d.view(torch.int32), ref[1].view(torch.int32)), (label, "banded depth")
    n_cams = len(cam.cam_dirs)
    base = np.cumsum([0] + [s.n_agents for s in scenes])
    rgb, d, p = rgb.cpu().numpy(), d.cpu().numpy(), p.cpu().numpy()
    for si, a, k in picks:
        ref = oracle.render_scene_view(scenes[si], cam, pal, a, k, light=light)
        v = (base[si] + a) * n_cams + k
        assert np.array_equal(rgb[v], ref.rgb), (label, si, a, k)
        assert np.array_equal(p[v], ref.primid), (label, si, a, k)
        assert np.array_equal(d[v].view(np.uint32), ref.depth.view(np.uint32)), (label, si, a, k)


@pytest.mark.parametrize("n_agents,radius,scenes,size", [
    (40, 10.0, 8, (64, 48)),       # lists that grow into the ring and the staging
    (64, 6.0, 1, (48, 48)),        # as many boxes as records, in sixteen wavefronts
    (65, 12.0, 1, (130, 40)),      # one more
    (90, 14.0, 1, (17, 61)),
    (110, 8.0, 1, (300, 210)),     # streamed by eight wavefronts
    (150, 5.0, 2, (64, 64)),       # streamed by four, more faces at once than the list holds
])
@pytest.mark.parametrize("lights", [0, 130])
@pytest.mark.parametrize("colours", [1, 2])
def test_crowds_through_the_split_division(n_agents, radius, scenes, size, lights, colours):
    print(f"general raster crowd: {scenes} x {n_agents} agents at {size}, {lights} lights, {colours} colours", flush=True)
    sc = [g.crowded_scene(700 + n_agents + k, n_agents=n_agents, n_roads=50, radius=radius) for k in range(scenes)]
    rng = np.random.default_rng(n_agents)
    for s in sc:
        if colours == 1:
            s.road_color[:] = 1
        if lights:
            s.signal_xyzr = np.stack([rng.uniform(-12, 12, lights), rng.uniform(-12, 12, lights),
                                      rng.uniform(0.5, 4, lights), rng.uniform(0.1, 1.2, lights)], 1).astype(np.float32)
            s.signal_color = rng.integers(6, 9, lights).astype(np.uint8)
    cam = g.Camera(width=size[0], height=size[1], focal_px=size[0] / 2.0, cam_dirs=g.FRONT_AND_SIDES)
    light = (0.6, -0.48, 0.64, 0.25) if lights else None
    _check_split(sc, cam, [(scenes - 1, a, k) for a in (0, n_agents // 2) for k in (0, 2)], (n_agents, size), light)


@pytest.mark.parametrize("size,raster", [((16, 16), 1), (g.STUDENT_RESOLUTIONS[0], 1), ((48, 48), 1), ((333, 41), 1),
                                         ((128, 128), 1), ((15, 15), 0), ((1, 9), 0)])
@pytest.mark.parametrize("colours", [1, 2])
def test_default_work_division(size, raster, colours):
    """Nobody asked for the banded kernels: from 16 samples a row on, sims of any
    road colours divide a view's work over its wavefronts, at ragged widths too; below,
    that division runs in no launch setting."""
    from paper_2606_19641_amd import gp
    print(f"default launch at {size}, {colours} colours", flush=True)
    s = g.crowded_scene(31, n_agents=7, n_roads=90, radius=15.0)
    if colours == 1:
        s.road_color[:] = 1
    cam = g.Camera(width=size[0], height=size[1], focal_px=max(size[0] / 2.0, 4.0), cam_dirs=g.FRONT_AND_SIDES)
    sim = gp.Sim([s], cam, g.mixed_palette())
    assert sim.get_launch()["raster"] == raster
    _check([s], cam, [(0, a, k) for a in (0, 4) for k in range(3)], (size, colours))
    _check_split([s], cam, [], (size, colours, "asked for"))


@pytest.mark.parametrize("first", [0, 1, 2])
def test_batch_of_mixed_and_single_colours(first):
    """A batch whose first sim has mixed road colours: the others take the split
    raster, and every sim gets what it gets alone."""
    from paper_2606_19641_amd import gp
    print(f"batch of mixed colours, sim {first} first", flush=True)
    scenes = [g.crowded_scene(41 + k, n_agents=6 + 5 * k, n_roads=60) for k in range(3)]
    scenes[1].road_color[:] = 1
    scenes[2].road_color[:] = 1
    scenes[2].signal_xyzr = np.array([[6.0, 1.0, 3.0, 0.5]], np.float32)
    scenes[2].signal_color = np.array([6], np.uint8)
    scenes = scenes[first:] + scenes[:first]
    cam, pal = g.camera_for(80, 50), g.default_palette()
    sims, alone = ([gp.Sim([s], cam, pal) for s in scenes] for _ in range(2))
    nb = gp.batch_required_bytes(sims)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    staging = torch.empty(nb, dtype=torch.uint8, pin_memory=True)
    rgbs = [x.new_rgb() for x in sims]
    for step in range(2):
        acts = [g.actions(5, step, np.full(s.n_agents, i), np.arange(s.n_agents)) for i, s in enumerate(scenes)]
        gp.batch_step_render(sims, acts, rgbs, ws, staging)
        torch.cuda.synchronize()
        for x, a, r, y in zip(alone, acts, rgbs, sims):
            x.step(torch.from_numpy(a).cuda())
            ref, _, _ = x.render()
            x.set_launch(raster=0)
            banded, _, _ = x.render()
            x.set_launch(raster=1)
            torch.cuda.synchronize()
            assert torch.equal(r, ref) and torch.equal(r, banded) and torch.equal(x.get_state(), y.get_state()), step
