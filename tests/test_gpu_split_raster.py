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
