"""GPU: bfloat16 renders where a step crosses 0.15 plane texels or more, whose
rows go through LDS with two lanes per row, against the float64 oracle of the
stored scene.

A batch's quads of lanes load for one another: n_max values leave every kind
of partial quad and batch.  Steps of 1/64 on the box of 2 x 2 x 1/4 cross 0.15
texels of planes of 21 x 21 x 4 texels (the smallest that qualify) and less
than that of 20 x 21 x 4.  Bar: counts exact, C, F and T within 1e-5; with and
without sparse blocks.
"""
import numpy as np
import pytest

import oracle
import paper_2404_09531_amd as om
import scenegen
import torch
from tests._scenes import micro_scene
from tests.gpu_util import bf16_round, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu

BG = (0.25, 0.5, 0.75)
SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")


@pytest.mark.parametrize("t_term,sparse", [(0.0, False), (0.3, False), (0.0, True)])
@pytest.mark.parametrize("planes", [(20, 21, 4), (21, 21, 4), (130, 257, 40)])
@pytest.mark.parametrize("n_max", [1, 2, 3, 6, 13, 16, 17, 64])
def test_two_lanes_per_row(planes, n_max, t_term, sparse):
    log(f"test_two_lanes_per_row: planes {planes}, n_max {n_max}, t_term {t_term}, sparse {sparse}")
    sc = micro_scene(grid=(21, 17, 9), planes=planes, m=8, zmin=0.02, zmax=0.23, seed=3)
    scene, t = upload_scene(sc, torch.bfloat16)
    if sparse:
        atlas, sg = om.sparse_grid(scene, 2)
        scene = om.Scene(atlas, t["plane_xy"], t["plane_xz"], t["plane_yz"], t["occ"], t["mlp"], sparse=sg)
    sc = dict(sc, **{k: bf16_round(sc[k]) for k in SOURCES})
    o, d = scenegen.oblique_rays(301, seed=9)
    d = d.copy()
    d[:, 2] *= 0.3  # shallow: up to 60 steps within the box
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    o = (np.array([0.0, 0.0, 0.12]) - 0.6 * d).astype(np.float32)
    o[:, :2] += np.random.default_rng(1).uniform(-0.3, 0.3, (301, 2)).astype(np.float32)
    kw = dict(n_max=n_max, delta=2.0 ** -6, c_bg=BG, t_term=t_term)
    res = om.render(scene, *rays_to(o, d), mlp_bf16=0, **kw)
    ref = oracle.oracle_render(sc, o, d, oracle.RenderParams(**kw), keep_k=False)
    if t_term == 0.0:  # with early termination it counts the samples placed up to the stop
        assert np.array_equal(res["n_placed"].cpu().numpy(), ref["n_placed"])
    assert np.array_equal(res["n_eval"].cpu().numpy(), ref["n_eval"])
    assert ref["n_placed"].max() >= min(n_max, 17)
    for key in ("C", "T", "F"):
        err = float(np.abs(res[key].double().cpu().numpy() - ref[key]).max())
        assert err <= 1e-5, (key, err)
