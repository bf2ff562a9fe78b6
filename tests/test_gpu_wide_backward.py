"""GPU: training steps on a grid whose index factors pass 24 bits (2 x 4100 x
4100 vertices, 1.1 GB in float32), which take the 64-bit address forms of the
forward with per-batch sums or records and of the backward; 8,192 rays are the
line between the backward's two forms.

Bar: the per-entry bar of tests/gradcheck.py.  201 copies of 41 rays stand for a
batch past that line: 201 times the gradient and the terms.  A step with records
is compared with the replay (test_gpu_records.py), which is checked here.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09531_amd as om
import scenegen
from tests._scenes import micro_scene
from tests.gpu_util import DEV, bf16_round, log, rays_to, upload_scene
from tests.gradcheck import SOURCES, check, oracle_reference, oracle_upstream
from tests.test_gpu_records import Step, assert_same, oblique

pytestmark = pytest.mark.gpu

BG = (0.25, 0.5, 0.75)
N_MAX = 100


def tall(planes):
    sc = micro_scene(grid=(2, 3, 2), planes=planes, m=8, zmin=0.05, zmax=0.2, seed=3)
    sc["grid"] = np.empty((4100, 4100, 2, 8), np.float32)
    scenegen.fill_normal(sc["grid"], 0.5, np.random.SeedSequence(5))
    return sc


@pytest.fixture(scope="module")
def tall_coarse():
    return tall((70, 34, 18))


@pytest.mark.parametrize("occ_eps", [0.0, 0.02])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_wide_backward_vs_oracle(tall_coarse, dtype, occ_eps):
    log(f"test_wide_backward_vs_oracle: {dtype}, occ_eps {occ_eps}")
    sc = tall_coarse
    scene, t = upload_scene(sc, dtype)
    if dtype == torch.bfloat16:
        sc = dict(sc, **{k: bf16_round(sc[k]) for k in SOURCES})
    o, d = scenegen.oblique_rays(41, seed=8)
    prm = oracle.RenderParams(n_max=N_MAX, c_bg=BG, occ_eps=occ_eps)
    target = np.random.default_rng(9).uniform(0, 1, (41, 3)).astype(np.float32)
    up, _ = oracle_upstream(sc, o, d, prm, target)
    ref1, scale1 = oracle_reference(sc, o, d, prm, up)
    keys = (*SOURCES, "mlp") + (("occ",) if occ_eps else ())
    kw = dict(n_max=N_MAX, c_bg=BG, occ_eps=occ_eps)
    for copies in (1, 201):
        at = np.random.default_rng(2).permutation(np.tile(np.arange(41), copies))
        og, dg = rays_to(o[at], d[at])
        dC = torch.from_numpy(up[at]).to(DEV)
        times = lambda r: (r[0], copies * r[1]) if isinstance(r, tuple) else copies * r  # noqa: E731
        ref = {k: times(v) for k, v in ref1.items()}
        scale = {k: (*v[:-3], *(copies * x for x in v[-3:])) for k, v in scale1.items()}
        for batch_wv in (False, True):
            res = om.render(scene, og, dg, mlp_bf16=0, batch_wv=batch_wv, **kw)
            grads = {k: torch.zeros(t[k].shape, device=DEV) for k in keys}
            om.render_backward(scene, og, dg, res, dC, grads, **kw)
            check({k: v.cpu().numpy() for k, v in grads.items()}, ref, scale,
                  f"{dtype}, {41 * copies} rays, batch_wv {batch_wv}")


@pytest.mark.parametrize("occ_eps", [0.0, 0.02])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_wide_step_with_records(dtype, occ_eps):
    log(f"test_wide_step_with_records: {dtype}, occ_eps {occ_eps}")
    s = Step(tall((1700, 1660, 210)), *oblique(76003), dtype=dtype, occ=occ_eps > 0, n_max=256, occ_eps=occ_eps)
    assert s.records > 0
    plain, recorded = s.both()
    assert int(((plain[0]["n_placed"] + 15) // 16).sum()) >= 1 << 19
    assert_same(plain, recorded)
