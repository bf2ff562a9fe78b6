"""GPU: the forward's address forms and partial batches against the oracle.

A scene is addressed with 32-bit byte offsets and 24-bit index factors where
every source allows it; others take 64-bit addresses.  A grid of 2 x 4100 x
4100 vertices (1.1 GB in float32) has index factors beyond 24 bits and so takes
the latter.  The float32 forward shades a batch in quarters of 4 samples:
n_max values around the quarters' and the batch's edges leave every kind of
partial batch.  Bar: counts exact, C, F and T within 1e-5 of the float64
oracle (of the decoded scene for 16- and 8-bit storage).
"""
import numpy as np
import pytest
import torch

import oracle
import oracle.quant
import paper_2404_09531_amd as om
import scenegen
from tests._scenes import micro_scene
from tests.gpu_util import DEV, bf16_round, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu

BG = (0.25, 0.5, 0.75)
SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")


def _compare(res, ref, tag):
    assert np.array_equal(res["n_placed"].cpu().numpy(), ref["n_placed"])
    assert np.array_equal(res["n_eval"].cpu().numpy(), ref["n_eval"])
    for key in ("C", "T", "F"):
        err = float(np.abs(res[key].double().cpu().numpy() - ref[key]).max())
        log(f"  {tag}: max |{key} - oracle| = {err:.3e}")
        assert err <= 1e-5, (tag, key, err)


@pytest.fixture(scope="module")
def tall():
    sc = micro_scene(grid=(2, 3, 2), planes=(70, 34, 18), m=8, zmin=0.05, zmax=0.2, seed=3)
    sc["grid"] = np.empty((4100, 4100, 2, 8), np.float32)
    scenegen.fill_normal(sc["grid"], 0.5, np.random.SeedSequence(5))
    return sc


@pytest.mark.parametrize("dtype", ["f32", "bf16", "u8"])
def test_wide_addresses(tall, dtype):
    log(f"test_wide_addresses: {dtype}, grid 2 x 4100 x 4100")
    sc, quant = tall, None
    if dtype == "u8":
        t = {k: torch.from_numpy(sc[k]).to(DEV) for k in (*SOURCES, "occ", "mlp")}
        codes, quant = om.quantize_features(t)
        scene = om.Scene(codes["grid"], codes["plane_xy"], codes["plane_xz"], codes["plane_yz"], t["occ"], t["mlp"],
                         quant=quant)
        sc = oracle.quant.dequantize_scene(oracle.quant.quantize_scene(sc))
    else:
        scene, t = upload_scene(sc, torch.bfloat16 if dtype == "bf16" else torch.float32)
        if dtype == "bf16":
            sc = dict(sc, **{k: bf16_round(sc[k]) for k in SOURCES})
    o, d = scenegen.oblique_rays(203, seed=8)
    og, dg = rays_to(o, d)
    for t_term in (0.0, 1e-2):
        res = om.render(scene, og, dg, n_max=100, c_bg=BG, t_term=t_term, mlp_bf16=0)
        ref = oracle.oracle_render(sc, o, d, oracle.RenderParams(n_max=100, c_bg=BG, t_term=t_term), keep_k=False)
        _compare(res, ref, f"{dtype}, t_term {t_term}")


@pytest.mark.parametrize("n_max", [3, 4, 5, 12, 15, 16, 20, 33])
def test_partial_batches_f32(n_max):
    log(f"test_partial_batches_f32: n_max {n_max}")
    sc = scenegen.make_scene(scenegen.TINY)
    scene, _ = upload_scene(sc)
    o, d = scenegen.oblique_rays(301, seed=9)
    og, dg = rays_to(o, d)
    res = om.render(scene, og, dg, n_max=n_max, c_bg=BG, batch_wv=True)
    _compare(res, oracle.oracle_render(sc, o, d, oracle.RenderParams(n_max=n_max, c_bg=BG), keep_k=False),
             f"n_max {n_max}")
    # the sums of the batches that were written add up to F
    ne, bw = res["n_eval"].cpu().numpy(), res["batch_wv"].double().cpu().numpy()
    live = np.arange(bw.shape[1])[None, :] < (ne[:, None] + 15) // 16
    total = np.where(live[..., None], bw, 0.0).sum(1)
    assert np.abs(total - res["F"].double().cpu().numpy()).max() <= 1e-6
