"""GPU: an 8-bit scene whose sources all have offsets far from zero that their
codes make up for, as baked features do (codes near 128, values near zero): each
source is decoded by itself, so the sum of the four keeps the accuracy of values
near zero and not that of the offsets' sum.

Straight-down rays over the vertices of every source meet samples whose
fractions are all zero, so the interpolated codes are exact and what is left is:
per source one rounding of a value of at most 1.6 (below 2: u/2 times 2), and the
three sums, of at most 6.5 (4 u each): 4 + 12 = 16 u in a feature, a quarter of that
through the sigmoid, weights that add up to one at most; the sigmoid and the
compositing have 2^-20, four times what the float32 forward is off by on the
benchmark's frame (2.5e-7).  With the four offsets summed first the features were
off by up to the rounding of 360, 15e-6.
"""
import numpy as np
import pytest
import torch

import oracle
import oracle.quant
import paper_2404_09531_amd as om
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log, rays_to

pytestmark = pytest.mark.gpu

SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")
U = 2.0 ** -24


@pytest.mark.parametrize("sparse", [0, 3])
@pytest.mark.parametrize("occ_eps", [0.0, 0.02])
def test_offsets_do_not_cost_accuracy(occ_eps, sparse):
    log(f"test_offsets_do_not_cost_accuracy: occ_eps {occ_eps}, sparse {sparse}")
    rng = np.random.default_rng(4)
    sc = micro_scene(grid=(17, 17, 513), planes=(17, 17, 513), m=8, seed=1)
    step = np.full((4, 8), 0.7, np.float32)
    lo = (-128 * step - rng.uniform(-0.2, 0.2, (4, 8))).astype(np.float32)
    lo[:, 0], step[:, 0] = 0.0, 0.01  # the density: no offsets, exp(5.12) a sample
    q8 = dict(sc, quant_lo=lo, quant_step=step)
    for k in SOURCES:
        q8[k] = rng.integers(126, 131, sc[k].shape, dtype=np.uint8)
    t = {k: torch.from_numpy(q8[k]).to(DEV) for k in (*SOURCES, "occ", "mlp")}
    args = [t[k] for k in (*SOURCES, "occ", "mlp")]
    scene = om.Scene(*args, quant=(lo, step))
    if sparse:
        atlas, sg = om.sparse_grid(scene, sparse)
        scene = om.Scene(atlas, *args[1:], quant=(lo, step), sparse=sg)
    x = -1.0 + np.arange(17) / 8.0
    o = np.stack([*(v.ravel() for v in np.meshgrid(x, x)), np.full(289, 0.25)], 1).astype(np.float32)
    d = np.tile(np.float32((0, 0, -1)), (289, 1))
    og, dg = rays_to(o, d)
    res = om.render(scene, og, dg, n_max=300, occ_eps=occ_eps)
    ref = oracle.oracle_render(oracle.quant.dequantize_scene(q8), o, d,
                               oracle.RenderParams(n_max=300, occ_eps=occ_eps), keep_k=False)
    assert np.array_equal(res["n_eval"].cpu().numpy(), ref["n_eval"]) and ref["n_eval"].max() == 300
    err = float(np.abs(res["F"].double().cpu().numpy() - ref["F"]).max())
    log(f"  max |F - oracle| = {err:.2e}")
    assert err <= 16 * U / 4 + 2.0 ** -20
