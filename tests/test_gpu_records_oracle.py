"""GPU: the gradients of a fused step with batch records against the float64
oracle, entry by entry.

Records need more rays than the oracle can follow, so the batch is 128 copies of
516 rays in a shuffled order, whose gradient is 128 times theirs (L2 is a mean
over the batch).  The bar is that of tests/gradcheck.py with 128 times the terms
per entry.  The fused step forms dL/dC itself: with |C - target| >= 0.45 and C
within 1e-6 of the oracle's, checked here, it is off by 2.3e-6 of itself, 39 u,
and by two roundings, so each term may be off by 41 u more.

The planes end at a tile's edge, one texel behind it and between (tiles of 17 x
20 base texels), and the rays aim at the whole footprint, edges included.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_09531_amd as om
import scenegen
from tests._scenes import micro_scene
from tests.gpu_util import DEV, bf16_round, log, rays_to, upload_scene
from tests.gradcheck import SOURCES, check

pytestmark = pytest.mark.gpu

BG = (0.25, 0.5, 0.75)
COPIES, RAYS, N_MAX = 128, 516, 256


# occupied up to the box's top, or from its floor up to where most rays reach it
@pytest.mark.parametrize("dtype,planes,zmax,occ_eps", [(torch.float32, (1701, 1702, 221), 0.25, 0.0),
                                                       (torch.float32, (1702, 1650, 222), 0.1, 0.02),
                                                       (torch.bfloat16, (1650, 1701, 241), 0.1, 0.0),
                                                       (torch.bfloat16, (1719, 1700, 222), 0.25, 0.02)])
def test_step_with_records_vs_oracle(dtype, planes, zmax, occ_eps):
    log(f"test_step_with_records_vs_oracle: {dtype}, planes {planes}, zmax {zmax}, occ_eps {occ_eps}")
    sc = micro_scene(grid=(20, 18, 9), planes=planes, m=8, zmax=zmax, seed=5)
    scene, t = upload_scene(sc, dtype)
    if dtype == torch.bfloat16:
        sc = dict(sc, **{k: bf16_round(sc[k]) for k in SOURCES})
    o, d = scenegen.oblique_rays(RAYS, seed=12)
    prm = oracle.RenderParams(n_max=N_MAX, c_bg=BG, occ_eps=occ_eps)
    C = oracle.oracle_render(sc, o, d, prm, keep_k=False)["C"]
    target = np.where(C < 0.5, C + 0.45, C - 0.45).astype(np.float32)
    target += np.where(C < 0.5, 1e-3, -1e-3).astype(np.float32)
    n = COPIES * RAYS
    up = 2.0 * (C - target.astype(np.float64)) / (3.0 * n)
    _, _, ref = oracle.oracle_loss_and_grads(sc, o, d, prm, upstream=up)
    scale = oracle.fp32_bound.gradient_error_scale(sc, o, d, prm, up)
    times = lambda r: (r[0], COPIES * r[1]) if isinstance(r, tuple) else COPIES * r  # noqa: E731
    ref = {k: times(v) for k, v in ref.items()}
    scale = {k: (*v[:-3], COPIES * v[-3], COPIES * (v[-2] + 41 * v[-3]), COPIES * v[-1]) for k, v in scale.items()}

    at = np.random.default_rng(3).permutation(np.tile(np.arange(RAYS), COPIES))
    og, dg = rays_to(o[at], d[at])
    tg = torch.from_numpy(target[at]).to(DEV)
    e = lambda *s, dt=torch.float32: torch.empty(s, dtype=dt, device=DEV)  # noqa: E731
    out = dict(C=e(n, 3), T=e(n), F=e(n, 7), n_placed=e(n, dt=torch.int32), n_eval=e(n, dt=torch.int32))
    grads = {k: torch.zeros(t[k].shape, device=DEV) for k in (*SOURCES, "mlp") + (("occ",) if occ_eps else ())}
    need, more = om.fwd_bwd_l2_workspace_size(n, N_MAX), om.fwd_bwd_l2_records_size(scene, n, N_MAX)
    assert more > 0
    om.render_fwd_bwd_l2(scene, og, dg, tg, out, grads, n_max=N_MAX, c_bg=BG, mlp_bf16=0, occ_eps=occ_eps,
                         workspace=e(need + more, dt=torch.uint8))
    assert int(((out["n_placed"] + 15) // 16).sum()) >= 1 << 19  # kept, not replayed
    assert np.abs(out["C"].double().cpu().numpy() - C[at]).max() <= 1e-6
    check({k: v.double().cpu().numpy() for k, v in grads.items()}, ref, scale, f"records {dtype} {planes}")
