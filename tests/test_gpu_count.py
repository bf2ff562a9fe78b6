"""GPU: the counts ahead of a fused step with batch records, which test four
windows of candidates at a time and jump over empty columns, against the
placement's counts: a scene of separate columns (gaps before, between and
within windows), with and without the occupancy pyramid, n_max inside a window,
at its edge and beyond the ray.  The records of a ray whose count were wrong
would overlap another's, so gradients are compared too (the floor of
test_backward_large_batch_equals_its_halves)."""
import numpy as np
import pytest
import torch

import paper_2404_09531_amd as om
import scenegen
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu

KEYS = ("grid", "plane_xy", "plane_xz", "plane_yz", "mlp")


@pytest.mark.parametrize("mips", [0, 3])
@pytest.mark.parametrize("n_max", [250, 256, 300])
def test_counts_of_a_step_with_records(n_max, mips):
    log(f"test_counts_of_a_step_with_records: n_max {n_max}, {mips} levels")
    n = 90001
    sc = micro_scene(grid=(20, 18, 9), planes=(1700, 1660, 210), m=64, zmin=0.0, zmax=0.25, seed=5)
    sc["occ"][np.random.default_rng(3).random((64, 64)) < 0.3] = (0.2, 0.1)  # nothing there
    scene, t = upload_scene(sc)
    if mips:
        scene.build_occupancy_mips(mips)
    o, d = rays_to(*scenegen.oblique_rays(n, seed=2))
    target = torch.rand(n, 3, device=DEV, generator=torch.Generator(device=DEV).manual_seed(4))
    need, more = om.fwd_bwd_l2_workspace_size(n, n_max), om.fwd_bwd_l2_records_size(scene, n, n_max)
    assert more > 0
    got = []
    for nbytes in (need, need + more):
        e = lambda *s, dt=torch.float32: torch.empty(s, dtype=dt, device=DEV)  # noqa: E731
        out = dict(C=e(n, 3), T=e(n), F=e(n, 7), n_placed=e(n, dt=torch.int32), n_eval=e(n, dt=torch.int32))
        grads = {k: torch.zeros(t[k].shape, device=DEV) for k in KEYS}
        om.render_fwd_bwd_l2(scene, o, d, target, out, grads, n_max=n_max, workspace=e(nbytes, dt=torch.uint8))
        got.append((out, grads))
    (a, ga), (b, gb) = got
    assert torch.equal(a["n_placed"], b["n_placed"]) and torch.equal(a["T"], b["T"])
    assert torch.equal(a["n_placed"], om.place_samples(scene, o, d, n_max)[1])
    assert int(((a["n_placed"] + 15) // 16).sum()) >= 1 << 19
    for k in KEYS:
        scale = float(ga[k].abs().max())
        assert scale > 0
        assert float(((ga[k] - gb[k]).abs() - (1e-3 * ga[k].abs() + 5e-5 * scale)).max()) <= 0, k
