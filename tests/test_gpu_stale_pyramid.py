"""GPU: a fused step with batch records while the attached occupancy pyramid
belongs to an older state of the plane (a program that trains the plane in
place and rebuilds the pyramid now and then).  Such a pyramid skips samples, and
which ones depends on the windows that a jump starts from: the counts that the
records are handed out by have to be those of the march itself.

The step in the smallest workspace, which marches once, is the reference:
counts equal, C, F and T within 1e-5, gradients as float32 sums in another order
(test_gpu_records.py).  Nothing behind the workspace is written.
"""
import numpy as np
import pytest
import torch

import paper_2404_09531_amd as om
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log
from tests.test_gpu_records import FINE, Step, assert_same

pytestmark = pytest.mark.gpu


def columns(rng, share):
    """Intervals of a 256 x 256 plane, `share` of them empty in blocks of 4 to
    16 columns a side (the pyramid is used after 512 empty candidates: 32 columns)."""
    empty = np.zeros((256, 256), bool)
    while empty.mean() < share:
        w, h = rng.choice((4, 8, 16, 16), 2)
        i, j = rng.integers(0, 256 - w + 1), rng.integers(0, 256 - h + 1)
        empty[j:j + h, i:i + w] = True
    return np.where(empty[..., None], np.float32((0.2, 0.1)), np.float32((0.0, 0.25)))


@pytest.mark.parametrize("occ_eps", [0.0, 0.02])
@pytest.mark.parametrize("levels", [1, 4])
def test_step_with_an_older_pyramid(levels, occ_eps):
    log(f"test_step_with_an_older_pyramid: {levels} levels, occ_eps {occ_eps}")
    rng = np.random.default_rng(levels)
    sc = micro_scene(grid=(20, 18, 9), planes=FINE, m=256, seed=5)
    sc["occ"] = columns(rng, 0.93)
    n = 60001
    yaw, pitch = rng.uniform(0, 2 * np.pi, n), np.radians(rng.uniform(4, 12, n))  # long ways through the box
    o = np.stack([rng.uniform(-1, 1, n), rng.uniform(-1, 1, n), np.full(n, 0.25)], 1)
    d = np.stack([np.cos(pitch) * np.cos(yaw), np.cos(pitch) * np.sin(yaw), -np.sin(pitch)], 1)
    s = Step(sc, o.astype(np.float32), d.astype(np.float32), n_max=384, occ_eps=occ_eps)
    s.scene.build_occupancy_mips(levels)
    s.t["occ"].copy_(torch.from_numpy(columns(rng, 0.8)))
    assert s.records > 0
    plain = s.buffers()
    s.run(*plain, s.need)
    batches = int(((plain[0]["n_placed"] + 15) // 16).sum())
    fresh = om.Scene(*(s.t[k] for k in ("grid", "plane_xy", "plane_xz", "plane_yz", "occ", "mlp")))
    exact = om.place_samples(fresh, s.o, s.d, 384)[1]
    log(f"  {batches} batches, {int((plain[0]['n_placed'] != exact).sum())} rays skip samples")
    assert batches >= 1 << 19 and int((plain[0]["n_placed"] != exact).sum()) > 1000
    recorded = s.buffers()
    buf = torch.full((s.need + s.records + 4096,), 171, dtype=torch.uint8, device=DEV)
    om.render_fwd_bwd_l2(s.scene, s.o, s.d, s.target, recorded[0], recorded[1], loss=recorded[2],
                         workspace=buf[:s.need + s.records], **s.kw)
    assert bool((buf[s.need + s.records:] == 171).all())
    assert_same(plain, recorded)
