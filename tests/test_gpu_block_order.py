"""GPU: every ray is rendered once whatever the number of blocks.

Blocks of 16 rays (march) and of 256 or fewer (MLP) take rays in an order that
follows the eight XCDs, in whole turns of 8 x 32 blocks and a remainder in
eighths: sizes around one and two turns and around the remainder's eighths.
Rays are independent, so a call's outputs equal those of calls of 2,000 rays,
which have no whole turn, bit by bit.
"""
import pytest
import torch

import paper_2404_09531_amd as om
import scenegen
from tests.gpu_util import DEV, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n", [4095, 4096, 4097, 4096 + 16 * 7, 4096 + 16 * 9 + 1, 8191, 8193, 65536 + 5, 131072 + 4111])
def test_blocks_cover_the_rays(n, dtype):
    log(f"test_blocks_cover_the_rays: {n} rays, {dtype}")
    scene, _ = upload_scene(scenegen.make_scene(scenegen.TINY), dtype)
    o, d = rays_to(*scenegen.oblique_rays(n, seed=12))
    kw = dict(n_max=40, c_bg=(0.25, 0.5, 0.75))
    whole = om.render(scene, o, d, **kw)
    parts = [om.render(scene, o[i:i + 2000].contiguous(), d[i:i + 2000].contiguous(), **kw) for i in range(0, n, 2000)]
    for k in ("n_placed", "n_eval", "C", "F", "T"):
        assert torch.equal(whole[k], torch.cat([p[k] for p in parts])), k
    assert float(whole["n_placed"].float().mean()) > 1
    assert whole["C"].device == torch.device(DEV)
