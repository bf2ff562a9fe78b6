"""GPU: the hand-out of rays to the waves of the march backward, at batch
sizes around its edges, against the same rays in small calls.

The chip holds 4,096 waves, each of which takes 4 rays per turn: up to 16,384
rays every wave has one turn by its number, beyond that it draws further ones
from a counter, and from 2 x 8 x 16,384 rays on it takes two at a time.  Calls
of 4,000 rays have no second turn.  Every third ray misses the scene, so the
edges are also met among the rays that are handed out.

Bar: the same float32 terms in another order, the floor of
test_backward_large_batch_equals_its_halves.
"""
import pytest
import torch

import paper_2404_09531_amd as om
import scenegen
from tests.gpu_util import DEV, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu

SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")


@pytest.mark.parametrize("n", [3, 16383, 16385, 30001, 262144 + 2, 400001])
def test_hand_out_equals_small_calls(n):
    log(f"test_hand_out_equals_small_calls: {n} rays")
    scene, t = upload_scene(scenegen.make_scene(scenegen.TINY))
    o, d = scenegen.oblique_rays(n, seed=n)
    d = d.copy()
    if n > 3 and n != 262144 + 2:  # 262,146 rays, all of them handed out
        d[::3, 2] = -d[::3, 2]
    og, dg = rays_to(o, d)
    kw = dict(n_max=48)
    res = om.render(scene, og, dg, batch_wv=True, **kw)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    dC = (torch.rand(n, 3, device=DEV, generator=gen) * 1e-5).contiguous()
    whole, parts = ({k: torch.zeros(t[k].shape, device=DEV) for k in (*SOURCES, "mlp")} for _ in range(2))
    om.render_backward(scene, og, dg, res, dC, whole, **kw)
    for i in range(0, n, 4000):
        sl = slice(i, min(n, i + 4000))
        part = {k: v[sl].contiguous() for k, v in res.items()}
        om.render_backward(scene, og[sl].contiguous(), dg[sl].contiguous(), part, dC[sl].contiguous(), parts, **kw)
    for k in SOURCES:
        scale = float(whole[k].abs().max())
        assert scale > 0
        assert float(((whole[k] - parts[k]).abs() - (1e-3 * parts[k].abs() + 5e-5 * scale)).max()) <= 0, k
