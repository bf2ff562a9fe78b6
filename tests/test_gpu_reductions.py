"""GPU: the loss sums, the small-batch ray order of the backward, and the
numbering of sparse blocks at the sizes where their launches change.

Loss bars: a sum of m float32 terms of one sign, each rounded a few times, is
within (chain + 4) u of its value, with chain the longest chain of additions:
a thread's strided terms (m / 1024 in one workgroup, m / 65536 over 256), the
16-lane reductions and the sum over the blocks, below m / 1024 + 300 in all.
"""
import numpy as np
import pytest
import torch

import paper_2404_09531_amd as om
import scenegen
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log, rays_to, upload_scene

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")


# one workgroup up to 10,922 rays (32,768 values); 85 / 86: a ragged and a
# full set of 256 values; 300,001: several values per thread of 256 blocks
@pytest.mark.parametrize("n", [1, 85, 86, 2731, 10922, 10923, 300001])
def test_l2_loss_and_gradient(n):
    log(f"test_l2_loss_and_gradient: {n} rays")
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    C, t = torch.rand(n, 3, device=DEV, generator=g), torch.rand(n, 3, device=DEV, generator=g)
    dC, loss = om.l2_loss_grad(C, t)
    dC2, loss2 = om.l2_loss_grad(C, t)
    only, none = om.l2_loss_grad(C, t, with_loss=False)
    assert torch.equal(loss, loss2) and torch.equal(dC, dC2) and torch.equal(dC, only) and none is None
    e = C.double() - t.double()
    want = float((e * e).sum() / (3 * n))
    assert abs(float(loss) - want) <= want * (3 * n / 1024 + 304) * U
    assert float((dC.double() - 2 * e / (3 * n)).abs().max()) <= 4 * U * 2 / (3 * n)
    l64 = om.l2_loss_fp64(C, t)
    assert abs(float(l64) - want) <= want * 1e-12


@pytest.mark.parametrize("cells", [1, 1023, 1024, 8192, 8193, 512 * 512])
def test_interval_loss(cells):
    log(f"test_interval_loss: {cells} cells")
    g = torch.Generator(device=DEV)
    g.manual_seed(cells)
    occ = torch.rand(1, cells, 2, device=DEV, generator=g)
    loss = om.occ_interval_loss(occ, 0.5)
    span = occ[..., 1].double() - occ[..., 0].double()
    want = 0.5 * float((span * span).sum())
    assert abs(float(loss) - want) <= want * (cells / 1024 + 304) * U


def test_small_order_equals_general_order():
    """16,385 rays (four launches) against 16,384 and 1 (one workgroup
    each), every fifth ray without samples: the same rays, so the same
    gradients up to the order of the float atomics."""
    n = 16385
    log(f"test_small_order_equals_general_order: {n} rays")
    sc = scenegen.make_scene(scenegen.TINY)
    scene, t = upload_scene(sc)
    o, d = scenegen.oblique_rays(n, seed=41)
    d = d.copy()
    d[::5, 2] = -d[::5, 2]
    og, dg = rays_to(o, d)
    kw = dict(n_max=1024)
    res = om.render(scene, og, dg, batch_wv=True, **kw)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    dC = (torch.randn(n, 3, device=DEV, generator=gen) * 1e-5).contiguous()
    zero = lambda: {k: torch.zeros(t[k].shape, device=DEV) for k in (*SOURCES, "mlp")}  # noqa: E731
    whole, parts = zero(), zero()
    om.render_backward(scene, og, dg, res, dC, whole, **kw)
    for sl in (slice(0, n - 1), slice(n - 1, n)):
        part = {k: v[sl].contiguous() for k, v in res.items()}
        om.render_backward(scene, og[sl].contiguous(), dg[sl].contiguous(), part, dC[sl].contiguous(), parts, **kw)
    for k in whole:
        scale = float(whole[k].abs().max())
        diff = (whole[k] - parts[k]).abs()
        assert scale > 0
        # the floor of test_backward_large_batch_equals_its_halves: the same
        # terms in another order
        assert float((diff - (1e-3 * parts[k].abs() + 5e-5 * scale)).max()) <= 0, k


# 8,192 entries are one slice of the numbering; 65 x 65 x 17 = 71,825 are
# nine, the last one ragged
@pytest.mark.parametrize("zmin,zmax", [(0.0, 0.25), (0.1, 0.2), (0.2, 0.1)])
def test_block_numbering(zmin, zmax):
    log(f"test_block_numbering: occupancy [{zmin}, {zmax}]")
    sc = micro_scene(grid=(131, 131, 35), planes=(8, 8, 8), m=8, zmin=zmin, zmax=zmax, seed=2)
    scene, _ = upload_scene(sc)
    atlas, sg = om.sparse_grid(scene, 1)
    idx = sg.blocks.cpu().numpy()
    assert idx.shape == (17, 65, 65)
    kept = idx[idx > 0]
    assert np.array_equal(kept, np.arange(1, sg.n_blocks + 1)) and not (idx < 0).any()
    assert (sg.n_blocks == idx.size) == (zmin == 0.0) and (sg.n_blocks == 0) == (zmin > zmax)
    # the last block's vertices are those of the grid
    if sg.n_blocks:
        z, y, x = (int(v[-1]) for v in np.nonzero(idx))
        want = sc["grid"][2 * z:2 * z + 3, 2 * y:2 * y + 3, 2 * x:2 * x + 3]
        assert np.array_equal(atlas[idx[z, y, x]].cpu().numpy()[:want.shape[0], :want.shape[1], :want.shape[2]], want)
