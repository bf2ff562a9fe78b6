"""GPU: which fused steps keep batch records, seen from the workspace: what lies
behind its smallest size is written if and only if records are kept, and what
lies behind the workspace never is."""
import pytest
import torch

import paper_2404_09531_amd as om
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log
from tests.test_gpu_records import FINE, Step, oblique

pytestmark = pytest.mark.gpu

GUARD = 4096


def written(s, nbytes):
    """Runs the step in a workspace of nbytes; returns whether its part behind
    the smallest size was written."""
    buf = torch.full((nbytes + GUARD,), 171, dtype=torch.uint8, device=DEV)
    out, grads, loss = s.buffers()
    om.render_fwd_bwd_l2(s.scene, s.o, s.d, s.target, out, grads, loss=loss, workspace=buf[:nbytes], **s.kw)
    assert bool((buf[nbytes:] == 171).all())
    return not bool((buf[s.need:] == 171).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_early_termination_replays(dtype):
    log(f"test_early_termination_replays: {dtype}")
    sc = micro_scene(grid=(20, 18, 9), planes=FINE, m=8, seed=5)
    for t_term in (0.0, 1e-30, 1e-2):
        s = Step(sc, *oblique(66003), dtype=dtype, n_max=256, t_term=t_term)
        assert s.records > 0  # those of a step without early termination
        assert (om.fwd_bwd_l2_records_size(s.scene, s.n, 256, t_term=t_term) > 0) == (t_term == 0)
        assert written(s, s.need + s.records) == (t_term == 0)


@pytest.mark.parametrize("n,zmax", [(66003, 0.25), (66003, 0.02), ((1 << 20) + 3, 0.25)])
def test_workspace_bounds(n, zmax):
    """Enough batches, too few (known only on the device), and more than there
    are records.  The size leaves 256 bytes for the alignment of the part behind
    the smallest size, so the least workspace that holds the records is shorter."""
    log(f"test_workspace_bounds: {n} rays, occupied up to {zmax}")
    s = Step(micro_scene(grid=(20, 18, 9), planes=FINE, m=8, zmax=zmax, seed=5), *oblique(n), n_max=256)
    least = (s.need + 255) // 256 * 256 + s.records - 256
    assert s.records > 0 and least <= s.need + s.records
    assert not written(s, s.need)
    assert not written(s, least - 1)
    assert written(s, least)
    assert written(s, s.need + s.records)
