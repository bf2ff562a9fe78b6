"""GPU: the numbering of sparse blocks, whose slices are of 16,384 entries and
whose loads are of four: index lengths around both, in index buffers that
start on a 16-byte boundary and behind one, against a cumulative sum of the
marks."""
import ctypes

import pytest
import torch

import paper_2404_09531_amd as om
from paper_2404_09531_amd import _lib
from tests._scenes import micro_scene
from tests.gpu_util import DEV, log, upload_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [(1, 1, 1), (3, 1, 1), (5, 3, 1), (128, 128, 1), (113, 29, 5), (65, 65, 17)])
def test_numbers(cells):
    log(f"test_numbers: {cells} blocks")
    sc = micro_scene(grid=tuple(2 * c + 1 for c in cells), planes=(8, 8, 8), m=16, zmin=0.0, zmax=0.25, seed=2)
    sc["occ"][3:9, 5:11] = (0.1, 0.05)  # columns without samples
    sc["occ"][10:, :4] = (0.0, 0.02)
    scene, _ = upload_scene(sc)
    n = cells[0] * cells[1] * cells[2]
    got = []
    for skip in (0, 1, 2, 3):
        buf = torch.full((n + 8,), -7, dtype=torch.int32, device=DEV)
        count = _lib.lib().om_sparse_grid_index(scene.handle, 1, ctypes.c_void_p(buf.data_ptr() + 4 * skip),
                                                ctypes.c_int64(n), ctypes.c_void_p(0))
        torch.cuda.synchronize()
        assert (buf[:skip] == -7).all() and (buf[skip + n:] == -7).all()
        idx = buf[skip:skip + n]
        kept = idx > 0
        assert torch.equal(idx, torch.where(kept, torch.cumsum(kept.int(), 0).int(), torch.zeros_like(idx)))
        assert count == int(kept.sum()) > 0
        got.append(idx)
    assert all(torch.equal(got[0], g) for g in got[1:])
    assert om.sparse_grid(scene, 1)[1].n_blocks == int((got[0] > 0).sum())
