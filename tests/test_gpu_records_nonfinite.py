"""GPU: a fused step with batch records in which one ray has an infinite
dL/dC.  Gradients that are not finite belong on the texels of that ray's
evaluated samples and nowhere else: not on those of samples that it placed
behind the one it stopped at, and of a partial batch only on the batch's own.

The rows that the ray's evaluated samples read come from the placement
(om_mark_rows), not from the step.  With t_term the replay may take the step
instead, which is held to the same.
"""
import pytest
import torch

import paper_2404_09531_amd as om
from tests._scenes import micro_scene
from tests.gpu_util import log
from tests.test_gpu_records import FINE, Step, oblique

pytestmark = pytest.mark.gpu

SOURCES = ("grid", "plane_xy", "plane_xz", "plane_yz")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("t_term", [0.0, 0.9])
def test_infinite_gradient_of_one_ray(dtype, t_term):
    log(f"test_infinite_gradient_of_one_ray: {dtype}, t_term {t_term}")
    n_max = 249
    sc = micro_scene(grid=(20, 18, 9), planes=FINE, m=8, zmin=0.01, zmax=0.24, seed=5)
    s = Step(sc, *oblique(70001), dtype=dtype, n_max=n_max, t_term=t_term)
    assert s.records > 0
    ne = om.render(s.scene, s.o, s.d, n_max=n_max, t_term=t_term)["n_eval"]
    assert not t_term or int((ne < 240).sum()) > len(ne) // 2  # most rays stop early
    ray = int(torch.nonzero((ne > 16) & (ne % 16 == 5))[0]) if t_term else 4321
    s.target[ray] = float("inf")
    (_, plain, _), (out, recorded, _) = s.both()
    log(f"  ray {ray}: {int(out['n_eval'][ray])} samples evaluated")
    assert int(out["n_eval"][ray]) % 16 in (5, 9)  # lanes of its last batch are without a sample
    read = om.mark_rows(s.scene, s.o[ray:ray + 1].contiguous(), s.d[ray:ray + 1].contiguous(), n_max,
                        n_eval=out["n_eval"][ray:ray + 1].contiguous())
    for k in SOURCES:
        want = read[k].bool()
        for tag, g in (("replay", plain[k]), ("records", recorded[k])):
            got = (~torch.isfinite(g)).any(-1)
            log(f"  {k}, {tag}: {int(got.sum())} rows not finite, {int(want.sum())} read")
            assert torch.equal(got, want), (k, tag)
