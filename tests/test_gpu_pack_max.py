"""Scale of the mixed form's M2L operands at small trees, where the packing
kernel finds each level's maximum itself (up to 16384 coefficients a level),
and just beyond.  Far potentials of the mixed form agree with the FP64 form's
within the mixed form's 1e-6, also with charges far from one in size, and zero
charges give zeros."""
import pytest

from conftest import rel_l2
from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


def _far(pos, q, p, leaf, precision):
    with fmm.Tree(pos, p=p, leaf_max=leaf, precision=precision) as t:
        levels = t.info()["levels"]
        return levels, t.evaluate(q, vec="field", part="far")[0].double().cpu().numpy()


@pytest.mark.parametrize("p,n,leaf,level", [
    (4, 1500, 60, 2), (15, 1500, 60, 2), (16, 1500, 60, 2),  # 64 boxes: up to 16384 coefficients
    (1, 10000, 64, 3), (4, 10000, 64, 3), (5, 10000, 64, 3),  # 512 boxes: 16384 at p = 5
    (6, 10000, 64, 3), (2, 60000, 64, 4),  # past the limit: two kernels
])
@pytest.mark.parametrize("scale", [1.0, 1e-18])
def test_mixed_far_field_matches_fp64(p, n, leaf, level, scale):
    pos, q = inputs.particles(n, 9)
    pos, q = torch.from_numpy(pos).cuda(), torch.from_numpy((q - 0.25) * scale).cuda()
    print("pack max", p, n, scale, flush=True)
    lm, mixed = _far(pos, q, p, leaf, "mixed")
    lf, ref = _far(pos, q, p, leaf, "fp64")
    assert lm == lf == level
    assert rel_l2(mixed, ref) < 1e-6
    _, zero = _far(pos, torch.zeros_like(q), p, leaf, "mixed")
    assert (zero == 0).all()
