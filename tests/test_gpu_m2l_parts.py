"""The mixed M2L's small levels in many parts, down to one merged group of
steps each, with partial sums of the columns that hold targets only: the far
field against the FP64 form, within the mixed form's 1e-6, at the orders with
the fewest and the most steps and with levels 2, 3 and 4 split."""
import numpy as np
import pytest

from conftest import rel_l2
from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


@pytest.mark.parametrize("p,n,leaf,level", [(2, 700, 30, 2), (3, 3000, 20, 3), (4, 10_000, 64, 3), (6, 12_000, 12, 4),
                                            (10, 700, 30, 2), (12, 3000, 20, 3), (16, 3000, 20, 3)])
def test_small_levels_match_fp64(p, n, leaf, level):
    pos, q = inputs.particles(n, 500 + p)
    P, Q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (pos, q))
    out = {}
    for form in ("fp64", "mixed"):
        with fmm.Tree(P, p=p, leaf_max=leaf, precision=form) as t:
            assert t.info()["levels"] == level
            phi, E = t.evaluate(Q, part="far")
            out[form] = phi.cpu().numpy(), E.cpu().numpy()
    assert rel_l2(out["mixed"][0], out["fp64"][0]) < 1e-6
    assert rel_l2(out["mixed"][1], out["fp64"][1]) < 1e-6
