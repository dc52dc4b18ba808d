"""Upward and downward translations of the adaptive tree: 16 split boxes to a
column tile and 32 rows to a block.  Far potentials and fields of the FP64
form equal the oracle's adaptive FMM (same lists, same truncation, sums that
differ by rounding only: 1e-10) for row counts on both sides of the tiles'
edges, K counts that are no multiple of four, and levels with one, sixteen and
more split boxes."""
import numpy as np
import pytest

from conftest import rel_l2
from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6, 7, 9, 12, 13, 16])
@pytest.mark.parametrize("n,leaf,ml", [(1200, 30, 7), (3000, 4, 6)])
def test_far_field_matches_oracle(oracle_mod, p, n, leaf, ml):
    pos, q = inputs.clustered(n, 21)
    q = q - 0.5
    pos[: n // 3] = pos[0] + (pos[: n // 3] - pos[0]) * 0.05  # one deep cluster: levels with one split box
    ref = oracle_mod.fmm_adaptive(pos, q, p, leaf, ml)
    print("adaptive vertical", p, n, leaf, ml, flush=True)
    with fmm.Tree(torch.from_numpy(pos).cuda(), p=p, leaf_max=leaf, max_level=ml, precision="fp64",
                  adaptive=True) as t:
        phi, E = t.evaluate(torch.from_numpy(q).cuda(), vec="field", part="far")
        phi, E = phi.cpu().numpy(), E.cpu().numpy()
        assert t.info()["levels"] == ref["depth"] >= 4
    assert rel_l2(phi, ref["phi_far"]) < 1e-10
    if np.linalg.norm(ref["E_far"]) > 0:
        assert rel_l2(E, ref["E_far"]) < 1e-10
