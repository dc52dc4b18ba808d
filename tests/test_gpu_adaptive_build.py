"""The adaptive tree's boxes are made from the box levels of every particle,
counted per block of 1024 particles in waves of 256.  Boxes, particle order,
leaf starts and the lists equal the oracle's at the edges of waves and blocks,
for caps from one particle to all of them, at the coarsest and finest level
limits, with coincident particles and with every particle in one corner."""
import numpy as np
import pytest

from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402

CASES = [  # kind, n, leaf_max, max_level
    ("uniform", 1, 1, 10),
    ("uniform", 2, 1, 0),
    ("uniform", 255, 1, 10),
    ("uniform", 257, 3, 1),
    ("clustered", 1023, 1, 10),
    ("clustered", 1024, 1024, 5),
    ("clustered", 1025, 1024, 5),
    ("clustered", 4097, 2, 10),
    ("clustered", 9001, 1500, 10),
    ("coincident", 3000, 16, 10),
    ("coincident", 3000, 16, 2),
    ("corner", 2049, 5, 10),
    ("corner", 5000, 64, 3),
]


@pytest.mark.parametrize("kind,n,leaf,ml", CASES)
def test_boxes_match_oracle(oracle_mod, kind, n, leaf, ml):
    pos, _ = inputs.particles(n, 7) if kind != "clustered" else inputs.clustered(n, 7)
    if kind == "coincident":
        pos[::3] = pos[0]
    if kind == "corner":
        pos = 1.0 - pos * 2.0**-8
    ref = oracle_mod.adaptive_tree(pos, leaf, ml)
    print("adaptive build", kind, n, leaf, ml, flush=True)
    with fmm.Tree(torch.from_numpy(pos).cuda(), p=2, leaf_max=leaf, max_level=ml, precision="fp64",
                  adaptive=True) as t:
        got = t.export_adaptive()
        info = t.info()
        perm, lstart = t.export()
    np.testing.assert_array_equal(got["boxes"], ref["boxes"])
    np.testing.assert_array_equal(got["order"], ref["order"])
    for name in "UVWX":
        for g, r in zip(got[name], ref[name]):
            np.testing.assert_array_equal(np.sort(np.asarray(g, dtype=np.int64)), np.sort(np.asarray(r, dtype=np.int64)))
    boxes = ref["boxes"]
    leaves = boxes[boxes[:, 7] == 1]
    leaves = leaves[np.argsort(leaves[:, 4])]
    np.testing.assert_array_equal(lstart.astype(np.int64), np.append(leaves[:, 4], n))
    assert info["max_leaf_count"] == int((leaves[:, 5] - leaves[:, 4]).max())
