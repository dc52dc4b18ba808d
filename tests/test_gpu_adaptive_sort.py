"""Key sort and scans of the adaptive build where their launch shapes change:
blocks of 4, 5 and 16 steps of 256 keys, scans of one block, of up to 1024
block sums and of more.  The order equals a stable sort of the keys, the boxes
equal those counted level by level, and W and X mirror each other (as many
multipole evaluations as local ones)."""
import numpy as np
import pytest

from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


def _spread(v):
    out = np.zeros(v.shape, dtype=np.int64)
    for b in range(10):
        out |= ((v >> b) & 1) << (3 * b)
    return out


@pytest.mark.parametrize("kind,n,leaf,ml", [
    ("uniform", 1023, 8, 10),
    ("uniform", 1025, 8, 10),
    ("clustered", 300_000, 64, 9),
    ("uniform", 1_400_000, 16, 7),
    ("clustered", 4_300_000, 128, 10),
])
def test_order_and_boxes(kind, n, leaf, ml):
    pos, _ = inputs.particles(n, 3) if kind == "uniform" else inputs.clustered(n, 3)
    side = 1 << ml
    c = np.minimum((pos * side).astype(np.int64), side - 1)
    key = _spread(c[:, 0]) | _spread(c[:, 1]) << 1 | _spread(c[:, 2]) << 2
    order = np.argsort(key, kind="stable")
    skey = key[order]
    rows, over = [], np.ones(1, dtype=bool)
    codes_up = np.zeros(1, dtype=np.int64)
    for lev in range(ml + 1):
        codes, start, cnt = np.unique(skey >> (3 * (ml - lev)), return_index=True, return_counts=True)
        if lev:
            keep = over[np.searchsorted(codes_up, codes >> 3)]
            codes, start, cnt = codes[keep], start[keep], cnt[keep]
        if len(codes) == 0:
            break
        split = (cnt > leaf) & (lev < ml)
        rows.append(np.stack([np.full(len(codes), lev), start, start + cnt, ~split], 1))
        # the next level looks its parents up among all of this level's keys
        codes_up, start, cnt = np.unique(skey >> (3 * (ml - lev)), return_counts=True, return_index=True)
        over = (cnt > leaf) & (lev < ml)
    ref = np.concatenate(rows)
    print("adaptive sort", kind, n, leaf, ml, len(ref), flush=True)
    with fmm.Tree(torch.from_numpy(pos).cuda(), p=2, leaf_max=leaf, max_level=ml, adaptive=True) as t:
        perm, lstart = t.export()
        info = t.info()
    np.testing.assert_array_equal(perm.astype(np.int64), order)
    leaves = ref[ref[:, 3] == 1]
    np.testing.assert_array_equal(lstart[:-1].astype(np.int64), np.sort(leaves[:, 1]))
    assert info["n_boxes"] == len(ref) and info["levels"] == ref[:, 0].max()
    assert info["max_leaf_count"] == (leaves[:, 2] - leaves[:, 1]).max()
    assert info["m2p_evals"] == info["p2l_evals"]
