"""The FP64 M2L folded by reflections against the oracle: orders with no
opposite pairs at all (p = 1), with single and with grouped row quads, with
eight- and four-wave tiles; one half-empty tile (level 2), tiles cut into
parts (levels 3 and 4) and whole tiles beside them (level 5).

Tolerance 1e-10 rel-L2, the FP64 form's against the oracle (the same
approximation in another basis; both sides round at 1e-16 over sums of a few
thousand terms that cancel by at most 1e3).
"""
import numpy as np
import pytest

from conftest import rel_l2
from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("p,n,leaf,level", [(1, 700, 30, 2), (2, 3000, 20, 3), (3, 700, 30, 2), (5, 12_000, 12, 4),
                                            (7, 3000, 20, 3), (9, 40_000, 10, 5), (10, 700, 30, 2), (12, 3000, 20, 3),
                                            (13, 700, 30, 2), (14, 12_000, 12, 4), (16, 3000, 20, 3)])
def test_far_field_and_adjoint_match_the_oracle(oracle_mod, p, n, leaf, level):
    pos, q = inputs.particles(n, 300 + p, "u11")
    w = inputs.weights(n, 300 + p)
    ref = oracle_mod.fmm(pos, q, p, leaf)
    assert ref["level"] == level
    with fmm.Tree(dev(pos), p=p, leaf_max=leaf, precision="fp64") as t:
        phi, E = t.evaluate(dev(q), part="far")
        full, field = t.evaluate(dev(q))
        gq, gx = t.backward(dev(q), dev(w), field)
        torch.cuda.synchronize()
    assert rel_l2(phi.cpu().numpy(), ref["phi_far"]) < 1e-10
    if p > 1:
        assert rel_l2(E.cpu().numpy(), ref["E_far"]) < 1e-10
    gq_o, gx_o, _ = oracle_mod.fmm_grad(pos, q, w, p, leaf)
    assert rel_l2(gq.cpu().numpy(), gq_o) < 1e-10
    assert rel_l2(gx.cpu().numpy(), gx_o) < 1e-10


@pytest.mark.parametrize("p,leaf", [(2, 8), (8, 32)])
def test_adaptive_noalloc_matches_evaluate(p, leaf):
    """The scratch form puts the adaptive tree's operands over the near and
    far partials (or beside them, where they do not fit): bitwise the same."""
    import ctypes
    pos, q = inputs.clustered(20_000, 310 + p)
    Q = dev(q)
    with fmm.Tree(dev(pos), p=p, leaf_max=leaf, precision="fp64", adaptive=True) as t:
        for part, flags in ((None, fmm.VEC_FIELD), ("far", fmm.VEC_FIELD | fmm.PART_FAR_ONLY)):
            phi, E = t.evaluate(Q, part=part)
            phi2, E2 = torch.full_like(phi, float("nan")), torch.full_like(E, float("nan"))
            rc = fmm.lib().fmm_evaluate_noalloc(t._h, ctypes.c_void_p(Q.data_ptr()), ctypes.c_void_p(phi2.data_ptr()),
                                                ctypes.c_void_p(E2.data_ptr()), flags,
                                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            torch.cuda.synchronize()
            assert rc == fmm.FMM_OK
            assert torch.equal(phi, phi2) and torch.equal(E, E2)
