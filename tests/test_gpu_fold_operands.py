"""The FP64 M2L's operands on the adaptive tree (the multipoles in K order):
over the near and far partials or, where these are too small, in the
multipoles' own place, so that they take no memory; and its whole tiles."""
import ctypes

import numpy as np
import pytest

from conftest import rel_l2
from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402

SCRATCH = 64 << 20


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def stride(p):
    return (p * p + 7) & ~7


def spiral(n):
    """Particles along a curve: many boxes with few neighbours."""
    rng = np.random.default_rng(503)
    t = np.sort(rng.random(n))
    a, r = 40 * np.pi * t, 0.35 * np.sin(np.pi * t)
    return np.stack([0.5 + r * np.cos(a), 0.5 + r * np.sin(a), 0.1 + 0.8 * t], 1), rng.random(n)


@pytest.mark.parametrize("p", [3, 4])
def test_the_scratch_array_takes_the_operands_in_the_multipoles_place(p):
    """200,000 boxes with less than a particle each: near and far partials,
    multipoles and locals fill most of the scratch array, a copy of the
    multipoles would not fit beside them nor over the partials."""
    pos, q = inputs.particles(140_000, 500)
    Q = dev(q)
    with fmm.Tree(dev(pos), p=p, leaf_max=1, precision="fp64", adaptive=True) as t:
        rows = 8 * stride(p) * (t.info()["n_boxes"] + 1)
        assert rows > 64 * len(q) and 64 * len(q) + 2 * rows < SCRATCH < 64 * len(q) + 3 * rows
        phi, E = t.evaluate(Q)
        phi2, E2 = torch.full_like(phi, float("nan")), torch.full_like(E, float("nan"))
        rc = fmm.lib().fmm_evaluate_noalloc(t._h, ctypes.c_void_p(Q.data_ptr()), ctypes.c_void_p(phi2.data_ptr()),
                                            ctypes.c_void_p(E2.data_ptr()), fmm.VEC_FIELD,
                                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == fmm.FMM_OK, fmm.lib().fmm_last_error_message()
        torch.cuda.synchronize()
        assert torch.equal(phi, phi2) and torch.equal(E, E2)


@pytest.mark.parametrize("p", [1, 3, 5, 10, 13, 16])
def test_operands_in_place_and_over_the_partials_give_the_same_bits(p):
    """Where the operands fit over the near and far partials but not over
    the far ones alone, the near field on the side stream decides: the same
    bits, forward and backward, call after call, and the same memory."""
    n = 20_000
    pos, q = inputs.clustered(n, 504)
    P, Q, W = dev(pos), dev(q), dev(inputs.weights(n, 504))
    for leaf in (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192):
        out, room = [], []
        for overlap in (False, True):
            with fmm.Tree(P, p=p, leaf_max=leaf, precision="fp64", adaptive=True, overlap_near=overlap) as t:
                info = t.info()
                fits = 32 * n < 8 * stride(p) * (info["n_boxes"] + 1) <= 64 * n
                if not fits:
                    break
                for _ in range(2):
                    phi, E = t.evaluate(Q)
                    out.append((phi, E, *t.backward(Q, W, E)))
                room.append(t.info()["workspace_bytes"])
        if out:
            break
    torch.cuda.synchronize()
    assert len(out) == 4 and room[0] == room[1]
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("p,n", [(4, 28_000), (13, 11_000)])
def test_whole_tiles_match_the_oracle(oracle_mod, p, n):
    """More tiles than compute units, with 128 targets (p = 4) and 64 (p = 13)
    each: whole tiles beside the ones cut into parts.  Tolerance 1e-10 rel-L2,
    the FP64 form's against the oracle on the same lists."""
    pos, q = inputs.particles(n, 502) if p == 4 else spiral(n)
    ref = oracle_mod.fmm_adaptive(pos, q, p, 1)
    assert ref["nbox"] > 256 * (128 if p <= 12 else 64)
    with fmm.Tree(dev(pos), p=p, leaf_max=1, precision="fp64", adaptive=True, max_level=10) as t:
        assert t.info()["n_boxes"] == ref["nbox"]
        phi, E = t.evaluate(dev(q))
        far, E_far = t.evaluate(dev(q), part="far")
        torch.cuda.synchronize()
    assert rel_l2(phi.cpu().numpy(), ref["phi"]) < 1e-10
    assert rel_l2(E.cpu().numpy(), ref["E"]) < 1e-10
    assert rel_l2(far.cpu().numpy(), ref["phi_far"]) < 1e-10
    assert rel_l2(E_far.cpu().numpy(), ref["E_far"]) < 1e-10


@pytest.mark.parametrize("p,n,leaf,adaptive", [(2, 3000, 20, False), (8, 12_000, 12, False), (12, 3000, 20, False),
                                               (16, 3000, 20, False), (8, 20_000, 32, True)])
def test_the_folded_products_round_like_the_direct_ones(oracle_mod, p, n, leaf, adaptive):
    """The far field of charges of both signs against the oracle.  A local
    coefficient sums up to 189 p^2 = 48,384 products; their roundings (1.1e-16
    each, of either sign) and the oracle's give about sqrt(48,384) 1.1e-16 =
    2.4e-14 of the terms' size at most: 1e-13 rel-L2."""
    pos, q = inputs.clustered(n, 505) if adaptive else inputs.particles(n, 505, "u11")
    q = q - q.mean()
    ref = oracle_mod.fmm_adaptive(pos, q, p, leaf) if adaptive else oracle_mod.fmm(pos, q, p, leaf)
    with fmm.Tree(dev(pos), p=p, leaf_max=leaf, precision="fp64", adaptive=adaptive, max_level=10) as t:
        phi, E = t.evaluate(dev(q), part="far")
        torch.cuda.synchronize()
    assert rel_l2(phi.cpu().numpy(), ref["phi_far"]) < 1e-13
    assert rel_l2(E.cpu().numpy(), ref["E_far"]) < 1e-13
