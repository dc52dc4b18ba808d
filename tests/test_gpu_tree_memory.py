"""Trees that come and go: pinned words and events handed on between trees
(more trees alive than are kept for the next one, from several threads), and
memory returned in stream order, give the results of a tree that is kept."""
import threading

import pytest

from paper_1106_2176_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1106_2176_amd as fmm  # noqa: E402


def _problem(n, seed):
    pos, q = inputs.particles(n, seed)
    return torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()


@pytest.mark.parametrize("adaptive", [False, True])
def test_many_trees_and_threads_equal_one(adaptive):
    sets = [_problem(n, 400 + n) for n in (300, 5000, 20_000)]
    want = []
    for P, Q in sets:
        with fmm.Tree(P, p=6, leaf_max=32, precision="fp64", adaptive=adaptive) as t:
            want.append([x.clone() for x in t.evaluate(Q)])
    alive = [fmm.Tree(sets[i % 3][0], p=6, leaf_max=32, precision="fp64", adaptive=adaptive) for i in range(12)]
    for i, t in enumerate(alive):
        phi, E = t.evaluate(sets[i % 3][1])
        assert torch.equal(phi, want[i % 3][0]) and torch.equal(E, want[i % 3][1])
    for t in alive:
        t.close()
    bad = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for j in range(6):
                P, Q = sets[(k + j) % 3]
                phi, E = fmm.evaluate(P, Q, p=6, leaf_max=32, precision="fp64", adaptive=adaptive)
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(phi, want[(k + j) % 3][0]) and torch.equal(E, want[(k + j) % 3][1])):
                    bad.append((k, j))

    th = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not bad


def test_a_tree_used_on_another_stream_keeps_its_memory_until_that_work_ends():
    P, Q = _problem(200_000, 410)
    with fmm.Tree(P, p=8, leaf_max=64, precision="fp64") as t:
        want = [x.clone() for x in t.evaluate(Q)]
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    t = fmm.Tree(P, p=8, leaf_max=64, precision="fp64")
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        got = t.evaluate(Q)
    t.close()
    junk = [torch.full((1 << 22,), float("nan"), device="cuda", dtype=torch.float64) for _ in range(8)]
    torch.cuda.synchronize()
    del junk
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
