"""The FP64 M2L's roofline in bench.py counts the matrix products that the
folded kernel runs (no GPU)."""
import re

import pytest

import bench
from conftest import ROOT
from test_bench_host import _fake_result


def test_fold_flop_counts_the_products_of_the_lists():
    """Against a plain enumeration of orbits, rows and K positions."""
    for p in range(1, 17):
        par = []
        for n in range(p):
            for m in range(n + 1):
                par += [((m + s) & 1) | (s << 1) | (((n + m) & 1) << 2) for s in range(2 if m else 1)]
        quads = sum(-(-par.count(k) // 4) for k in range(8))
        pairs = sum(min(par.count(k), par.count(7 - k)) for k in range(4))
        flop = 0
        for o in range(64):
            d = (o & 3, (o >> 2) & 3, o >> 4)
            if max(d) < 2:
                continue  # a neighbour
            for chunk in range(-(-p * p // 8)):
                half = min(d) == 0 and 4 * (chunk + 1) <= pairs
                flop += 2 * 4 * quads * (4 if half else 8)
        assert bench.fold_flop(p) == flop


def test_fp64_rooflines_are_of_the_kernel_that_runs_and_below_its_peak():
    wl, res = _fake_result()
    res["stages_ms"]["M2L"] = res["dom_ms"] = 0.99
    roof, _ = bench.rooflines(wl, res, "fp64", None, False)
    assert roof["kernel_run"] == "k_m2l_fold<10>"
    assert roof["flop_per_launch"] == bench.fold_flop(10) * (64 + 512 + 4096 + 32768)
    assert roof["achieved"] == pytest.approx(roof["flop_per_launch"] / 0.99e-3 / 1e12) and roof["frac"] < 1
    assert roof["unfolded_tflops"] == pytest.approx(2e4 * 6_039_504 / 0.99e-3 / 1e12)
    res["info"].update(n_boxes=60_000)
    ad, _ = bench.adaptive_rooflines(8, res)
    assert ad["kernel_run"] == ad["kernel"] == "k_ad_m2l_fold<8>"
    assert ad["flop_per_launch"] == bench.fold_flop(8) * 59_991
    for src, name in (("m2l_fold.hip", "k_m2l_fold"), ("m2l_fold_ad.hip", "k_ad_m2l_fold")):
        text = open("%s/paper_1106_2176_amd/csrc/%s" % (ROOT, src)).read()
        assert re.search(r"\b%s\(" % name, text)
