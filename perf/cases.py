"""What a user of the library has it do, as cases that can be timed.

A case is a dict of plain values:
  call      "step"      a time step: Tree.rebuild on the current positions, then Tree.evaluate
            "evaluate"  new charges on a tree that is kept (an iterative solver's product)
            "oneshot"   the module's evaluate(): tree, evaluation and release in one call
            "grad"      the differentiable potential() and its gradients for a weighted-potential loss
  n, p, leaf_max, precision ("mixed" / "fp64"), dtype ("f64" / "f32"), vec ("field" / "force" / None)
  adaptive  the adaptive octree, on particles in Gaussian blobs ("blobs"), else the uniform one
  charges   "u01" (U[0,1)) or "u11" (U[-1,1), zero mean)
  lo, size  root cube
"""
import math

import torch

import paper_1106_2176_amd as fmm

# direct sums of exact() up to this many particles
EXACT_MAX = 100_000


def _case(name, call, n, p, leaf_max, precision="mixed", dtype="f64", vec="field", adaptive=False,
          points="uniform", charges="u01", lo=0.0, size=1.0):
    c = dict(call=call, n=n, p=p, leaf_max=leaf_max, precision=precision, dtype=dtype, vec=vec,
             adaptive=adaptive, points=points, charges=charges, lo=lo, size=size)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest problem of the benchmark: an evaluation on a kept tree,
        # where latency and launches count
        _case("evaluate_1e4_p4", "evaluate", 10_000, 4, 64),
        # the same size as a time step, with the build's wait for the host
        _case("step_1e4_p4", "step", 10_000, 4, 64, vec="force"),
        # a small problem in the plain FP64 form (a reference result, a test)
        _case("evaluate_20011_p8_fp64", "evaluate", 20_011, 8, 48, precision="fp64"),
        # the flagship workload: a million particles at order 10
        _case("step_1e6_p10", "step", 1_000_000, 10, 64),
        # the same in the plain FP64 form
        _case("step_1e6_p10_fp64", "step", 1_000_000, 10, 64, precision="fp64"),
        # ten million charges of both signs (zero mean), fuller leaves
        _case("step_1e7_p10", "step", 10_000_000, 10, 128, charges="u11"),
        # the largest: a hundred million particles in FP32
        _case("step_1e8_p8_f32", "step", 100_000_000, 8, 128, dtype="f32"),
        # training: forward and backward through autograd, trees made inside
        _case("grad_1e6_p8", "grad", 1_000_000, 8, 64),
        # gradients in FP64 at a high order, a ragged size
        _case("grad_87641_p12_fp64", "grad", 87_641, 12, 50, precision="fp64", charges="u11"),
        # one call from FP32 tensors, a box away from the origin, forces
        _case("oneshot_300007_p6_f32", "oneshot", 300_007, 6, 40, dtype="f32", vec="force", lo=-5.0, size=10.0),
        # clustered particles on the adaptive tree, both forms
        _case("adaptive_1e6_p8", "step", 1_000_000, 8, 64, adaptive=True, points="blobs"),
        _case("adaptive_1e6_p8_fp64", "step", 1_000_000, 8, 64, precision="fp64", adaptive=True, points="blobs"),
    ]


def draw(rng):
    precision = rng.choice(["mixed", "mixed", "fp64"])
    adaptive = rng.random() < 0.25
    call = rng.choice(["step", "step", "evaluate", "oneshot", "grad"])
    p = rng.randint(3, 14)
    leaf_max = rng.randint(32, 128)
    # up to 10^7 particles, fewer where the order, the form or the pass is
    # dearer, so that no draw costs more than the largest listed case
    top = 1e7 / (max(1.0, (p / 10.0) ** 3) * (3.0 if precision == "fp64" else 1.0) * (2.5 if call == "grad" else 1.0)
                 * (3.0 if adaptive else 1.0))
    n = int(math.exp(rng.uniform(math.log(1e3), math.log(top)))) | 1
    return _case(None, call, n, p, leaf_max, precision=precision, dtype=rng.choice(["f64", "f64", "f32"]),
                 vec=rng.choice(["field", "force", None]) if call != "grad" else "field", adaptive=adaptive,
                 points="blobs" if adaptive else "uniform", charges=rng.choice(["u01", "u11"]),
                 lo=rng.choice([0.0, -1.0]), size=rng.choice([1.0, 2.0]))


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, dt = case["n"], torch.float64 if case["dtype"] == "f64" else torch.float32

    def rand(*shape, dtype=dt):
        return torch.rand(*shape, generator=g, device="cuda", dtype=dtype)

    if case["points"] == "blobs":
        # six blobs of widths 0.005 .. 0.06 of the box
        cen = 0.2 + 0.6 * rand(6, 3, dtype=torch.float64)
        width = torch.logspace(math.log10(0.005), math.log10(0.06), 6, dtype=torch.float64, device="cuda")
        lab = torch.randint(0, 6, (n,), generator=g, device="cuda")
        x = cen[lab] + torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64) * width[lab, None]
        pos = x.clamp_(0.0, 1.0 - 2.0 ** -20).to(dt)
    else:
        pos = rand(n, 3)
    pos = (pos * case["size"] + case["lo"]).clamp_(case["lo"], case["lo"] + case["size"])
    q = rand(n)
    if case["charges"] == "u11":
        q = 2.0 * q - 1.0
    w = torch.randn(n, generator=g, device="cuda", dtype=dt) if case["call"] == "grad" else None
    return pos, q, w


def _options(case):
    return dict(p=case["p"], leaf_max=case["leaf_max"], precision=case["precision"], adaptive=case["adaptive"],
                box_lo=(case["lo"],) * 3, box_size=case["size"])


def prepare(case, seed):
    pos, q, w = _inputs(case, seed)
    s = dict(case=case, pos=pos, q=q, w=w, opt=_options(case), tree=None)
    if case["call"] in ("step", "evaluate"):
        s["tree"] = fmm.Tree(pos, **s["opt"])
    elif case["call"] == "grad":
        pos.requires_grad_(True)
        q.requires_grad_(True)
    return s


def run(s):
    case = s["case"]
    if case["call"] == "step":
        return s["tree"].rebuild(s["pos"]).evaluate(s["q"], vec=case["vec"])
    if case["call"] == "evaluate":
        return s["tree"].evaluate(s["q"], vec=case["vec"])
    if case["call"] == "oneshot":
        return fmm.evaluate(s["pos"], s["q"], vec=case["vec"], **s["opt"])
    phi = fmm.potential(s["pos"], s["q"], **s["opt"])
    gx, gq = torch.autograd.grad(phi, (s["pos"], s["q"]), grad_outputs=s["w"])
    return phi.detach(), gq, gx


def _level(n, leaf_max):
    """The uniform tree's leaf level: the fullest of 8^l Poisson leaves holds leaf_max."""
    for lev in range(10):
        mean = n / 8.0 ** lev
        if mean + (3.0 + 0.3 * lev) * math.sqrt(mean) <= leaf_max or n <= leaf_max:
            return lev
    return 10


def work(case):
    n, p = case["n"], case["p"]
    size = 8 if case["dtype"] == "f64" else 4
    if case["adaptive"]:
        # per particle on the blobs, for fuller leaves more pairs and fewer
        # translations (measured at leaf_max 64)
        pairs = 1290.0 * n * case["leaf_max"] / 64.0
        v = 7.2 * n * 64.0 / case["leaf_max"]
        other = 8.7 * n * 35.0 * p * p  # the W and X lists
    else:
        lev = _level(n, case["leaf_max"])
        side = 2 ** lev
        pairs = float(n) * n / 8.0 ** lev * ((3.0 * side - 2.0) / side) ** 3
        v, other = 0.0, 0.0
        for j in range(2, lev + 1):
            m = 2 ** j
            # ordered pairs of boxes whose parents touch and which do not
            v += (6.0 * m - 8.0) ** 3 - (3.0 * m - 2.0) ** 3
    flops = 19.0 * pairs + 2.0 * p ** 4 * v + 11.0 * p * p * n + other
    words = 3 + 1 + 1 + (3 if case["vec"] else 0)
    if case["call"] == "grad":
        # the field is computed with the potential; back: w, dL/dq, dL/dx
        flops, words = 2.0 * flops, 3 + 1 + 1 + 1 + 1 + 3
    return {"bytes": float(words * size * n), "flops": flops}


def exact(case, seed):
    if case["n"] > EXACT_MAX:
        return None
    pos, q, w = (None if t is None else t.double() for t in _inputs(case, seed))
    n = case["n"]

    def direct(charges):
        phi, field = torch.empty_like(charges), torch.empty_like(pos)
        rows = max(1, 20_000_000 // n)
        for i in range(0, n, rows):
            d = pos[i:i + rows, None, :] - pos[None, :, :]
            r2 = d.square().sum(-1)
            k = torch.where(r2 > 0, r2.rsqrt(), torch.zeros_like(r2)) * charges
            phi[i:i + rows] = k.sum(1)
            k = torch.where(r2 > 0, k / r2, k)
            field[i:i + rows] = (k[:, :, None] * d).sum(1)
        return phi, field

    phi, field = direct(q)
    if case["call"] == "grad":
        phi_w, field_w = direct(w)
        return phi, phi_w, -(w[:, None] * field + q[:, None] * field_w)
    if case["vec"] is None:
        return phi, None
    return phi, field * q[:, None] if case["vec"] == "force" else field
