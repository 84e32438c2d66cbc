"""Performance cases of the float-float library.

Each case is one call (or one forward and backward step) through the package's
public entry points, at sizes from the benchmark, the tests and between:

* elementwise operators, from a few thousand values (launch latency) to the
  benchmark's 2^28 mixed pairs (HBM streaming);
* batched dots and sums over uneven vectors, binary32 and float-float terms,
  from a batch that fits one workgroup's worth of work to the benchmark's 4096
  vectors of 2^6 to 2^20 elements; a training step (forward and backward
  through autograd) on such batches;
* matrix-vector products, forward alone and forward plus backward, square,
  tall, wide and odd-sized;
* matrix products with int8 and BF16 digits and by the plain loop, small,
  ragged and the benchmark's 4096^3, on float-float matrices or, as programs
  that hold binary64 data do, converted on the way in and out;
* polynomial evaluation at many points.
"""
import math

import torch

import paper_cs_0603115_amd as ff
from paper_cs_0603115_amd import autograd as ffa

DEVICE = "cuda"

ELEMENTWISE = {
    "add": ff.ff_add, "sub": ff.ff_sub, "mul": ff.ff_mul, "div": ff.ff_div,
    "mul_dekker": ff.ff_mul_dekker, "add_accurate": ff.ff_add_accurate,
    "mul_accurate": ff.ff_mul_accurate, "div_accurate": ff.ff_div_accurate,
}
# entry point, input vectors, planes per input
REDUCTIONS = {
    "dot": (ff.ff_dot_batched, 2, 1), "dot_ff": (ff.ff_dot_ff_batched, 2, 2),
    "sum": (ff.ff_sum_batched, 1, 1), "sum_ff": (ff.ff_sum_ff_batched, 1, 2),
    "dot2": (ff.ff_dot2_batched, 2, 1), "sum2": (ff.ff_sum2_batched, 1, 1),
}
GEMM = {"int8": ff.GEMM_SLICED_I8, "bf16": ff.GEMM_SLICED_BF16, "loop": ff.GEMM_FMA_LOOP}
# binary32 operations per point and degree
HORNER_OPS = {"f32": 2, "comp": 11, "ff": 23}


def listed():
    return [
        # A few thousand values: what an interactive program or the inner loop
        # of a small solver calls; the launch and the call itself count.
        {"name": "add_small", "kind": "elementwise", "op": "add", "n": 4099},
        # The benchmark's step: 2^28 mixed pairs resident in HBM.
        {"name": "div_large", "kind": "elementwise", "op": "div", "n": 1 << 28},
        # A small batch of short dots, as in an orthogonalisation step.
        {"name": "dot_small", "kind": "reduction", "terms": "dot", "nvec": 61,
         "log2_min": 6.0, "log2_max": 11.0},
        # The benchmark's batch: 4096 uneven vectors, 439 M elements.
        {"name": "dot_large", "kind": "reduction", "terms": "dot", "nvec": 4096,
         "log2_min": 6.0, "log2_max": 20.0},
        # One training step over an ordinary batch of float-float vectors.
        {"name": "dot_train", "kind": "dot_train", "nvec": 500, "log2_min": 6.0,
         "log2_max": 16.0},
        # An ordinary matrix with odd dimensions, forward only.
        {"name": "matvec_odd", "kind": "matvec", "m": 1000, "n": 1531, "train": False},
        # The benchmark's matrix: forward and both gradients.
        {"name": "matvec_train", "kind": "matvec", "m": 8192, "n": 8192, "train": True},
        # A small product of binary64 matrices done in float-float.
        {"name": "gemm_small_f64", "kind": "gemm", "algo": "int8", "m": 200, "n": 300, "k": 257,
         "f64": True},
        # An ordinary product, no dimension a multiple of a tile.
        {"name": "gemm_ragged", "kind": "gemm", "algo": "int8", "m": 1000, "n": 1531, "k": 2047,
         "f64": False},
        # The benchmark's product.
        {"name": "gemm_large", "kind": "gemm", "algo": "int8", "m": 4096, "n": 4096, "k": 4096,
         "f64": False},
        # The BF16 matrix cores, for programs that choose them.
        {"name": "gemm_bf16", "kind": "gemm", "algo": "bf16", "m": 2048, "n": 2048, "k": 2048,
         "f64": False},
        # A polynomial of the benchmark's degree at an ordinary number of points.
        {"name": "horner_comp", "kind": "horner", "form": "comp", "n": (1 << 22) + 3,
         "degree": 25},
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["elementwise", "reduction", "dot_train", "matvec", "gemm", "gemm", "horner"])
    if kind == "elementwise":
        return {"kind": kind, "op": rng.choice(sorted(ELEMENTWISE)),
                "n": _log_uniform(rng, 1000, 1 << 28)}
    if kind in ("reduction", "dot_train"):
        case = {"kind": kind}
        if kind == "reduction":
            case["terms"] = rng.choice(sorted(REDUCTIONS))
        log2_max = round(rng.uniform(8.0, 20.0 if kind == "reduction" else 17.0), 2)
        most = 4096 if log2_max <= 16.0 else 1024   # bounds the elements of a batch
        case.update(nvec=_log_uniform(rng, 1, most), log2_min=round(rng.uniform(2.0, 7.0), 2),
                    log2_max=log2_max)
        return case
    if kind == "matvec":
        m = _log_uniform(rng, 64, 16384)
        return {"kind": kind, "m": m, "n": _log_uniform(rng, 64, min(16384, (1 << 26) // m)),
                "train": rng.random() < 0.5}
    if kind == "gemm":
        algo = rng.choice(["int8", "int8", "int8", "bf16", "loop"])
        most = {"int8": 4096, "bf16": 3072, "loop": 1024}[algo]
        m, n, k = (_log_uniform(rng, 64, most) for _ in range(3))
        return {"kind": kind, "algo": algo, "m": m, "n": n, "k": k, "f64": rng.random() < 0.3}
    return {"kind": kind, "form": rng.choice(sorted(HORNER_OPS)),
            "n": _log_uniform(rng, 1000, 1 << 26), "degree": rng.randint(3, 40)}


# ------------------------------------------------------------------- inputs

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _split(x):
    """binary64 values -> float-float planes, in the layout of ff_empty."""
    out = ff.ff_empty(x.shape, device=DEVICE)
    out[0] = x
    out[1] = x - out[0].double()
    return out


def _join(t):
    return t[0].double() + t[1].double()


def _sign(n, g):
    return torch.randint(0, 2, (n,), generator=g, device=DEVICE, dtype=torch.int8).double() * 2 - 1


def _operands(n, seed):
    """Operand pairs: magnitudes 2^-20 to 2^20, a quarter that nearly cancel
    (b = -a (1 + eps)) and a tenth 24 to 60 binades apart."""
    g = _generator(seed)

    def uniform(lo, hi):
        return torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64) * (hi - lo) + lo

    a = _sign(n, g) * torch.exp2(uniform(-20, 20))
    b = _sign(n, g) * torch.exp2(uniform(-20, 20))
    pick = torch.rand(n, generator=g, device=DEVICE)
    b = torch.where(pick < 0.25, -a * (1 + _sign(n, g) * torch.exp2(uniform(-40, -10))), b)
    b = torch.where(pick > 0.90, a.abs() * torch.exp2(uniform(-60, -24)), b)
    return a, b


def _normal(shape, seed):
    return torch.randn(shape, generator=_generator(seed), device=DEVICE, dtype=torch.float64)


def _lengths(case):
    """Uneven vectors: lengths 2^U, U evenly spread over its range."""
    u = (torch.arange(case["nvec"], dtype=torch.float64) + 0.5) / case["nvec"]
    u = u * (case["log2_max"] - case["log2_min"]) + case["log2_min"]
    return torch.floor(torch.exp2(u)).to(torch.int64)


def _offsets(case, seed):
    """The vectors back to back in a random order: their starts."""
    g = torch.Generator()
    g.manual_seed(int(seed))
    starts = torch.zeros(case["nvec"] + 1, dtype=torch.int64)
    starts[1:] = torch.cumsum(_lengths(case)[torch.randperm(case["nvec"], generator=g)], 0)
    return starts


def _terms(total, seed, planes):
    """normal(0,1) * 2^k, k in [-10, 10]: binary32, or binary64 values to be
    split."""
    g = _generator(seed)
    dtype = torch.float32 if planes == 1 else torch.float64
    z = torch.randn(total, generator=g, device=DEVICE, dtype=dtype)
    k = torch.randint(-10, 11, (total,), generator=g, device=DEVICE, dtype=torch.int32)
    return torch.ldexp(z, k)


def _polynomial(case, seed):
    coef = _normal((case["degree"] + 1,), seed).float()
    x = torch.rand(case["n"], generator=_generator(seed + 1), device=DEVICE,
                   dtype=torch.float64) * 2.5 - 1.25
    return coef, x


def prepare(case, seed):
    kind, seed = case["kind"], 1000 * int(seed)
    if kind == "elementwise":
        a, b = _operands(case["n"], seed)
        return case, _split(a), _split(b)
    if kind == "reduction":
        _, count, planes = REDUCTIONS[case["terms"]]
        starts = _offsets(case, seed)
        data = [_terms(int(starts[-1]), seed + 1 + i, planes) for i in range(count)]
        return case, [d if planes == 1 else _split(d) for d in data], starts.to(DEVICE)
    if kind == "dot_train":
        starts = _offsets(case, seed)
        x, y = (_split(_terms(int(starts[-1]), seed + 1 + i, 2)).requires_grad_()
                for i in range(2))
        return case, x, y, starts.to(DEVICE), _split(_normal((case["nvec"],), seed + 3))
    if kind == "matvec":
        a = _split(_normal((case["m"], case["n"]), seed))
        x = _split(_normal((case["n"],), seed + 1))
        if case["train"]:
            a.requires_grad_()
            x.requires_grad_()
        return case, a, x, _split(_normal((case["m"],), seed + 2))
    if kind == "gemm":
        a = _normal((case["m"], case["k"]), seed)
        b = _normal((case["k"], case["n"]), seed + 1)
        return (case, a, b) if case["f64"] else (case, _split(a), _split(b))
    coef, x = _polynomial(case, seed)
    return case, coef, _split(x) if case["form"] == "ff" else x.float()


# --------------------------------------------------------------------- pass

def run(state):
    case, kind = state[0], state[0]["kind"]
    if kind == "elementwise":
        return ELEMENTWISE[case["op"]](state[1], state[2])
    if kind == "reduction":
        return REDUCTIONS[case["terms"]][0](*state[1], state[2])
    if kind == "dot_train":
        _, x, y, offsets, g = state
        s = ffa.FFDotBatched.apply(x, y, offsets)
        return (s.detach(), *torch.autograd.grad(s, (x, y), g))
    if kind == "matvec":
        _, a, x, g = state
        if not case["train"]:
            return ff.ff_matvec(a, x)
        y = ffa.FFMatVec.apply(a, x)
        return (y.detach(), *torch.autograd.grad(y, (a, x), g))
    if kind == "gemm":
        _, a, b = state
        if case["f64"]:
            return ff.ff_to_f64(ff.ff_gemm(ff.ff_from_f64(a), ff.ff_from_f64(b),
                                           algo=GEMM[case["algo"]]))
        return ff.ff_gemm(a, b, algo=GEMM[case["algo"]])
    _, coef, x = state
    if case["form"] == "f32":
        return ff.ff_horner_f32(coef, x)
    if case["form"] == "comp":
        return ff.ff_horner_comp(coef, x)
    return ff.ff_horner_ff(coef, x)


def work(case):
    kind = case["kind"]
    if kind == "elementwise":
        return {"bytes": 24 * case["n"], "flops": 0}
    if kind == "reduction":
        _, count, planes = REDUCTIONS[case["terms"]]
        return {"bytes": 4 * count * planes * int(_lengths(case).sum()) + 16 * case["nvec"],
                "flops": 0}
    if kind == "dot_train":   # x and y read twice (forward, backward), dx and dy written
        return {"bytes": 48 * int(_lengths(case).sum()) + 32 * case["nvec"], "flops": 0}
    if kind == "matvec":      # A read (twice with the backward), dA written
        m, n = case["m"], case["n"]
        return {"bytes": 8 * (m * n * (3 if case["train"] else 1) + 2 * (m + n)), "flops": 0}
    if kind == "gemm":        # a float-float multiply-add counted as two operations
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 8 * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    planes = 2 if case["form"] == "ff" else 1
    return {"bytes": 8 * planes * case["n"],
            "flops": HORNER_OPS[case["form"]] * case["degree"] * case["n"]}


# -------------------------------------------------------------------- exact

def _planes64(x):
    """Value in 64 bits, in float-float layout: the nearest binary32 and the
    rest of it."""
    hi = x.float().double()
    return torch.stack([hi, x - hi])


def exact(case, seed):
    kind = case["kind"]
    state = prepare(case, seed)
    if kind == "elementwise":
        a, b = _join(state[1]), _join(state[2])
        op = case["op"].split("_")[0]
        value = {"add": torch.add, "sub": torch.sub, "mul": torch.mul, "div": torch.div}[op]
        return _planes64(value(a, b))
    if kind in ("reduction", "dot_train"):
        if kind == "reduction":
            planes = REDUCTIONS[case["terms"]][2]
            data = [d.double() if planes == 1 else _join(d) for d in state[1]]
        else:
            data = [_join(state[1].detach()), _join(state[2].detach())]
        starts = _offsets(case, 1000 * int(seed))
        lengths = starts[1:] - starts[:-1]
        products = data[0] * data[1] if len(data) == 2 else data[0]
        sums = torch.stack([part.sum() for part in torch.split(products, lengths.tolist())])
        if kind == "reduction":
            return _planes64(sums)
        g = torch.repeat_interleave(_join(state[4]), lengths.to(DEVICE))
        return _planes64(sums), _planes64(g * data[1]), _planes64(g * data[0])
    if kind == "matvec":
        a, x, g = (_join(t.detach()) for t in state[1:])
        y = _planes64((a * x).sum(1))
        if not case["train"]:
            return y
        return y, _planes64(torch.outer(g, x)), _planes64((a * g[:, None]).sum(0))
    if kind == "gemm":
        if case["f64"]:
            return state[1] @ state[2]
        return _planes64(_join(state[1]) @ _join(state[2]))
    coef, x = state[1].double(), _join(state[2]) if case["form"] == "ff" else state[2].double()
    value = torch.zeros_like(x) + coef[-1]
    for c in coef.flip(0)[1:]:
        value = value * x + c
    return _planes64(value) if case["form"] == "ff" else value
