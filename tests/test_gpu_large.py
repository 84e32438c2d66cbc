"""Maximum sizes: every entry point on inputs of more than 2^31 elements,
where any 32-bit element index would wrap.  The HBM of one MI355X (288 GB)
holds these comfortably; each case frees its tensors before the next.

* elementwise Add22 at N = 2^31 + 7 (mixed workload): bit-exact against the
  oracle on the last 2^20 pairs, a window across index 2^31 and a strided
  sample;
* batched dot with a vector of 2^31 + 3 ones times ones: the exact result
  2^31 + 3 (sums of integers below 2^48 are exact in float-float);
* matvec forward and backward on a 65536 x 32769 matrix of ones: y = 32769
  and dx = 65536 exactly, dA = g x^T bit for bit on sampled rows;
* sliced GEMM (int8 digits) with A of 65536 x 32800 (> 2^31 entries, K split
  into chunks): sampled entries within 2^-44 (|A||B|) of the exact product;
* compensated Horner and the binary64 conversions at 2^31 + 5 points:
  bit-exact on the tail, the 2^31 window and a strided sample;
* the batched dot backward over a vector of 2^31 + 3 ones (plus elements
  outside every vector) and the single-dot backward at 2^31 + 9: every
  sampled gradient word equals its closed form (Mul22(g, 1) = g);
* the paper's Add12 stream operator and the copy probe at 2^31 + 11
  elements (closed forms).
"""
import sys
from fractions import Fraction

import numpy as np
import pytest
import torch

import ff_inputs as fi
import oracle
from fpexact import ff_value, same_bits

pytestmark = pytest.mark.gpu

BIG = 1 << 31


def _ff():
    import paper_cs_0603115_amd as ff
    return ff


def _announce(msg):
    print(msg, file=sys.stderr, flush=True)


def _sample_index(n, device):
    """Indices below n: the last 2^20, the window [2^31 - 2048, 2^31 + 2048)
    clipped to n, and every 1000003rd element.  Checked on the host before
    any gather uses them."""
    parts = [torch.arange(n - (1 << 20), n), torch.arange(BIG - 2048, min(n, BIG + 2048)),
             torch.arange(0, n, 1000003)]
    idx = torch.unique(torch.cat(parts))
    assert int(idx.min()) >= 0 and int(idx.max()) < n, "sample index out of range"
    return idx.to(device)


def _free():
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def test_elementwise_beyond_2p31():
    n = BIG + 7
    _announce(f"[gpu] large: ff_add at n={n}")
    ff = _ff()
    a, b, _ = fi.mixed_ff_pair(n, 3101, device="cuda")
    r = ff.ff_add(a, b)
    idx = _sample_index(n, "cuda")
    an, bn, rn = (t[:, idx].cpu().numpy() for t in (a, b, r))
    del a, b, r
    _free()
    rh, rl = oracle.elementwise("add", an[0], an[1], bn[0], bn[1])
    assert same_bits(rn[0], rh) and same_bits(rn[1], rl)


def test_batched_dot_vector_beyond_2p31():
    lengths = [5, BIG + 3, 7]
    _announce(f"[gpu] large: batched dot, vector lengths {lengths}")
    ff = _ff()
    total = sum(lengths)
    x = torch.ones(total, device="cuda")
    y = torch.ones(total, device="cuda")
    offs = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int64,
                        device="cuda")
    d = ff.ff_dot_batched(x, y, offs).cpu().numpy()
    del x, y, offs
    _free()
    for v, length in enumerate(lengths):
        assert ff_value(d[0, v], d[1, v]) == length, (v, d[:, v])


def test_matvec_beyond_2p31():
    M, N = 1 << 16, (1 << 15) + 1
    _announce(f"[gpu] large: matvec {M} x {N} of ones, forward and backward")
    ff = _ff()
    A = torch.zeros((2, M, N), device="cuda")
    A[0].fill_(1.0)
    x = torch.zeros((2, N), device="cuda")
    x[0].fill_(1.0)
    y = ff.ff_matvec(A, x).cpu().numpy()
    assert np.all(y[0] == N) and np.all(y[1] == 0)
    g = torch.stack([fi.gaussian_f32((M,), 3102, device="cuda"), torch.zeros(M, device="cuda")])
    dA, dx = ff.ff_matvec_backward(A, x, g)
    rows = torch.tensor([0, 1, M // 2, M - 2, M - 1], device="cuda")
    dAs = dA[:, rows].cpu().numpy()
    gn = g.cpu().numpy()
    dxn = dx.cpu().numpy()
    del A, x, dA, dx, g
    _free()
    # dA = g x^T with x = 1: every entry of row i is Mul22((g_i, 0), (1, 0)) = (g_i, 0)
    for k, i in enumerate(rows.cpu().numpy()):
        assert np.all(dAs[0, k] == gn[0, i]) and np.all(dAs[1, k] == 0)
    # dx = A^T g: every column sums all of g, exactly as a float-float value
    # to within 2^-44 of the exact sum of |g|
    exact = sum((Fraction(float(v)) for v in gn[0]), Fraction(0))
    scale = sum((abs(Fraction(float(v))) for v in gn[0]), Fraction(0))
    for j in (0, 1, N // 2, N - 1):
        assert abs(ff_value(dxn[0, j], dxn[1, j]) - exact) <= scale / 2 ** 44, j


def test_gemm_operand_beyond_2p31():
    M, K, N = 1 << 16, 32800, 64
    _announce(f"[gpu] large: sliced GEMM {M} x {K} x {N}")
    ff = _ff()
    A = fi.gaussian_ff((M, K), 3103, device="cuda")
    B = fi.gaussian_ff((K, N), 3104, device="cuda")
    C = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_I8).cpu().numpy()
    rows = np.array([0, 1, M // 2, M - 1])
    Asub = A[:, torch.from_numpy(rows).cuda()].cpu().numpy()
    Bn = B.cpu().numpy()
    del A, B
    _free()
    cols = np.array([0, 17, N - 1])
    rr, cc = np.meshgrid(np.arange(rows.size), cols, indexing="ij")
    ex = oracle.exact_gemm_entries(Asub[0], Asub[1], Bn[0], Bn[1], rr.ravel(), cc.ravel())
    ab = oracle.exact_absgemm_entries(Asub[0], Asub[1], Bn[0], Bn[1], rr.ravel(), cc.ravel())
    for t, (i, j) in enumerate(zip(rr.ravel(), cc.ravel())):
        got = ff_value(C[0, rows[i], j], C[1, rows[i], j])
        assert abs(got - ex[t]) <= ab[t] / 2 ** 44, (rows[i], j)


def test_horner_and_conversions_beyond_2p31():
    n = BIG + 5
    _announce(f"[gpu] large: compensated Horner and conversions at n={n}")
    ff = _ff()
    coef = fi.random_poly(3, 3105)
    x = fi.horner_points(n, 3106, -1.5, 1.5, device="cuda")
    y = ff.ff_horner_comp(coef.cuda(), x)
    idx = _sample_index(n, "cuda")
    xs, ys = x[idx].cpu().numpy(), y[idx].cpu().numpy()
    del y
    _free()
    assert same_bits(ys, oracle.horner_comp(coef.numpy(), xs))
    # binary64 -> float-float -> binary64 over the same points
    xd = x.double()
    del x
    _free()
    pair = ff.ff_from_f64(xd)
    ps = pair[:, idx].cpu().numpy()
    xds = xd[idx].cpu().numpy()
    del xd
    _free()
    back = ff.ff_to_f64(pair)
    bs = back[idx].cpu().numpy()
    del pair, back
    _free()
    hi, lo = oracle.from_f64(xds)
    assert same_bits(ps[0], hi) and same_bits(ps[1], lo)
    assert np.array_equal(bs.view(np.uint64), oracle.to_f64(hi, lo).view(np.uint64))


def test_dot_backward_beyond_2p31():
    # x = y = 1: Mul22(g, (1, 0)) = g exactly, so every gradient word is a
    # closed form; the batched form gives each vector's own g and zeros
    # outside all vectors
    lengths = [5, BIG + 3, 7]
    lead, trail = 2, 3
    total = lead + sum(lengths) + trail
    _announce(f"[gpu] large: batched dot backward, total {total}")
    ff = _ff()
    offs_h = np.concatenate([[lead], lead + np.cumsum(lengths)]).astype(np.int64)
    x = torch.ones(total, device="cuda")
    g = torch.tensor([[1.5, -2.0, 0.75], [2.0 ** -30, 2.0 ** -31, -(2.0 ** -27)]], device="cuda")
    dx, dy = ff.ff_dot_batched_backward(g, x, x, torch.from_numpy(offs_h).cuda())
    idx = _sample_index(total, "cuda")
    dxs, dys = dx[:, idx].cpu().numpy(), dy[:, idx].cpu().numpy()
    # every element, segment by segment: a vector's words are its g, the rest zero
    bounds = [0] + [int(o) for o in offs_h] + [total]
    for seg in range(len(bounds) - 1):
        a, b = bounds[seg], bounds[seg + 1]
        v = seg - 1
        for plane in range(2):
            want = float(g[plane, v]) if 0 <= v < len(lengths) else 0.0
            for t in (dx, dy):
                assert bool((t[plane, a:b] == want).all()), (seg, plane)
    del dx, dy
    _free()
    owner = np.searchsorted(offs_h, idx.cpu().numpy(), side="right") - 1
    gn = g.cpu().numpy()
    for k, v in enumerate(owner):
        want = gn[:, v] if 0 <= v < len(lengths) else np.zeros(2, np.float32)
        assert np.array_equal(dxs[:, k], want) and np.array_equal(dys[:, k], want), (k, v)
    # the single-dot backward over float-float inputs of the same length
    n = BIG + 9
    _announce(f"[gpu] large: dot backward, n {n}")
    del x
    _free()
    xf = torch.zeros((2, n), device="cuda")
    xf[0].fill_(1.0)
    g1 = torch.tensor([-3.25, 2.0 ** -29], device="cuda")
    dx, dy = ff.ff_dot_backward(g1, xf, xf)
    idx = _sample_index(n, "cuda")
    dxs, dys = dx[:, idx].cpu().numpy(), dy[:, idx].cpu().numpy()
    del dx, dy, xf
    _free()
    want = g1.cpu().numpy()[:, None]
    assert np.all(dxs == want) and np.all(dys == want)


def test_stream_operators_and_copy_beyond_2p31():
    # Add12 of a = 1 + k 2^-10 (k = i mod 1024) and b = 2^-30: s = a exactly
    # (b is below half an ulp of a), r = b; the copy probe on the same data
    n = BIG + 11
    _announce(f"[gpu] large: Add12 and the copy probe at n={n}")
    ff = _ff()
    a = (torch.arange(n, device="cuda", dtype=torch.int64) % 1024).to(torch.float32)
    a.mul_(2.0 ** -10).add_(1.0)
    b = torch.full((n,), 2.0 ** -30, device="cuda")
    out = ff.ff_add12(a, b)
    idx = _sample_index(n, "cuda")
    outs, as_ = out[:, idx].cpu().numpy(), a[idx].cpu().numpy()
    del out, b
    _free()
    assert np.array_equal(outs[0], as_) and np.all(outs[1] == np.float32(2.0 ** -30))
    dst = torch.empty_like(a)
    ff.ff_copy(a, dst)
    ds = dst[idx].cpu().numpy()
    del a, dst
    _free()
    assert np.array_equal(ds, as_)


def test_horner_beyond_one_launch():
    # more points than one launch has threads for four of each, off 16-byte
    # alignment and in place (69 GB): both parts against torch's two roundings
    import paper_cs_0603115_amd as ff

    n = (1 << 34) + 5
    print(f"[gpu] horner {n} points", flush=True)
    base = torch.full((n + 2,), 7.0, device="cuda")
    x = base[1:n + 1]
    step = 1 << 30
    pattern = torch.arange(step, device="cuda", dtype=torch.float32).remainder_(8191.0).div_(4096.0)
    for at in range(0, n, step):
        m = min(step, n - at)
        x[at:at + m] = pattern[:m] + (at // step)
    coef = torch.tensor([0.3, 1.7], device="cuda")
    ff.ff_horner_f32(coef, x, out=x)
    torch.cuda.synchronize()
    for at in range(0, n, step):
        m = min(step, n - at)
        want = (pattern[:m] + (at // step)).mul_(coef[1]).add_(coef[0])
        assert torch.equal(x[at:at + m], want), at
    assert float(base[0]) == 7.0 and float(base[n + 1]) == 7.0
    del base, x, pattern, want
    torch.cuda.empty_cache()


# Calls whose launches would have 2^32 threads or more, which HIP takes modulo
# 2^32: small integers make every result exact, checked whole in pieces.
STEP = 1 << 30


def _pieces(n):
    for at in range(0, n, STEP):
        yield at, min(STEP, n - at)


def _pattern(period):
    return torch.arange(STEP, device="cuda", dtype=torch.int32).remainder_(period).float()


def test_elementwise_beyond_2p33():
    n = (1 << 33) + 9
    _announce(f"[gpu] large: ff_add in place at n={n}")
    ff = _ff()
    a, b = (torch.zeros((2, n), device="cuda") for _ in range(2))
    p, q = _pattern(1021), _pattern(4093)
    for at, m in _pieces(n):
        a[0, at:at + m], b[0, at:at + m] = p[:m], q[:m]
    ff.ff_add(a, b, out=a)
    for at, m in _pieces(n):
        assert torch.equal(a[0, at:at + m], p[:m] + q[:m]), at
        assert not a[1, at:at + m].any(), at
    del a, b, p, q
    _free()


def test_stream_operator_and_copy_beyond_2p34():
    n = (1 << 34) + 5
    _announce(f"[gpu] large: binary32 add in place and the copy probe at n={n}")
    ff = _ff()
    a, b = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    p, q = _pattern(1021), _pattern(4093)
    for at, m in _pieces(n):
        a[at:at + m], b[at:at + m] = p[:m], q[:m]
    ff.f32_add(a, b, out=a)
    for at, m in _pieces(n):
        assert torch.equal(a[at:at + m], p[:m] + q[:m]), at
    ff.ff_copy(a, b)
    assert torch.equal(a[-4096:], b[-4096:]) and torch.equal(a[:STEP], b[:STEP])
    for at, m in _pieces(n):
        assert torch.equal(b[at:at + m], a[at:at + m]), at
    del a, b, p, q
    _free()


def test_conversions_beyond_2p33():
    n = (1 << 33) + 3
    _announce(f"[gpu] large: conversions at n={n}")
    ff = _ff()
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    p = _pattern(1021).double().add_(2.0 ** -30)
    for at, m in _pieces(n):
        x[at:at + m] = p[:m]
    pair = ff.ff_from_f64(x)
    hi = p.float()
    for at, m in _pieces(n):
        assert torch.equal(pair[0, at:at + m], hi[:m]), at
        assert torch.equal(pair[1, at:at + m].double(), p[:m] - hi[:m].double()), at
        x[at:at + m] = -1.0
    ff.ff_to_f64(pair, out=x)
    for at, m in _pieces(n):
        assert torch.equal(x[at:at + m], p[:m]), at
    del x, pair, p, hi
    _free()


def test_matvec_of_2p28_rows():
    M, N = (1 << 28) + 5, 3
    _announce(f"[gpu] large: matvec {M} x {N}")
    ff = _ff()
    A, x = ff.ff_zeros((M, N)), ff.ff_zeros((N,))
    A[0] = torch.arange(M, device="cuda", dtype=torch.int32).remainder_(1021).float()[:, None]
    x[0] = torch.tensor([1.0, 2.0, 4.0])
    want = A[0, :, 0] * 7
    for algo in (ff.MATVEC_FAST, ff.MATVEC_PLAIN):
        y = ff.ff_matvec(A, x, algo=algo)
        assert torch.equal(y[0], want) and not y[1].any()
    del A, x, y, want
    _free()


@pytest.mark.parametrize("nvec,cfg", [((1 << 24) + 77, None), ((1 << 23) + 5, (512, 0, 0, 1)),
                                      ((1 << 26) + 5, (64, 0, 0, 1))])
def test_reductions_of_many_vectors(nvec, cfg):
    # vectors of 0, 1 and 2 elements in turn
    _announce(f"[gpu] large: reductions of {nvec} vectors, cfg {cfg}")
    ff = _ff()
    lengths = torch.arange(nvec, device="cuda").remainder_(3)
    offs = torch.zeros(nvec + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lengths, 0, out=offs[1:])
    total = int(offs[-1])
    x = torch.arange(total, device="cuda", dtype=torch.int32).remainder_(1021).float()
    first = torch.where(lengths > 0, x[offs[:-1].clamp(max=total - 1)], 0)
    second = torch.where(lengths > 1, x[(offs[:-1] + 1).clamp(max=total - 1)], 0)
    s = ff.ff_sum_batched(x, offs, cfg=cfg)
    assert torch.equal(s[0], first + second) and not s[1].any()
    d = ff.ff_dot_batched(x, x, offs, cfg=cfg)
    assert torch.equal(d[0], first * first + second * second) and not d[1].any()
    del lengths, offs, x, first, second, s, d
    _free()


def test_dot_backward_beyond_2p32_threads():
    total, cut = (1 << 32) + 300, (1 << 32) - 1000
    _announce(f"[gpu] large: batched dot backward, total {total}")
    ff = _ff()
    x = torch.empty(total, device="cuda")
    p = _pattern(1021)
    for at, m in _pieces(total):
        x[at:at + m] = p[:m]
    offs = torch.tensor([3, cut, total - 2], device="cuda")
    g = torch.tensor([[2.0, -3.0], [0.0, 0.0]], device="cuda")
    dx, _ = ff.ff_dot_batched_backward(g, x, x, offs, want_dy=False)
    for at, m in _pieces(total):
        i = torch.arange(at, at + m, device="cuda")
        want = torch.where(i < 3, 0.0, torch.where(i < cut, 2.0 * p[:m],
                                                   torch.where(i < total - 2, -3.0 * p[:m], 0.0)))
        assert torch.equal(dx[0, at:at + m], want), at
        assert not dx[1, at:at + m].any(), at
        del i, want
    del x, dx, p
    _free()
    n = (1 << 33) + 77
    _announce(f"[gpu] large: dot backward, n {n}")
    u = torch.zeros((2, n), device="cuda")
    p = _pattern(1021)
    for at, m in _pieces(n):
        u[0, at:at + m] = p[:m]
    dx, _ = ff.ff_dot_backward(torch.tensor([3.0, 0.0], device="cuda"), u, u, want_dy=False)
    for at, m in _pieces(n):
        assert torch.equal(dx[0, at:at + m], 3.0 * p[:m]), at
        assert not dx[1, at:at + m].any(), at
    del u, dx, p
    _free()


def test_rows_of_2p29_and_2p30_columns():
    M, N = 2, (1 << 29) + 5
    _announce(f"[gpu] large: matvec backward {M} x {N}")
    ff = _ff()
    A, x = ff.ff_zeros((M, N)), ff.ff_zeros((N,))
    row = torch.arange(N, device="cuda", dtype=torch.int32).remainder_(1021).float()
    A[0, 0], A[0, 1] = row, 5.0
    g = torch.tensor([[2.0, 3.0], [0.0, 0.0]], device="cuda")
    _, dx = ff.ff_matvec_backward(A, x, g, want_dA=False)
    assert torch.equal(dx[0], 2.0 * row + 15.0) and not dx[1].any()
    del A, x, row, dx
    _free()
    N = (1 << 30) + 3
    _announce(f"[gpu] large: plain product 1 x {N} x 1")
    B = ff.ff_zeros((1, N))
    B[0, 0] = torch.arange(N, device="cuda", dtype=torch.int32).remainder_(1021).float()
    C = ff.ff_gemm(torch.tensor([[[3.0]], [[0.0]]], device="cuda"), B, algo=ff.GEMM_FMA_LOOP)
    assert torch.equal(C[0, 0], 3.0 * B[0, 0]) and not C[1].any()
    del B, C
    _free()
