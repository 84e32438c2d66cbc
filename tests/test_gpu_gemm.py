"""GPU parity of the float-float GEMM.

* FMA loop: bit-exact against the oracle's plain float-float GEMM (Add22
  accumulation of Mul22 terms, k ascending).
* Sliced (int8 and BF16 digits on matrix cores): against the exact product
  (long accumulator) entry by entry, normwise |C - exact| <= 2^-44 (|A||B|);
  exactly equal to each other (both sum the same digit products exactly);
  exact on integer data and on A times the identity when every row of A sits
  in one binade; on rows and columns spanning 40 binades, within the bound
  the algorithm documents for that case.
"""
import math
import sys
from fractions import Fraction

import numpy as np
import pytest
import torch

import ff_inputs as fi
import oracle
from fpexact import frac, same_bits

pytestmark = pytest.mark.gpu

TWO_M44 = Fraction(1, 1 << 44)


def _ff():
    import paper_cs_0603115_amd as ff
    return ff


def _announce(msg):
    print(msg, file=sys.stderr, flush=True)


def check_entries(A, B, C, rows, cols, label, target=TWO_M44):
    """C at (rows x cols) against the exact product, normwise."""
    An, Bn, Cn = A.cpu().numpy(), B.cpu().numpy(), C.cpu().numpy()
    ri, ci = np.meshgrid(np.asarray(rows), np.asarray(cols), indexing="ij")
    ri, ci = ri.ravel(), ci.ravel()
    exact = oracle.exact_gemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    scale = oracle.exact_absgemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    worst = -math.inf
    for t, (i, j) in enumerate(zip(ri, ci)):
        err = abs(frac(Cn[0, i, j]) + frac(Cn[1, i, j]) - exact[t])
        if scale[t] == 0:
            assert err == 0, (label, i, j)
            continue
        assert err <= target * scale[t], (label, i, j, float(err / scale[t]))
        if err:
            worst = max(worst, math.log2(err / scale[t]))
    return worst


ALGOS = ["i8", "bf16"]


def _algo(name):
    ff = _ff()
    return {"i8": ff.GEMM_SLICED_I8, "bf16": ff.GEMM_SLICED_BF16, "fma": ff.GEMM_FMA_LOOP}[name]


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 3, 7), (64, 64, 64), (100, 70, 333),
                                   (130, 257, 200), (33, 65, 1000)])
def test_fma_loop_is_bitexact(M, N, K):
    ff = _ff()
    A = fi.gaussian_ff((M, K), 11 + M)
    B = fi.gaussian_ff((K, N), 12 + N)
    C = ff.ff_gemm(A.cuda(), B.cuda(), algo=ff.GEMM_FMA_LOOP).cpu().numpy()
    Ch, Cl = oracle.gemm_ff_seq(A[0].numpy(), A[1].numpy(), B[0].numpy(), B[1].numpy())
    assert same_bits(C[0], Ch) and same_bits(C[1], Cl)


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 3, 7), (64, 64, 64), (100, 70, 333),
                                   (130, 257, 200), (33, 65, 1000)])
def test_sliced_against_exact(algo, M, N, K):
    ff = _ff()
    A = fi.gaussian_ff((M, K), 21 + M).cuda()
    B = fi.gaussian_ff((K, N), 22 + N).cuda()
    C = ff.ff_gemm(A, B, algo=_algo(algo))
    check_entries(A, B, C, range(M), range(N), f"{algo} {M}x{N}x{K}")


def test_sliced_int8_and_bf16_agree_bitwise():
    ff = _ff()
    A = fi.gaussian_ff((200, 700), 31).cuda()
    B = fi.gaussian_ff((700, 150), 32).cuda()
    C8 = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_I8)
    C16 = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_BF16)
    again = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_I8)
    assert torch.equal(C8.view(torch.int32), C16.view(torch.int32))
    assert torch.equal(C8.view(torch.int32), again.view(torch.int32))


@pytest.mark.parametrize("algo", ALGOS + ["fma"])
def test_integer_matrices_are_exact(algo):
    ff = _ff()
    rng = np.random.default_rng(41)
    Ai = rng.integers(-3000, 3000, (96, 300))
    Bi = rng.integers(-3000, 3000, (300, 80))
    A = torch.stack([torch.from_numpy(Ai.astype(np.float32)), torch.zeros(96, 300)]).cuda()
    B = torch.stack([torch.from_numpy(Bi.astype(np.float32)), torch.zeros(300, 80)]).cuda()
    C = ff.ff_gemm(A, B, algo=_algo(algo)).cpu().numpy()
    want = Ai @ Bi
    got = C[0].astype(np.int64) + C[1].astype(np.int64)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("algo", ALGOS)
def test_identity_reproduces_single_binade_rows(algo):
    # rows of A inside one binade: the 54-bit fixed point holds every entry's
    # 48 significant bits, and B = I keeps one digit-pair column per entry
    ff = _ff()
    M, K = 70, 96
    mant = fi.random_ff(M * K, 51, 0, 0, max_gap=5).reshape(2, M, K).abs()   # hi in [1, 2)
    lo_sign = torch.sign(fi.random_ff(M * K, 52, 0, 0)[1]).reshape(M, K)
    mant[1] *= lo_sign
    scale = torch.exp2(torch.randint(-20, 20, (M, 1)).float())
    A = (mant * scale).cuda()
    B = torch.stack([torch.eye(K), torch.zeros(K, K)]).cuda()
    C = ff.ff_gemm(A, B, algo=_algo(algo))
    # high words bit for bit; low words by value (an exact zero comes back +0)
    assert torch.equal(C[0].view(torch.int32), A[0].view(torch.int32))
    assert torch.equal(C[1], A[1])


def test_long_k_is_split_into_exact_chunks():
    ff = _ff()
    M, N, K = 64, 48, 16384 + 96
    A = fi.gaussian_ff((M, K), 61).cuda()
    B = fi.gaussian_ff((K, N), 62).cuda()
    for algo in ALGOS:
        C = ff.ff_gemm(A, B, algo=_algo(algo))
        check_entries(A, B, C, range(0, M, 7), range(0, N, 5), f"{algo} long K")


def test_zero_k_gives_zero():
    ff = _ff()
    A = torch.zeros(2, 5, 0, device="cuda")
    B = torch.zeros(2, 0, 6, device="cuda")
    for algo in ALGOS + ["fma"]:
        C = ff.ff_gemm(A, B, algo=_algo(algo))
        torch.cuda.synchronize()
        assert C.shape == (2, 5, 6) and torch.count_nonzero(C) == 0


def test_full_size_4096():
    # C = A B, M = N = K = 4096, entries normal(0,1) split into float-float:
    # 16 seeded 64 x 64 blocks (corners included) against the exact product,
    # the FMA loop bit-exact on one block.
    ff = _ff()
    n = 4096
    _announce("[gpu] gemm 4096^3: generating")
    A = fi.gaussian_ff((n, n), 115004, device="cuda")
    B = fi.gaussian_ff((n, n), 115014, device="cuda")
    _announce("[gpu] gemm 4096^3: sliced int8 and bf16")
    C8 = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_I8)
    C16 = ff.ff_gemm(A, B, algo=ff.GEMM_SLICED_BF16)
    torch.cuda.synchronize()
    assert torch.equal(C8.view(torch.int32), C16.view(torch.int32))
    rng = np.random.default_rng(115004)
    starts = [(0, 0), (0, n - 64), (n - 64, 0), (n - 64, n - 64)]
    starts += [tuple(int(v) for v in rng.integers(0, n - 64, 2)) for _ in range(12)]
    worst = -math.inf
    for bi, (r0, c0) in enumerate(starts):
        _announce(f"  block {bi} at ({r0}, {c0})")
        w = check_entries(A, B, C8, range(r0, r0 + 64), range(c0, c0 + 64), f"block {r0},{c0}")
        worst = max(worst, w)
    _announce(f"  sliced worst normwise log2 error {worst:.2f}")
    _announce("[gpu] gemm 4096^3: FMA loop, one block bit-exact")
    Cp = ff.ff_gemm(A, B, algo=ff.GEMM_FMA_LOOP)
    torch.cuda.synchronize()
    r0, c0 = starts[5]
    An, Bn = A.cpu().numpy(), B.cpu().numpy()
    Ch, Cl = oracle.gemm_ff_seq(An[0], An[1], Bn[0], Bn[1], rows=(r0, r0 + 64), cols=(c0, c0 + 64))
    Cpn = Cp[:, r0:r0 + 64, c0:c0 + 64].cpu().numpy()
    assert same_bits(Cpn[0], Ch) and same_bits(Cpn[1], Cl)
    del A, B, C8, C16, Cp
    torch.cuda.empty_cache()


@pytest.mark.parametrize("algo", ALGOS + ["fma"])
def test_zero_rows_columns_and_power_of_two_maxima(algo):
    # an all-zero row of A and column of B (no largest entry to scale by)
    # give exact zero words; rows and columns whose largest magnitude is an
    # exact power of two (the boundary of the scale choice) and rows holding
    # a single nonzero entry stay within the normwise bound
    M, K, N = 70, 129, 66
    _announce(f"[gpu] gemm zero rows/columns and power-of-two maxima ({algo})")
    A = fi.gaussian_ff((M, K), 7401)
    B = fi.gaussian_ff((K, N), 7402)
    A[:, 3] = 0.0
    B[:, :, 5] = 0.0
    A[:, 10] = 0.0
    A[0, 10, 17] = 2.0 ** 7                      # a single power-of-two entry
    A[:, 11] = A[:, 11] * 2.0 ** -4              # |entries| < 1, then
    A[0, 11, 40], A[1, 11, 40] = -1.0, 0.0       # largest entry exactly -1
    B[:, :, 7] = B[:, :, 7] * 2.0 ** -7          # |entries| < 2^-3, then
    B[0, 64, 7], B[1, 64, 7] = 2.0 ** -3, 0.0    # largest entry exactly 2^-3
    A, B = A.cuda(), B.cuda()
    C = _ff().ff_gemm(A, B, algo=_algo(algo))
    torch.cuda.synchronize()
    Cn = C.cpu().numpy()
    assert np.all(Cn[:, 3, :] == 0) and np.all(Cn[:, :, 5] == 0)
    rows = [0, 3, 10, 11, M - 1]
    cols = [0, 5, 7, 33, N - 1]
    check_entries(A, B, C, rows, cols, f"zero/pow2 {algo}")


def _wide_range_operands(M, K, N, seed):
    """Rows of A and columns of B spanning 40 binades: half the rows (and
    columns) have every entry scaled by 2^s, s uniform in {-40..0}; the other
    half hold one normal(0,1) entry among entries scaled by 2^-40.  Scaling
    by powers of two keeps both words exact."""
    rng = np.random.default_rng(seed)
    A = fi.gaussian_ff((M, K), seed).double()
    B = fi.gaussian_ff((K, N), seed + 1).double()
    sa = rng.integers(-40, 1, (M, K)).astype(np.float64)
    sa[M // 2:] = -40.0
    sa[np.arange(M // 2, M), rng.integers(0, K, M - M // 2)] = 0.0
    sb = rng.integers(-40, 1, (K, N)).astype(np.float64)
    sb[:, N // 2:] = -40.0
    sb[rng.integers(0, K, N - N // 2), np.arange(N // 2, N)] = 0.0
    A = (A * torch.from_numpy(np.exp2(sa))).float()
    B = (B * torch.from_numpy(np.exp2(sb))).float()
    return A, B


@pytest.mark.parametrize("algo", ALGOS)
def test_wide_dynamic_range_within_the_documented_bound(algo):
    # Rows and columns whose entries span 40 binades, where the normwise
    # 2^-44 target is not promised: every entry must still meet the bound the
    # algorithm documents, |C - exact| <= 2^(e_i - 54) sum_k |B_kj|
    # + 2^(f_j - 54) sum_k (|A_ik| + 2^(e_i - 54))   (digit rounding)
    # + K 2^(e_i + f_j - 47)                          (dropped digit pairs)
    # + 2^-47 |C|                                     (final rounding),
    # with 2^e_i above row i's largest |A_ik| and 2^f_j above column j's
    # largest |B_kj| (taken one binade higher here, for either convention).
    M, K, N = 32, 2048, 32
    _announce(f"[gpu] gemm wide dynamic range {M}x{K}x{N} ({algo})")
    A, B = _wide_range_operands(M, K, N, 7301)
    C = _ff().ff_gemm(A.cuda(), B.cuda(), algo=_algo(algo)).cpu().numpy()
    An, Bn = A.numpy(), B.numpy()
    Av = An[0].astype(np.float64) + An[1].astype(np.float64)
    Bv = Bn[0].astype(np.float64) + Bn[1].astype(np.float64)
    e = np.frexp(np.abs(Av).max(axis=1))[1] + 1
    f = np.frexp(np.abs(Bv).max(axis=0))[1] + 1
    ri, ci = np.meshgrid(np.arange(M), np.arange(N), indexing="ij")
    ri, ci = ri.ravel(), ci.ravel()
    exact = oracle.exact_gemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    scale = oracle.exact_absgemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    sumB = np.abs(Bv).sum(axis=0)
    sumA = np.abs(Av).sum(axis=1)
    worst_ratio, worst_normwise = 0.0, -math.inf
    for t, (i, j) in enumerate(zip(ri, ci)):
        err = abs(frac(C[0, i, j]) + frac(C[1, i, j]) - exact[t])
        bound = (math.ldexp(sumB[j], int(e[i]) - 54)
                 + math.ldexp(sumA[i] + K * math.ldexp(1.0, int(e[i]) - 54), int(f[j]) - 54)
                 + K * math.ldexp(1.0, int(e[i] + f[j]) - 47)
                 + math.ldexp(abs(float(exact[t])), -47)) * 1.001
        assert float(err) <= bound, (algo, i, j, float(err), bound)
        worst_ratio = max(worst_ratio, float(err) / bound)
        if err and scale[t]:
            worst_normwise = max(worst_normwise, math.log2(err / scale[t]))
    _announce(f"  worst error / documented bound {worst_ratio:.3g}; "
              f"worst normwise log2 error {worst_normwise:.1f}")


@pytest.mark.parametrize("algo", ALGOS + ["fma"])
def test_strided_operands_and_output(algo):
    # leading dimensions larger than the rows (views into wider buffers),
    # one of them not a multiple of 4 and one operand starting 4 bytes past
    # 16-byte alignment: the slicing kernels take their element paths
    ff = _ff()
    M, N, K = 70, 45, 133
    baseA = fi.gaussian_ff((M, K + 5), 71).cuda()
    baseB = fi.gaussian_ff((K, N + 9), 72).cuda()
    A = baseA[:, :, :K]                       # lda = K + 5
    B = baseB[:, :, 1:N + 1]                  # ldb = N + 9, base + 4 bytes
    Cbuf = torch.full((2, M, N + 3), 7.0, device="cuda")
    C = Cbuf[:, :, :N]                        # ldc = N + 3
    ff.ff_gemm(A, B, algo=_algo(algo), out=C)
    torch.cuda.synchronize()
    assert torch.all(Cbuf[:, :, N:] == 7.0)   # padding columns untouched
    Ac, Bc = A.contiguous(), B.contiguous()
    if algo == "fma":
        Cn = C.cpu().numpy()
        Ch, Cl = oracle.gemm_ff_seq(Ac[0].cpu().numpy(), Ac[1].cpu().numpy(),
                                    Bc[0].cpu().numpy(), Bc[1].cpu().numpy())
        assert same_bits(Cn[0], Ch) and same_bits(Cn[1], Cl)
    else:
        check_entries(Ac, Bc, C.contiguous(), range(M), range(N), f"{algo} strided")
        Cref = ff.ff_gemm(Ac, Bc, algo=_algo(algo))
        assert torch.equal(Cref.view(torch.int32), C.contiguous().view(torch.int32))


def _constant_operands(M, N, K, seed):
    """Every row of A and column of B holds one value throughout, of 48
    random bits: a modulus then sees K equal residue products, up to the
    largest sum it can meet, and C_ij = K a_i b_j exactly."""
    a = fi.random_ff(M, seed, 0, 0, max_gap=0)
    b = fi.random_ff(N, seed + 1, 0, 0, max_gap=0)
    A = a[:, :, None].expand(2, M, K).contiguous()
    B = b[:, None, :].expand(2, K, N).contiguous()
    return a, b, A, B


@pytest.mark.parametrize("algo,M,N,K", [
    ("i8", 130, 190, 31), ("i8", 64, 64, 65), ("i8", 192, 128, 4096),     # small tiles
    ("i8", 192, 128, 4097), ("i8", 700, 650, 449),                        # middle tiles
    ("i8", 2049, 1800, 4096), ("i8", 1900, 2050, 4160),                   # large tiles
    ("bf16", 130, 190, 31), ("bf16", 64, 64, 513), ("bf16", 192, 128, 1537),
    ("bf16", 700, 650, 1024), ("bf16", 2049, 1800, 1000), ("bf16", 1900, 2050, 1600)])
def test_largest_residue_sums_and_tile_edges(algo, M, N, K):
    # C_ij = K a_i b_j: the fixed point (54 bits from the row's power of two)
    # holds a_i and b_j exactly, the integer product is exact, so the only
    # error is the final rounding, at most 2^-48 |C_ij|
    _announce(f"[gpu] gemm constant rows and columns {M}x{N}x{K} ({algo})")
    a, b, A, B = _constant_operands(M, N, K, 8100 + K)
    C = _ff().ff_gemm(A.cuda(), B.cuda(), algo=_algo(algo)).cpu().numpy()
    a, b = a.numpy(), b.numpy()
    rng = np.random.default_rng(K)
    rows = np.unique(np.concatenate([[0, M // 2, M - 1], rng.integers(0, M, 60)]))
    cols = np.unique(np.concatenate([[0, N // 2, N - 1], rng.integers(0, N, 60)]))
    for i in rows:
        ai = K * (frac(a[0, i]) + frac(a[1, i]))
        for j in cols:
            exact = ai * (frac(b[0, j]) + frac(b[1, j]))
            err = abs(frac(C[0, i, j]) + frac(C[1, i, j]) - exact)
            assert err <= abs(exact) / (1 << 48), (i, j)


@pytest.mark.parametrize("algo,M,N,K", [
    # 256 x 128 tiles, one to four stages in a ring of three, and more
    ("i8", 1000, 1000, 33), ("i8", 900, 1020, 65), ("i8", 1024, 1024, 130), ("i8", 1001, 993, 200),
    ("bf16", 1000, 1000, 17), ("bf16", 900, 1020, 33), ("bf16", 1024, 1024, 65),
    ("bf16", 1001, 993, 1100),
    # 256 x 256 tiles, few and many
    ("i8", 2040, 2041, 3100), ("bf16", 2040, 2041, 1600), ("i8", 2950, 3001, 3073),
    # many 64 x 64 tiles, their number no multiple of 8
    ("i8", 60, 8300, 65), ("bf16", 8300, 60, 40)])
def test_tile_choice_and_order(algo, M, N, K):
    # every tile by the rule on M, N and K, in both orders of the workgroups
    test_largest_residue_sums_and_tile_edges(algo, M, N, K)


@pytest.mark.parametrize("M,N,K", [
    (16, 17, 32), (15, 33, 31), (33, 16, 65),          # one output per thread
    (1024, 993, 33), (993, 1025, 64), (1001, 999, 1),  # 2 x 2
    (1985, 2048, 16), (2048, 2001, 35)])               # 4 x 4
def test_fma_loop_tiles_match_the_sequential_definition(M, N, K):
    ff = _ff()
    _announce(f"[gpu] gemm loop {M}x{N}x{K}")
    A, B = fi.gaussian_ff((M, K), 8800 + M), fi.gaussian_ff((K, N), 8801 + N)
    C = ff.ff_gemm(A.cuda(), B.cuda(), algo=_algo("fma")).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(M, 3)), np.linspace(0, M - 1, 9).astype(int),
                                     np.arange(max(0, M - 3), M)]))
    Ar = A[:, rows].numpy()
    Ch, Cl = oracle.gemm_ff_seq(Ar[0], Ar[1], B[0].numpy(), B[1].numpy())
    assert same_bits(C[0, rows], Ch) and same_bits(C[1, rows], Cl)
    cols = np.unique(np.concatenate([np.arange(3), np.arange(max(0, N - 3), N)]))
    Bc = np.ascontiguousarray(B[:, :, cols].numpy())
    Ch, Cl = oracle.gemm_ff_seq(A[0].numpy(), A[1].numpy(), Bc[0], Bc[1])
    assert same_bits(np.ascontiguousarray(C[0][:, cols]), Ch)
    assert same_bits(np.ascontiguousarray(C[1][:, cols]), Cl)


def _residue_operand(n, seed):
    """n float-float numbers 0.75 + t 2^-54 (fixed-point integer 3 2^52 + t):
    number i has, modulo modulus i % 16, one of the residues farthest from
    zero, of either sign."""
    moduli = [256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197, 193]
    rng = np.random.default_rng(seed)
    t = np.empty(n, dtype=np.int64)
    for i in range(n):
        m = moduli[i % 16]
        r = m // 2 - (i // 32) % 4
        t[i] = ((r if i // 16 % 2 else -r) - 3 * 2 ** 52) % m + m * int(rng.integers(0, 1 << 15))
    x = np.empty((2, n), dtype=np.float32)
    x[0], x[1] = 0.75, np.ldexp(t.astype(np.float64), -54)
    assert np.all(x[1].astype(np.float64) == np.ldexp(t.astype(np.float64), -54))
    return x


@pytest.mark.parametrize("algo,M,N,K", [
    # BF16: as many k as pass between two reductions of a sum, every tile
    ("bf16", 128, 128, 640), ("bf16", 128, 128, 656), ("bf16", 128, 128, 703),
    ("bf16", 128, 128, 763), ("bf16", 512, 512, 656), ("bf16", 512, 512, 763),
    ("bf16", 1000, 1000, 763), ("bf16", 1024, 1024, 719), ("bf16", 2048, 2048, 2033),
    ("bf16", 128, 128, 16385),
    # int8: both ends of one and two reductions of a sum
    ("i8", 128, 128, 4095), ("i8", 128, 128, 4096), ("i8", 128, 128, 4097),
    ("i8", 512, 512, 4096), ("i8", 1024, 1024, 4096), ("i8", 128, 128, 16384)])
def test_sums_of_the_farthest_residues(algo, M, N, K):
    # constant rows a_i and columns b_j: C_ij = K a_i b_j, the integer product
    # is exact, and the final rounding is at most 2^-48 |C_ij| (per chunk of
    # 16384 k, and the sum of two chunks 2^-44).  Rows and columns repeat
    # after 128, so that every tile and position sees the same 128 x 128.
    _announce(f"[gpu] gemm farthest residues {M}x{N}x{K} ({algo})")
    a, b = _residue_operand(128, 8500 + K), _residue_operand(128, 8501 + K)
    a[:, ::3] *= -1
    row, col = torch.arange(M) % 128, torch.arange(N) % 128
    A = torch.from_numpy(a).cuda()[:, row, None].expand(2, M, K).contiguous()
    B = torch.from_numpy(b).cuda()[:, None, col].expand(2, K, N).contiguous()
    C = _ff().ff_gemm(A, B, algo=_algo(algo))
    first = C[:, :128, :128].contiguous()
    got = first.cpu().numpy()
    fa = [K * (frac(a[0, i]) + frac(a[1, i])) for i in range(128)]
    fb = [frac(b[0, j]) + frac(b[1, j]) for j in range(128)]
    part = 1 << (48 if K <= 16384 else 44)
    for i in range(128):
        for j in range(128):
            exact = fa[i] * fb[j]
            err = abs(frac(got[0, i, j]) + frac(got[1, i, j]) - exact)
            assert err * part <= abs(exact), (i, j, float(err / exact))
    repeated = first.view(torch.int32)[:, row.cuda()][:, :, col.cuda()]
    assert torch.equal(C.view(torch.int32), repeated)


@pytest.mark.parametrize("algo,M,N,K", [
    # panels of rows, of columns, of both, with one chunk of K and with two
    ("i8", 16500, 70, 40), ("i8", 70, 16500, 40), ("i8", 16500, 16700, 33),
    ("bf16", 33000, 16500, 20), ("i8", 16500, 300, 16390), ("bf16", 200, 16500, 16390),
    # as many rows as the library takes
    ("i8", 262140, 16500, 3)])
def test_panels_of_a_large_product(algo, M, N, K):
    # rows and columns repeat after 127, which no panel or tile is a multiple of,
    # and are scaled by powers of two of their own, so that an entry formed with
    # another panel's rows, columns or scales differs from the 127 x 127 product
    _announce(f"[gpu] gemm panels {M}x{N}x{K} ({algo})")
    ff = _ff()
    a, b = fi.gaussian_ff((127, K), 8700 + K), fi.gaussian_ff((K, 127), 8701 + K)
    a *= torch.exp2((torch.arange(127) % 31 - 15.0))[None, :, None]
    b *= torch.exp2((torch.arange(127) % 29 - 14.0))[None, None, :]
    want = ff.ff_gemm(a.cuda(), b.cuda(), algo=_algo(algo))
    check_entries(a, b, want, range(0, 127, 9), range(0, 127, 9), "panel", TWO_M44)
    A, B = ff.ff_empty((M, K)), ff.ff_empty((K, N))
    A.copy_(a.cuda()[:, torch.arange(M) % 127])
    B.copy_(b.cuda()[:, :, torch.arange(N) % 127])
    C = ff.ff_gemm(A, B, algo=_algo(algo))
    wide = want.view(torch.int32)[:, :, (torch.arange(N) % 127).cuda()]
    for r in range(0, M, 127 * 64):
        rows = min(127 * 64, M - r)
        assert torch.equal(C[:, r:r + rows].view(torch.int32),
                           wide[:, (torch.arange(rows) % 127).cuda()]), r
    del A, B, C, wide
    torch.cuda.empty_cache()


def test_workspace_of_a_large_product_is_bounded():
    size = _ff().ff_gemm_workspace_size
    for n, algo in ((65536, "i8"), (65536, "bf16"), (200000, "i8")):
        assert size(n, n, n, _algo(algo)) < 25 << 30
    assert size(4096, 4096, 1 << 21, _algo("i8")) < 4 << 30
    planes = 16 * (2 * 4096 * 4096 + 4096 * 4096)      # those of 4096^3, all held
    assert planes <= size(4096, 4096, 4096, _algo("i8")) < planes + (1 << 20)


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("M,K,N", [(32, 2048, 32), (40, 17000, 36)])
def test_fixed_point_and_final_rounding_are_the_only_errors(algo, M, K, N):
    # the header's bound as it stands, with 2^e_i the power of two above row i's
    # largest |hi| and 2^f_j above column j's: no digit product is dropped, so
    # rows and columns spanning 40 binades meet it without a term in K; each
    # further chunk of 16384 k adds its own rounding and one Add22 (2^-44)
    _announce(f"[gpu] gemm documented bound {M}x{K}x{N} ({algo})")
    A, B = _wide_range_operands(M, K, N, 7501)
    C = _ff().ff_gemm(A.cuda(), B.cuda(), algo=_algo(algo)).cpu().numpy()
    An, Bn = A.numpy(), B.numpy()
    Av, Bv = An.astype(np.float64).sum(0), Bn.astype(np.float64).sum(0)
    e = np.frexp(np.abs(An[0]).max(axis=1))[1]
    f = np.frexp(np.abs(Bn[0]).max(axis=0))[1]
    ri, ci = (t.ravel() for t in np.meshgrid(np.arange(0, M, 3), np.arange(0, N, 3), indexing="ij"))
    exact = oracle.exact_gemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    scale = oracle.exact_absgemm_entries(An[0], An[1], Bn[0], Bn[1], ri, ci)
    sumA, sumB = np.abs(Av).sum(axis=1), np.abs(Bv).sum(axis=0)
    for t, (i, j) in enumerate(zip(ri, ci)):
        err = abs(frac(C[0, i, j]) + frac(C[1, i, j]) - exact[t])
        bound = Fraction(math.ldexp(sumB[j], int(e[i]) - 54)
                         + math.ldexp(sumA[i] + K * math.ldexp(1.0, int(e[i]) - 54),
                                      int(f[j]) - 54)) * Fraction(1000001, 1000000)
        bound += abs(exact[t]) / (1 << 47) + (scale[t] / (1 << 44) if K > 16384 else 0)
        assert err <= bound, (i, j, float(err / bound))
