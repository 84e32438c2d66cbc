"""A workspace sized for a caller's largest call serves its smaller ones: the
queried sizes never fall when a dimension grows (no GPU needed)."""
import itertools
import random

import pytest

import paper_cs_0603115_amd as ff


def _never_falls(size, axes, seed, n=4000):
    """size(*v) over random pairs v <= w of the given (low, high) ranges, spread
    over their logarithm, and one step either side of powers of two."""
    rng = random.Random(seed)

    def draw(lo, hi):
        v = int(lo * (hi / lo) ** rng.random())
        if rng.random() < 0.4:
            v = (1 << max(v.bit_length() - 1, 0)) + rng.randint(-1, 1)
        return max(lo, min(hi, v))

    for _ in range(n):
        v = [draw(*a) for a in axes]
        w = [x if rng.random() < 0.4 else draw(x, a[1]) for x, a in zip(v, axes)]
        assert size(*v) <= size(*w), (v, w)


@pytest.mark.parametrize("algo", [ff.GEMM_SLICED_I8, ff.GEMM_SLICED_BF16])
def test_product_workspace_never_falls(algo):
    _never_falls(lambda m, n, k: ff.ff_gemm_workspace_size(m, n, k, algo),
                 [(1, 100000), (1, 100000), (1, 50000)], 11)
    for m, n in itertools.product((64, 65, 128, 129, 256, 257, 512, 16384, 16385), repeat=2):
        assert ff.ff_gemm_workspace_size(m, n, 500, algo) <= \
            ff.ff_gemm_workspace_size(m + 1, n + 1, 500, algo)


def test_matvec_backward_workspace_never_falls():
    _never_falls(lambda m, n: ff.ff_matvec_backward_workspace_size(m, n), [(1, 200000), (1, 70000)], 12)
    # 8192 x 8000 makes more bands than 8192 x 8192
    size = ff.ff_matvec_backward_workspace_size
    assert size(8192, 8000) <= size(8192, 8192)


@pytest.mark.parametrize("cfg", [None, (256, 8192, 0, 32), (64, 0, 0, 1)])
def test_reduction_workspace_never_falls(cfg):
    _never_falls(lambda total, nvec: ff.ff_dot_batched_workspace_size(total, nvec, cfg),
                 [(1, 1 << 31), (1, 300000)], 13)
    size = ff.ff_dot_batched_workspace_size
    assert size(1 << 25, 65536, cfg) <= size(1 << 25, 65537, cfg)
