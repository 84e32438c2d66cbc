"""The reductions of the sliced product's sums to one signed byte per modulus,
compiled for the host from the kernels' own header and run over whole ranges
of sums: the byte has to be congruent to the sum (no GPU needed)."""
import os
import subprocess

import pytest

from paper_cs_0603115_amd import build as B

SOURCE = r"""
#include "ff_gemm_residue.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
using namespace ffk;

static bool holds(uint32_t word, int64_t s, int m)
{
    return (static_cast<int64_t>(static_cast<int8_t>(word & 255u)) - s) % m == 0;
}

int main(int argc, char **argv)
{
    const int i = std::atoi(argv[2]), m = kModulus[i];
    const float inv = 1.0f / static_cast<float>(m);
    long wrong = 0, seen = 0;
    auto check = [&](bool ok, long s) {
        ++seen;
        if (!ok && ++wrong <= 3)
            std::printf("modulus %d sum %ld\n", m, s);
    };
    if (!std::strcmp(argv[1], "float")) {         // FP32 sums, every one that 640 products reach
        const int start = kFoldUnits * m, most = 640 * (1 << 14) + 130;
        for (int s = start - most; s <= start + most; ++s) {
            const float c = static_cast<float>(s), f = reduce_float(c, m, inv);
            check(static_cast<int>(c) == s && holds(residue_of_float(c, m, inv), s, m), s);
            const int around = static_cast<int>(f) - start;
            check(around >= -129 && around <= 129 && (static_cast<int>(f) - s) % m == 0, s);
        }
    } else if (!std::strcmp(argv[1], "int")) {    // int32 sums next to the halves
        for (int64_t q = -(int64_t(1) << 28) / m; q <= (int64_t(1) << 28) / m; ++q)
            for (int d = m / 2 - 3; d <= m / 2 + 4; ++d) {
                const int64_t s = q * m + d;
                if (s < -(1 << 28) || s > 1 << 28)
                    continue;
                const int v = static_cast<int>(s);
                check(holds(reduce_low_byte(reduce_once(v, m, inv), m, inv), s, m), s);
                if (m <= 244 && s >= -(1 << 26) && s <= 1 << 26)   // K up to 4096
                    check(holds(reduce_low_byte(v, m, inv), s, m), s);
            }
    } else {                                      // sums of digit products, every one
        const BiasedModulus b = kBiased.of[i];
        for (int s = -7 * (1 << 14); s <= 7 * (1 << 14); ++s) {
            check(holds(residue_from_biased(b.bits + s, b), s, m), s);
            const float f = residue_float_from_biased(b.bits + s, b);
            check(f >= -128.0f && f <= 128.0f && (static_cast<int64_t>(f) - s) % m == 0, s);
        }
    }
    std::printf("%ld sums, %ld wrong\n", seen, wrong);
    return wrong || !seen;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = tmp_path_factory.mktemp("residue")
    src, exe = os.path.join(out, "reduction.hip"), os.path.join(out, "reduction")
    with open(src, "w") as f:
        f.write(SOURCE)
    # (-mfma: the host's fused multiply-add instead of a library call)
    proc = subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-mfma", src, "-o", exe],
                          capture_output=True, text=True)
    assert proc.returncode == 0, proc.stderr[-2000:]
    return exe


@pytest.mark.parametrize("modulus", range(16))
@pytest.mark.parametrize("sums", ["float", "int", "digits"])
def test_every_sum_keeps_its_residue(program, sums, modulus):
    proc = subprocess.run([program, sums, str(modulus)], capture_output=True, text=True,
                          timeout=300)
    assert proc.returncode == 0, proc.stdout
