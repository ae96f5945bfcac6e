"""CPU check of the folding butterflies' bounds: what the compile-time rule admits (the header's own constants) against the 32-bit
arithmetic of the normalisation and of the product, in exact integers."""
import os
import shutil
import subprocess

import pytest

from paper_2604_09975_amd import build

PROGRAM = """
#include <cstdio>
#include "ckks_internal.h"
#include "ntt_device.h"
int main() {
    using F = ckks::FieldPm;
    printf("%u %u %u\\n", F::LIMIT, F::NORMED, F::INV_BASE);
    for (unsigned b = 0; b <= F::LIMIT; ++b) printf("%u ", F::product(b));
}
"""


def _i32(x):
    return (x + 2**31) % 2**32 - 2**31


def _norm(x, b, c):
    """FieldPm::norm as its instructions do it."""
    s, hi = b - 32, _i32(x >> 32)
    lo = (hi + (1 << (s - 1))) % (1 << s) - (1 << (s - 1))
    return (_i32(hi - lo) >> s) * c + (lo << 32) + x % 2**32


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("bounds")
    (d / "b.hip").write_text(PROGRAM)
    subprocess.run([hipcc, "-std=c++17", "-w", "--cuda-host-only", "-I", build.CSRC, "-I", os.path.join(os.path.dirname(build.HERE), "include"),
                    str(d / "b.hip"), "-o", str(d / "b")], check=True, capture_output=True)
    v = [int(x) for x in subprocess.run([str(d / "b")], check=True, capture_output=True, text=True).stdout.split()]
    return v[0], v[1], v[2], v[3:]


def _folding(b):
    """c at both ends of what folds, for q = 2^b - c."""
    return 1, (1 << (b - 35)) - 1


@pytest.mark.parametrize("b", range(51, 61))
def test_values_up_to_the_limit_are_normalised(bounds, b):
    limit, normed = bounds[0], bounds[1]
    for c in _folding(b):
        q = (1 << b) - c
        top = limit * q // 256
        near = [k * (1 << (b - 1)) + e for k in range(16) for e in (-1, 0, 1)]
        for x in [v for v in near + [top, top - 1, top - (1 << 32)] if v <= top]:
            for y in (x, -x):
                z = _norm(y, b, c)
                assert (z - y) % q == 0 and abs(z) * 256 <= normed * q, (b, c, y / q)


@pytest.mark.parametrize("b", range(51, 61))
def test_sums_that_fold30_normalises(bounds, b):
    """top 2^b + low 2^30 folded, plus lo: up to 2^61 whatever the prime."""
    for c in _folding(b):
        q = (1 << b) - c
        for hi in (0, 1, (1 << (b - 1)) - 1):
            for lo in (0, (1 << 59) - 1):
                top, low = hi >> (b - 30), hi % (1 << (b - 30))
                z = _norm(top * c + lo + (low << 30), b, c)
                assert (z - lo - (hi << 30)) % q == 0 and abs(z) <= (1 << (b - 1)) + 2**26


def test_bounds_of_the_schedules(bounds):
    """A product is bounded by (25/32 + 9/256 |y|/q) q; what any sum of the rule may reach stays within 63 bits less the rounding of
    the halves, and a value between an inverse pass's groups can still be summed."""
    limit, normed, inv_base, product = bounds
    assert all(p >= 200 + 9 * b / 256 for b, p in enumerate(product))
    assert limit * 2**60 // 256 < 2**63 - 2**33 and limit < 2048
    assert normed >= 129 and max(product) <= limit and 2 * inv_base <= limit
