"""GPU parity of rescale on every ring its fused kernels are instantiated for (N = 2^12 .. 2^16), the rings beside them and
a chain with a prime above 2^50 (plain form): levels from 2 up, more limbs than one group of eight targets, extreme
residues in the dropped limb, and more rows than one call of the scratch chunk."""
import numpy as np
import pytest

from tests import helpers
from tests.gpu_util import make_pair, to_dev, to_host
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,L,level,qbits,n_ct", [(11, 4, 4, 50, 2), (12, 3, 3, 50, 3), (12, 11, 11, 40, 1), (12, 4, 3, 52, 2),
                                                     (13, 10, 9, 50, 2), (13, 2, 2, 50, 1), (14, 6, 5, 50, 2),
                                                     (15, 9, 9, 50, 1), (16, 18, 17, 50, 1), (16, 2, 2, 50, 2), (17, 3, 3, 50, 1),
                                                     (12, 2, 2, 50, 70),
                                                     # three groups of limbs among three workgroups, two and one
                                                     (13, 18, 18, 50, 8), (13, 18, 18, 50, 12), (13, 18, 18, 50, 25)])
def test_rescale_shapes(logN, L, level, qbits, n_ct):
    from paper_2604_09975_amd import binding as B
    O = helpers.small_oracle(logN, L=L, K=1, dnum=2 if L % 2 == 0 else 1, qbits=qbits, pbits=57)
    _, P = make_pair(O)
    r = W.rng(100 * logN + L)
    ct = W.uniform_residues(r, O.q[:level], O.N, lead=(n_ct, 2))
    ql = int(O.q[level - 1])
    # dropped limbs at the rounding boundary: constants floor(q_l/2), floor(q_l/2) + 1, q_l - 1 in the coefficient domain
    for c, v in enumerate([ql // 2, ql // 2 + 1, ql - 1][:2 * n_ct]):
        ct[c // 2, c % 2, level - 1] = v                     # the transform of a constant is the constant
    got = to_host(B.ckks_rescale(P, to_dev(ct), level, n_ct))
    assert (got == O.rescale(ct, level)).all()
