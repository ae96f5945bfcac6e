"""GPU parity: ctmul + relinearisation and the relinearisation key generation against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from tests import helpers
from tests.gpu_util import make_pair, to_dev, to_host
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


def _case(O, P, level, seed, scale, hw):
    from paper_2604_09975_amd import binding as B
    cl = helpers.Client(O, seed, hamming_weight=hw)
    r = W.rng(seed)
    za, zb = W.unit_disk_slots(r, O.n), W.unit_disk_slots(r, O.n)
    ca, cb = cl.encrypt_slots(za, scale, level), cl.encrypt_slots(zb, scale, level)
    rk = cl.relin_key()
    h = B.ckks_relin_key_load(P, to_dev(rk))
    got = to_host(B.ckks_ctmul(P, to_dev(ca), to_dev(cb), level, h))
    want = O.ctmul(ca, cb, level, rk)
    assert (got == want).all()
    return cl, za, zb, got


@pytest.mark.parametrize("level", [3, 2, 1])
def test_toy_ring(level):
    O, P = make_pair(W.TOY_RING)
    from paper_2604_09975_amd import binding as B
    cl, za, zb, got = _case(O, P, level, 70 + level, 2.0**30, 64)
    if level > 1:
        out = to_host(B.ckks_rescale(P, to_dev(got[None]), level, 1))[0]
        zz = cl.decrypt_slots(out, level - 1, 2.0**60 / O.q[level - 1], nlimbs=min(level - 1, 2))
        assert np.abs(zz - za * zb).max() < 2e-3


@pytest.mark.parametrize("L,K,dnum,level,qbits,pbits", [(4, 2, 2, 3, 40, 45), (6, 3, 2, 6, 52, 55)])
def test_small_rings_generic_path(L, K, dnum, level, qbits, pbits):
    O = helpers.small_oracle(10, L=L, K=K, dnum=dnum, qbits=qbits, pbits=pbits)
    _, P = make_pair(O)
    _case(O, P, level, 80 + L, 2.0**30, 16)


@pytest.mark.parametrize("logN,L,K,dnum,level,qbits,pbits", [(12, 4, 2, 2, 3, 50, 60), (12, 4, 4, 1, 4, 52, 60), (12, 3, 3, 1, 2, 61, 62),
                                                              (13, 4, 2, 2, 4, 50, 60), (14, 3, 2, 3, 3, 56, 61),
                                                              (17, 18, 3, 6, 17, 50, 60),      # 544 tiles
                                                              # primes from 2^50 up: in one kernel from 2^15 on
                                                              (15, 4, 4, 1, 4, 52, 60), (15, 3, 2, 3, 3, 58, 61),
                                                              (16, 4, 2, 2, 3, 61, 62), (17, 18, 3, 6, 17, 58, 60)])
def test_tensor_product_within_the_first_transform_pass(logN, L, K, dnum, level, qbits, pbits):
    """Rows of either kind of prime, the ring whose tile is the whole transform, more tiles than go out wide; residues of q - 1
    among uniform ones, and a ciphertext times itself."""
    from paper_2604_09975_amd import binding as B
    O = helpers.small_oracle(logN, L=L, K=K, dnum=dnum, qbits=qbits, pbits=pbits)
    _, P = make_pair(O)
    r = W.rng(logN + L)
    top = np.array(O.q[:level], dtype=np.uint64)[:, None] - np.uint64(1)
    a, b = (np.where(r.integers(0, 5, x.shape) == 0, top, x) for x in W.uniform_residues(r, O.q[:level], O.N, lead=(2, 2)))
    rk = W.uniform_residues(r, O.moduli, O.N, lead=(dnum, 2))
    h = B.ckks_relin_key_load(P, to_dev(rk))
    for y in (b, a):
        da = to_dev(a)
        got = to_host(B.ckks_ctmul(P, da, da if y is a else to_dev(y), level, h))
        assert (got == O.ctmul(a, y, level, rk)).all()


def test_full_ring():
    O, P = make_pair(W.BIG_RING)
    from paper_2604_09975_amd import binding as B
    cl, za, zb, got = _case(O, P, 24, 90, 2.0**40, 64)
    out = to_host(B.ckks_rescale(P, to_dev(got[None]), 24, 1))[0]
    zz = cl.decrypt_slots(out, 23, 2.0**80 / O.q[23], nlimbs=2)
    assert np.abs(zz - za * zb).max() < 1e-5


def test_relin_keygen_bit_exact_and_errors():
    from paper_2604_09975_amd import binding as B
    O, P = make_pair(W.TOY_RING)
    r = W.rng(7)
    s = W.ternary_secret(r, O.N)
    S = B.ckks_client_secret_load(P, s)
    a = W.uniform_residues(r, O.moduli, O.N, lead=(O.dnum,))
    e = W.gaussian_error(r, (O.dnum, O.N))
    got = to_host(B.ckks_client_relin_keygen(P, S, to_dev(a), to_dev(e)))
    assert (got == O.relin_keygen(s, a, e)).all()
    ct = torch.zeros((2, 3, O.N), dtype=torch.int64, device="cuda")
    with pytest.raises(B.CkksError) as err:
        B.ckks_ctmul(P, ct, ct, 3, None)
    assert err.value.code == -3
    cl = helpers.Client(O, 8)
    gk = B.ckks_galois_key_load(P, O.galois_elt(1), to_dev(cl.galois_key(O.galois_elt(1))))
    with pytest.raises(B.CkksError) as err:
        B.ckks_ctmul(P, ct, ct, 3, gk)
    assert err.value.code == -1
    out = torch.zeros_like(ct)
    assert B.lib.ckks_ctmul(P.h, ct.data_ptr(), ct.data_ptr(), 4, gk.h, out.data_ptr(), None) == -2
    assert B.lib.ckks_ctmul(P.h, ct.data_ptr(), ct.data_ptr(), 0, gk.h, out.data_ptr(), None) == -2
