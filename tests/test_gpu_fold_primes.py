"""GPU parity of the integer transforms at the edges of what their two butterflies take: primes 2^b - c fold at 2^b while c <
2^(b-35) and b <= 60, others are reduced by quotients."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import make_pair, to_dev, to_host
from tests.test_gpu_mid_rings import _edge_residues
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


def _is_prime(n):
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        x = pow(a, d, n)
        if x not in (1, n - 1) and all((x := x * x % n) != n - 1 for _ in range(s - 1)):
            return False
    return True


def _edge_primes(b, logN):
    """Two primes on either side of c = 2^(b-35) (where there are none below it: the first ones above)."""
    step, k0 = 2 << logN, (1 << (b - 35)) // (2 << logN)
    at = lambda ks: [p for p in ((1 << b) - k * step + 1 for k in ks) if _is_prime(p)]
    below, above = at(range(k0, max(0, k0 - 400), -1))[:2], at(range(k0 + 1, k0 + 400))[:2]
    assert all((1 << b) - p < 1 << (b - 35) for p in below) and all((1 << b) - p >= 1 << (b - 35) for p in above)
    return below + above


@pytest.mark.parametrize("logN,batch", [(12, 4), (12, 70), (13, 3), (14, 40), (15, 2), (16, 9), (17, 1)])
def test_transforms_either_side_of_the_fold(logN, batch):
    """Wide tiles and others, one to five stages per column: residues of zero and q - 1 in turn, in runs of every length the
    stages have, among uniform ones."""
    from paper_2604_09975_amd import binding as B
    p = [x for b in (51, 56, 60) for x in _edge_primes(b, logN)]
    O, P = make_pair(oracle.Oracle(logN, p[:len(p) // 2], p[len(p) // 2:], 1))
    ids = list(range(len(p)))
    x = _edge_residues(W.rng(logN), O.moduli, O.N, (batch,))
    top = np.array(O.moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    for row, run in zip(range(1, batch), (1 << logN, 1, 1 << (logN - 1), 64, 4096, 16, 2)):
        x[row] = top * np.uint64(1) * ((np.arange(O.N) // run + 1) % 2).astype(np.uint64)
    for inverse in (False, True):
        d = to_dev(x)
        (B.ckks_intt if inverse else B.ckks_ntt)(P, d, ids, batch)
        got, some = to_host(d), list(range(min(batch, 8)))
        assert (got[some] == O.ntt_batch(x[some], ids, inverse=inverse)).all()
        (B.ckks_ntt if inverse else B.ckks_intt)(P, d, ids, batch)
        assert (to_host(d) == x).all()


@pytest.mark.parametrize("logN,batch", [(12, 4), (12, 300), (13, 3), (14, 150), (15, 2), (16, 40), (17, 1), (17, 5)])
def test_transforms_of_rows_of_one_kind(logN, batch):
    """Rows none of which folds have a kernel of their own, rows that all fold share one with these: each kind alone, in few tiles
    (1024 threads), many and streamed, against the rows of a transform of both kinds in turn, and the first ones against the oracle."""
    from paper_2604_09975_amd import binding as B
    p = [x for b in (58, 60) for x in _edge_primes(b, logN)] + oracle.find_primes(61, logN, 2)
    O, P = make_pair(oracle.Oracle(logN, p[:len(p) // 2], p[len(p) // 2:], 1))
    folds = [i for i, q in enumerate(p) if q.bit_length() <= 60 and (1 << q.bit_length()) - q < 1 << (q.bit_length() - 35)]
    assert 2 <= len(folds) <= len(p) - 4
    x = _edge_residues(W.rng(70 + logN), O.moduli, O.N, (batch,))
    for inverse in (False, True):
        fn = B.ckks_intt if inverse else B.ckks_ntt
        both = to_dev(x)
        fn(P, both, list(range(len(p))), batch)
        both = to_host(both)
        assert (both[:2] == O.ntt_batch(x[:2], list(range(len(p))), inverse=inverse)).all()
        for ids in (folds, [i for i in range(len(p)) if i not in folds]):
            d = to_dev(x[:, ids])
            fn(P, d, ids, batch)
            assert (to_host(d) == both[:, ids]).all()


@pytest.mark.parametrize("logN,L,dnum,steps", [(12, 4, 2, 1), (13, 4, 1, 20), (14, 3, 3, 2), (15, 4, 2, 1), (16, 4, 2, 1)])
def test_key_switch_either_side_of_the_fold(logN, L, dnum, steps):
    """Special primes on both sides: one kernel then serves rows of either kind."""
    from paper_2604_09975_amd import binding as B
    sp = _edge_primes(60, logN)[:4] + _edge_primes(57, logN)[:2]
    O, P = make_pair(oracle.Oracle(logN, oracle.find_primes(50, logN, L), sp, dnum))
    r = W.rng(logN)
    ct, key = _edge_residues(r, O.q, O.N, (2,)), _edge_residues(r, O.moduli, O.N, (dnum, 2))
    h = B.ckks_galois_key_load(P, O.galois_elt(3), to_dev(key))
    got = to_host(B.ckks_rotate_hoisted(P, to_dev(ct), L, [3] * steps, [h] * steps))
    want = O.rotate_hoisted(ct, L, [O.galois_elt(3)], [key])[0]
    assert all((g == want).all() for g in got)
