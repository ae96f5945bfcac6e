"""GPU parity: negacyclic NTT / INTT against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from tests import helpers
from tests.gpu_util import make_pair, to_dev, to_host
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


def _B():
    from paper_2604_09975_amd import binding as B
    return B


def test_roots_match_oracle():
    B = _B()
    for spec in (W.TOY_RING, W.BIG_RING):
        O, P = make_pair(spec)
        for limb in range(O.L + O.K):
            assert B.ckks_params_root(P, limb) == O.psi(limb)


@pytest.mark.parametrize("logN,batch", [(10, 3), (11, 2), (12, 5), (13, 3), (14, 2), (15, 1), (17, 1)])
def test_small_rings_bit_exact(logN, batch):
    """One-tile rings (N <= 4096) and two-pass rings up to the largest admitted degree (2^17), odd batch sizes,
    limbs listed out of order."""
    B = _B()
    O = helpers.small_oracle(logN, L=3, K=2, dnum=3, qbits=50, pbits=60)
    _, P = make_pair(O)
    ids = [4, 0, 2, 3, 1]
    r = W.rng(logN)
    x = W.uniform_residues(r, [O.moduli[i] for i in ids], O.N, lead=(batch,))
    x[0, :, :3] = 0
    x[0, :, 3] = np.array([O.moduli[i] - 1 for i in ids], dtype=np.uint64)
    d = to_dev(x)
    B.ckks_ntt(P, d, ids, batch)
    fwd = to_host(d)
    assert (fwd == O.ntt_batch(x, ids)).all()
    B.ckks_intt(P, d, ids, batch)
    assert (to_host(d) == x).all()
    d2 = to_dev(x)
    B.ckks_intt(P, d2, ids, batch)
    assert (to_host(d2) == O.ntt_batch(x, ids, inverse=True)).all()


@pytest.mark.parametrize("logN,ids,batch", [(12, [0], 512), (12, [0], 513), (12, [3], 512), (12, [3], 513),
                                            (12, [4, 1], 256), (12, [4, 1], 257), (13, [2, 4], 128), (13, [2, 4], 129)])
def test_either_side_of_the_wide_tiles(logN, ids, batch):
    """Up to 512 workgroups take a tile with 1024 threads, more with 256: rows of primes below 2^50, above, and both."""
    B = _B()
    O = helpers.small_oracle(logN, L=3, K=2, dnum=3, qbits=50, pbits=60)
    _, P = make_pair(O)
    x = W.uniform_residues(W.rng(batch), [O.moduli[i] for i in ids], O.N, lead=(batch,))
    x[-1] = np.array([O.moduli[i] - 1 for i in ids], dtype=np.uint64)[:, None]
    for inverse in (False, True):
        d = to_dev(x)
        (B.ckks_intt if inverse else B.ckks_ntt)(P, d, ids, batch)
        assert (to_host(d) == O.ntt_batch(x, ids, inverse=inverse)).all()


@pytest.mark.parametrize("logN,batch", [(12, 700), (14, 300), (14, 720)])
def test_many_rows_of_both_kinds(logN, batch):
    """More than 2048 workgroups of rows below and above 2^50 in one launch, cached and (the last, 270 MiB) streamed: the
    words that separate calls for the primes of each kind give, and the oracle's in the first and the last polynomial."""
    B = _B()
    O = helpers.small_oracle(logN, L=3, K=2, dnum=3, qbits=50, pbits=60)
    _, P = make_pair(O)
    ids = [4, 0, 1]
    x = W.uniform_residues(W.rng(batch), [O.moduli[i] for i in ids], O.N, lead=(batch,))
    for inverse in (False, True):
        f = B.ckks_intt if inverse else B.ckks_ntt
        d = to_dev(x)
        parts = [d[:, :1].clone(), d[:, 1:].clone()]
        f(P, d, ids, batch)
        for part, own in zip(parts, (ids[:1], ids[1:])):
            f(P, part, own, batch)
        assert torch.equal(d, torch.cat(parts, dim=1))
        ends = np.stack([x[0], x[-1]])
        assert (to_host(d[[0, batch - 1]]) == O.ntt_batch(ends, ids, inverse=inverse)).all()


def test_toy_ring_bit_exact():
    B = _B()
    O, P = make_pair(W.TOY_RING)
    ids = list(range(4))
    x = W.uniform_residues(W.rng(1), O.moduli, O.N, lead=(7,))
    d = to_dev(x)
    B.ckks_ntt(P, d, ids, 7)
    assert (to_host(d) == O.ntt_batch(x, ids)).all()


def test_full_size_batch_sampled_rows_and_roundtrip():
    """NTT microbench shape: 64 polynomials x 24 limbs x 2^16; the oracle checks a sample of rows
    bit for bit, the round trip checks every residue."""
    B = _B()
    O, P = make_pair(W.NTT_RING)
    ids = list(range(24))
    r = W.rng(W.NTT_SEED)
    x = W.uniform_residues(r, O.q, O.N, lead=(W.NTT_BATCH,))
    d = to_dev(x)
    B.ckks_ntt(P, d, ids, W.NTT_BATCH)
    fwd = to_host(d)
    pick = W.rng(99)
    rows = {(int(pick.integers(64)), int(pick.integers(24))) for _ in range(40)} | {(0, 0), (63, 23)}
    for b, i in rows:
        assert (fwd[b, i] == O.ntt(i, x[b, i])).all(), (b, i)
        assert (fwd[b, i] < np.uint64(O.q[i])).all()
    B.ckks_intt(P, d, ids, W.NTT_BATCH)
    assert (to_host(d) == x).all()
    # special primes of the full chain as well
    O2, P2 = make_pair(W.BIG_RING)
    ids2 = [24, 31, 0, 23]
    y = W.uniform_residues(r, [O2.moduli[i] for i in ids2], O2.N, lead=(3,))
    d = to_dev(y)
    B.ckks_ntt(P2, d, ids2, 3)
    assert (to_host(d) == O2.ntt_batch(y, ids2)).all()
    B.ckks_intt(P2, d, ids2, 3)
    assert (to_host(d) == y).all()


def test_ntt_argument_errors():
    B = _B()
    O, P = make_pair(W.TOY_RING)
    d = torch.zeros(O.N, dtype=torch.int64, device="cuda")
    with pytest.raises(B.CkksError) as e:
        B.ckks_ntt(P, d, [9], 1)
    assert e.value.code == -1
    with pytest.raises(ValueError):
        B.ckks_ntt(P, d, [0, 1], 1)
    B.ckks_ntt(P, d[:0], [0], 0)       # empty batch is a no-op
