"""GPU parity of the key switch with the column passes of the transforms inside the base conversions, on every ring these
kernels are instantiated for (N = 2^12 .. 2^16, 1 to 16 rows per column) and the ring above them: digit sizes and
special-prime counts at and off the powers of two their factor tables are padded to, partial last digits, more rows of
digits than one launch describes, special primes below and above 2^50."""
import numpy as np
import pytest

from tests import helpers
from tests.gpu_util import make_pair, to_dev, to_host
from tests.test_gpu_matmul import run_case
from tests.test_gpu_rotate import _run
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,L,K,dnum,level,pbits",
                         [(12, 3, 1, 3, 3, 60), (12, 10, 6, 2, 8, 60), (12, 8, 8, 1, 8, 60), (12, 6, 3, 2, 4, 49),
                          (13, 3, 1, 3, 2, 60), (13, 12, 4, 3, 11, 60), (13, 6, 3, 2, 5, 60), (13, 8, 8, 1, 7, 60),
                          (13, 12, 1, 12, 12, 60), (13, 9, 9, 1, 9, 59),
                          (14, 6, 2, 3, 5, 60), (14, 10, 5, 2, 9, 60), (14, 3, 1, 3, 3, 49), (14, 8, 7, 1, 8, 60),
                          (15, 12, 4, 3, 9, 60), (15, 2, 1, 2, 1, 60), (15, 4, 2, 2, 4, 60), (15, 7, 8, 1, 7, 60),
                          (16, 3, 1, 3, 3, 60), (16, 4, 2, 2, 3, 60), (16, 4, 4, 1, 4, 60),
                          (17, 4, 2, 2, 3, 60)])
def test_key_switch_shapes(logN, L, K, dnum, level, pbits):
    O = helpers.small_oracle(logN, L=L, K=K, dnum=dnum, qbits=50 if pbits > 50 else 45, pbits=pbits)
    _, P = make_pair(O)
    _run(O, P, level, [1, "conj"], 1000 * logN + 10 * L + level, 2.0**40, hw=16)


@pytest.mark.parametrize("logN,m,C,N1", [(12, 64, 8, 4), (13, 64, 8, 2), (14, 256, 8, 4), (15, 512, 4, 2)])
def test_projection_with_fused_rescale(logN, m, C, N1):
    """Merged giant step, ModDown and rescale in one pass (compared with the call without the flag and with the oracle)."""
    O = helpers.small_oracle(logN, L=4, K=2, dnum=2, qbits=50, pbits=60)
    _, P = make_pair(O)
    r = W.rng(logN)
    X, Wm = r.uniform(-1, 1, (m, C + 3)), r.uniform(-0.5, 0.5, (C + 3, 2 * C - 1))
    Y, ref, _, _ = run_case(O, P, X, Wm, r.uniform(-0.5, 0.5, 2 * C - 1), m, C, N1, 40, 4, 40 + logN, hw=16, real=True,
                            merged=True)
    assert np.abs(Y - ref).max() <= 1e-3


@pytest.mark.parametrize("logN,L,K,dnum,level,qbits,pbits,blocks,N1",
                         [(12, 6, 6, 3, 6, 50, 60, 27, 1), (12, 6, 6, 3, 5, 50, 60, 27, 1),     # 324 and 297 workgroups
                          (12, 8, 4, 2, 7, 45, 49, 30, 2), (12, 5, 6, 1, 5, 50, 60, 32, 4),     # special primes below 2^50; one digit
                          (13, 5, 2, 5, 5, 50, 60, 24, 2), (13, 4, 2, 2, 3, 52, 60, 33, 2),     # five digits; integer rows; two batches
                          (14, 6, 2, 3, 6, 50, 60, 10, 4), (17, 2, 2, 2, 2, 50, 60, 3, 4),
                          (15, 4, 8, 4, 4, 50, 60, 4, 4), (15, 4, 7, 4, 4, 50, 60, 4, 4),       # four digits of four: 384 and 352
                          (12, 6, 8, 3, 6, 52, 60, 32, 4), (12, 6, 8, 3, 6, 52, 60, 31, 4),     # three digits, integer rows: 448 and 434,
                          (13, 6, 8, 3, 6, 52, 60, 19, 4), (13, 6, 8, 3, 6, 52, 60, 23, 4),     # 532 and 644
                          (14, 8, 4, 4, 8, 52, 60, 16, 4), (14, 8, 4, 4, 8, 52, 60, 24, 4),     # four digits, integer rows: 768 and 1152
                          (12, 12, 1, 12, 12, 50, 60, 25, 4)])                                  # 156 rows of digits
def test_merged_giant_step_on_either_side_of_the_fused_tile_pass(logN, L, K, dnum, level, qbits, pbits, blocks, N1):
    """From 320 workgroups on the giant step's digits are transformed where their products are taken, with more than three
    digits of few ciphertexts from 384 on, with three and more on integer rows where rounds of 512 are 7/8 full and above 640
    (three digits) or 1152."""
    O = helpers.small_oracle(logN, L=L, K=K, dnum=dnum, qbits=qbits, pbits=pbits)
    _, P = make_pair(O)
    r = W.rng(logN + blocks)
    m, C = O.n // 8, 8
    Wm = r.uniform(-0.5, 0.5, (C, blocks * C))
    Y, ref, _, _ = run_case(O, P, r.uniform(-1, 1, (m, C)), Wm, None, m, C, N1, 40, level, 50 + logN, hw=16, merged=True,
                            oracle_blocks=[0, blocks // 2, blocks - 1])
    assert np.abs(Y - ref).max() <= 1e-3


def test_rotation_of_a_ciphertext_that_is_not_16_byte_aligned():
    """The switches gather pairs of residues from the caller's ciphertext; its address need only be that of a word."""
    import torch
    from paper_2604_09975_amd import binding as B
    O = helpers.small_oracle(13, L=4, K=2, dnum=2, qbits=50, pbits=60)
    _, P = make_pair(O)
    r = W.rng(77)
    buf = torch.empty(2 * 4 * O.N + 1, dtype=torch.int64, device="cuda")
    ct = torch.from_numpy(W.uniform_residues(r, O.q, O.N, lead=(2,)).view(np.int64)).cuda()
    key = torch.from_numpy(W.uniform_residues(r, O.moduli, O.N, lead=(O.dnum, 2)).view(np.int64)).cuda()
    h = B.ckks_galois_key_load(P, O.galois_elt(5), key)
    odd = buf[1:].view(2, 4, O.N)
    odd.copy_(ct)
    assert odd.data_ptr() % 16 == 8
    assert torch.equal(B.ckks_rotate_hoisted(P, odd, 4, [5], [h]), B.ckks_rotate_hoisted(P, ct, 4, [5], [h]))


@pytest.mark.parametrize("steps", [[5], [5] * 32, [5, 9] * 16])
def test_rotations_by_either_gather(steps):
    """Few workgroups gather digits residue by residue, many by pairs, whose loads must not need more than a word's alignment:
    32 switches at 2^15 with six special primes are above the lines between the two in both kernels, one is below; keys
    shared by neighbours and not."""
    import torch
    from paper_2604_09975_amd import binding as B
    O = helpers.small_oracle(15, L=6, K=6, dnum=1, qbits=50, pbits=60)
    _, P = make_pair(O)
    r = W.rng(78)
    ct = W.uniform_residues(r, O.q, O.N, lead=(2,))
    keys = {s: W.uniform_residues(r, O.moduli, O.N, lead=(O.dnum, 2)) for s in set(steps)}
    h = {s: B.ckks_galois_key_load(P, O.galois_elt(s), torch.from_numpy(k.view(np.int64)).cuda()) for s, k in keys.items()}
    buf = torch.empty(2 * 6 * O.N + 1, dtype=torch.int64, device="cuda")
    odd = buf[1:].view(2, 6, O.N)
    odd.copy_(torch.from_numpy(ct.view(np.int64)))
    got = B.ckks_rotate_hoisted(P, odd, 6, steps, [h[s] for s in steps])
    for s in set(steps):
        want = torch.from_numpy(O.rotate_hoisted(ct, 6, [O.galois_elt(s)], [keys[s]])[0].view(np.int64)).cuda()
        for i in range(len(steps)):
            assert steps[i] != s or torch.equal(got[i], want), i


@pytest.mark.parametrize("logN,L,K,dnum,level,pbits", [(13, 8, 8, 1, 8, 60), (13, 3, 1, 3, 1, 60), (13, 12, 4, 3, 11, 49), (14, 8, 5, 1, 7, 55),
                                                       (14, 9, 2, 9, 5, 60), (15, 8, 4, 2, 8, 49), (15, 7, 7, 1, 7, 61),
                                                       (16, 6, 6, 1, 6, 49), (16, 4, 3, 2, 3, 60), (16, 12, 2, 6, 9, 60)])
def test_target_groups_of_a_lone_switch(logN, L, K, dnum, level, pbits):
    """Conversions of few workgroups take small groups of targets, down to one and with a shorter last one, of digits whose targets
    are not all as many; twenty switches of the same rotation take groups of eight."""
    from paper_2604_09975_amd import binding as B
    O = helpers.small_oracle(logN, L=L, K=K, dnum=dnum, qbits=50 if pbits > 50 else 45, pbits=pbits)
    _, P = make_pair(O)
    r = W.rng(1500 + logN + L)
    ct, key = _edge_residues(r, O.q[:level], O.N, (2,)), _edge_residues(r, O.moduli, O.N, (O.dnum, 2))
    h = B.ckks_galois_key_load(P, O.galois_elt(3), to_dev(key))
    one = to_host(B.ckks_rotate_hoisted(P, to_dev(ct), level, [3], [h]))[0]
    assert (one == O.rotate_hoisted(ct, level, [O.galois_elt(3)], [key])[0]).all()
    many = to_host(B.ckks_rotate_hoisted(P, to_dev(ct), level, [3] * 20, [h] * 20))
    assert all((g == one).all() for g in many)


@pytest.mark.parametrize("logN,level", [(12, 11), (13, 12), (16, 12)])
def test_more_digit_rows_than_one_launch_describes(logN, level):
    """Twelve digits of one limb: 132 rows and more of extended digits, above the 128 of one row map; the forward tile passes go
    out digit by digit."""
    O = helpers.small_oracle(logN, L=12, K=1, dnum=12, qbits=50, pbits=60)
    _, P = make_pair(O)
    _run(O, P, level, [3], 1300 + logN, 2.0**40, hw=16)


def _edge_residues(r, moduli, N, lead):
    """Uniform residues, one in five q - 1."""
    x = W.uniform_residues(r, moduli, N, lead=lead)
    top = np.array(moduli, dtype=np.uint64)[:, None] - np.uint64(1)
    return np.where(r.integers(0, 5, x.shape) == 0, top, x)


def _large_primes(logN, L, K, qbits, pbits):
    import oracle
    p = oracle.find_primes(pbits, logN, K + (L if pbits == qbits else 0))
    return (p[K:] if pbits == qbits else oracle.find_primes(qbits, logN, L)), p[:K]


@pytest.mark.parametrize("logN,L,K,dnum,level,qbits,pbits,steps", [(12, 4, 2, 4, 4, 50, 62, 2), (12, 4, 4, 4, 4, 62, 62, 3),
                                                                   (13, 8, 4, 4, 8, 61, 62, 2), (13, 4, 4, 1, 4, 62, 61, 1),
                                                                   (14, 4, 4, 4, 4, 62, 62, 20), (16, 4, 2, 4, 3, 50, 61, 2)])
def test_key_switch_at_the_largest_primes(logN, L, K, dnum, level, qbits, pbits, steps):
    """Four digits on primes next to 2^62, where the key inner product's four products of residues leave the reduction the least
    room (4 q^2 < q 2^64): residues of q - 1 among uniform ones, and a ciphertext whose every residue is q - 1 under keys whose
    every residue is; a launch of wide tiles, and one above them (20 switches at 2^14)."""
    import oracle
    from paper_2604_09975_amd import binding as B
    O, P = make_pair(oracle.Oracle(logN, *_large_primes(logN, L, K, qbits, pbits), dnum))
    r = W.rng(100 * logN + pbits)
    st = [3, 5, 7][:steps] if steps < 4 else [3] * steps
    cts = [_edge_residues(r, O.q[:level], O.N, (2,)), np.empty((2, level, O.N), dtype=np.uint64)]
    keys = [{s: _edge_residues(r, O.moduli, O.N, (dnum, 2)) for s in set(st)}, {}]
    cts[1][:] = np.array(O.q[:level], dtype=np.uint64)[:, None] - np.uint64(1)
    for s in set(st):
        keys[1][s] = np.broadcast_to(np.array(O.moduli, dtype=np.uint64)[:, None] - np.uint64(1), keys[0][s].shape).copy()
    for ct, ks in zip(cts, keys):
        h = {s: B.ckks_galois_key_load(P, O.galois_elt(s), to_dev(k)) for s, k in ks.items()}
        got = to_host(B.ckks_rotate_hoisted(P, to_dev(ct), level, st, [h[s] for s in st]))
        for s in set(st):
            want = O.rotate_hoisted(ct, level, [O.galois_elt(s)], [ks[s]])[0]
            for i in range(len(st)):
                assert st[i] != s or (got[i] == want).all(), i


@pytest.mark.parametrize("logN,L,K,dnum,qbits,pbits,blocks,pair", [(13, 4, 4, 4, 50, 62, 20, False), (13, 4, 4, 4, 62, 62, 28, False),
                                                                   (14, 6, 2, 3, 50, 60, 10, True), (15, 4, 2, 2, 50, 60, 7, True)])
def test_merged_projection_of_uniform_residues(logN, L, K, dnum, qbits, pbits, blocks, pair):
    """The fused tile pass of the giant step (320 workgroups and more) at the largest primes, whose transform values reach 2^64
    where it multiplies them, with residues of q - 1 among the inputs and keys; and in a layer of complex-packed pairs."""
    import oracle
    from paper_2604_09975_amd import binding as B
    O, P = make_pair(oracle.Oracle(logN, *_large_primes(logN, L, K, qbits, pbits), dnum))
    r = W.rng(logN + blocks)
    m, C, N1, G = O.n // 8, 8, 2, 1
    N2 = C // N1
    diag = r.integers(-1 << 40, 1 << 40, (blocks, N2, G, N1, O.N))
    x = _edge_residues(r, O.q, O.N, (G, 2))
    steps = [q * m for q in range(1, N1)], [p * N1 * m for p in range(1, N2)], ["conj"] if pair else []
    keys = [[_edge_residues(r, O.moduli, O.N, (dnum, 2)) for _ in s] for s in steps]
    baby, giant, conj = [[B.ckks_galois_key_load(P, O.galois_elt(s), to_dev(k)) for s, k in zip(ss, kk)]
                         for ss, kk in zip(steps, keys)]
    w = B.ckks_weights_create(P, L, m, C, G, blocks, N1)
    B.ckks_weights_set_diagonals(w, 0, to_dev(diag.reshape(-1, O.N)))
    y, _ = B.ckks_ctpt_matmul(P, w, to_dev(x), baby, giant, conj_key=conj[0] if pair else None, flags=B.MATMUL_MERGED_GIANT)
    got = to_host(y)
    for b in (0, blocks // 2, blocks - 1):
        want = O.ctpt_matmul(L, m, G, blocks, N1, N2, diag, None, 0, x, keys[0], keys[1], b_first=b, b_count=1,
                             conj_key=keys[2][0] if pair else None, merged=True)
        assert (got[b] == want[b]).all(), b
