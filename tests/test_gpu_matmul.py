"""GPU parity: the ct-pt projection Y = XW (+ bias) and rescale against the oracle, bit for bit,
and the decrypted result against the fp64 product."""
import numpy as np
import pytest
import torch

from oracle import encoding as E
from tests import helpers
from tests.gpu_util import load_keys, make_pair, to_dev, to_host
from paper_2604_09975_amd import workload as W

pytestmark = pytest.mark.gpu


def _B():
    from paper_2604_09975_amd import binding as B
    return B


def make_real(m):
    """Force c[N-j] = -c[j] (and c[N/2] = 0) on encoded coefficient arrays: the exact form of a plaintext
    with real slots.  The library recognises such diagonals and reads half of each weight limb."""
    N = m.shape[-1]
    m = m.copy()
    m[..., N // 2 + 1:] = -m[..., 1:N // 2][..., ::-1]
    m[..., N // 2] = 0
    return m


def run_case(O, P, X, Wm, bias, m, C, N1, log_scale, level, seed, hw=64, oracle_blocks=None, real=False,
             merged=False):
    """Runs the projection on both sides from identical integer inputs; returns everything."""
    B = _B()
    N, n = O.N, O.n
    sx = sw = 2.0**log_scale
    d_in, d_out = Wm.shape
    G, B_out, N2 = -(-d_in // C), -(-d_out // C), C // N1
    cl = helpers.Client(O, seed, hamming_weight=hw)
    mx = E.encode(E.pack_columns(X, n, C) + 0j, sx, N)
    ct_x = np.stack([cl.encrypt_coeffs(mx[g], level) for g in range(G)])
    diag = E.encode_diagonals(Wm, m, N, C, N1, sw)
    if real == "first_upload":                     # real diagonals first, general ones later in the same block
        flat = diag.reshape(-1, N)
        flat[:max(1, flat.shape[0] // 2)] = make_real(flat[:max(1, flat.shape[0] // 2)])
    elif real:
        diag = make_real(diag)
    bias_c = None
    if bias is not None:
        bias_c = np.stack([E.encode(E.bias_slots(bias, m, n, C, b) + 0j, sx, N) for b in range(B_out)])
    baby_np, baby_h = load_keys(P, O, cl, [q * m for q in range(1, N1)])
    giant_np, giant_h = load_keys(P, O, cl, [p * N1 * m for p in range(1, N2)])

    w = B.ckks_weights_create(P, level, m, C, G, B_out, N1)
    flat = diag.reshape(-1, N)
    half = max(1, flat.shape[0] // 2)                 # two uploads: exercises the `first` offset
    B.ckks_weights_set_diagonals(w, 0, to_dev(flat[:half]))
    if flat.shape[0] > half:
        B.ckks_weights_set_diagonals(w, half, to_dev(flat[half:]))
    if bias_c is not None:
        B.ckks_weights_set_bias(w, to_dev(bias_c), int(sw))
    y_dev, cnt = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h,
                                    flags=B.MATMUL_MERGED_GIANT if merged else 0)
    y_res = B.ckks_rescale(P, y_dev, level, B_out)
    # the same projection with the rescale inside the call: identical residues
    y_fused, _ = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h,
                                    flags=(B.MATMUL_MERGED_GIANT if merged else 0) | B.MATMUL_RESCALE)
    torch.cuda.synchronize()
    assert torch.equal(y_fused, y_res)
    got, got_res = to_host(y_dev), to_host(y_res)

    blocks = list(range(B_out)) if oracle_blocks is None else oracle_blocks
    for b in blocks:
        want = O.ctpt_matmul(level, m, G, B_out, N1, N2, diag, bias_c, int(sw), ct_x, baby_np, giant_np,
                             b_first=b, b_count=1, merged=merged)
        assert (got[b] == want[b]).all(), f"block {b}"
        assert (got_res[b] == O.rescale(want[b:b + 1], level)[0]).all(), f"rescaled block {b}"
    assert cnt.key_switches == sum(1 for k in baby_np if k is not None) * G + sum(1 for k in giant_np if k is not None) * B_out
    assert cnt.ptmuls == G * N1 * B_out * N2
    scale = sx * sw / O.q[level - 1]
    slots = np.stack([cl.decrypt_slots(got_res[b], level - 1, scale, nlimbs=min(level - 1, 2)) for b in range(B_out)])
    Y = E.unpack_columns(slots.real, m, C, d_out)
    ref = X @ Wm + (bias if bias is not None else 0.0)
    return Y, ref, cnt, slots


def test_toy_config():
    """N = 2^12, scale 2^30, 16x64 times 64x64, the 64 rotations of the plain diagonal method, one rescale."""
    O, P = make_pair(W.TOY_RING)
    spec = W.TOY_MATMUL
    X, Wm, _ = W.matmul_inputs(spec)
    Y, ref, cnt, _ = run_case(O, P, X, Wm, None, spec.m, spec.C, spec.N1, 30, 3, spec.seed)
    assert np.abs(Y - ref).max() <= 1e-3
    assert cnt.key_switches == 63


@pytest.mark.parametrize("N1,qbits,pbits", [(1, 40, 42), (4, 40, 42), (16, 40, 42), (4, 52, 55), (2, 50, 60)])
def test_bsgs_bias_ragged_shapes(N1, qbits, pbits):
    """n = 512 slots, m = 4, C = 16 (eight periods of the active columns), d_in = 40 (ragged last group),
    d_out = 20 (ragged last block), bias, every split of the 16 diagonals; primes below 2^50 (fp64
    arithmetic inside the library) and above (Montgomery arithmetic)."""
    O = helpers.small_oracle(10, L=3, K=1, dnum=3, qbits=qbits, pbits=pbits)
    _, P = make_pair(O)
    r = W.rng(9)
    X = r.uniform(-1, 1, (4, 40))
    Wm = r.uniform(-0.5, 0.5, (40, 20))
    bias = r.uniform(-0.5, 0.5, 20)
    Y, ref, cnt, slots = run_case(O, P, X, Wm, bias, 4, 16, N1, qbits - 10, 3, 19, hw=16)
    assert np.abs(Y - ref).max() <= 1e-3
    assert np.abs(slots.imag).max() <= 1e-3
    assert cnt.key_switches == 3 * (N1 - 1) + 2 * (16 // N1 - 1)


def test_real_plaintexts_on_a_chain_with_small_and_large_primes():
    """One 52-bit prime (Montgomery arithmetic) and two 40-bit primes (fp64 arithmetic, palindrome kernel on
    unpacked weights): the packed store needs every prime below 2^50, so this chain keeps the full one."""
    import oracle
    q = oracle.find_primes(52, 11, 1) + oracle.find_primes(40, 11, 2)
    O = oracle.Oracle(11, q, oracle.find_primes(55, 11, 1), 3)
    _, P = make_pair(O)
    r = W.rng(31)
    X = r.uniform(-1, 1, (4, 40))
    Wm = r.uniform(-0.5, 0.5, (40, 20))
    Y, ref, _, _ = run_case(O, P, X, Wm, r.uniform(-0.5, 0.5, 20), 4, 16, 4, 35, 3, 32, hw=16, real=True)
    assert np.abs(Y - ref).max() <= 1e-3


def test_block_turns_general_after_real_diagonals_were_stored():
    """One output block loaded in two uploads, the first all real (stored in the packed half-limb form), the
    second not: the block's diagonals move to the full store and the general kernel runs."""
    O, P = make_pair(W.TOY_RING)
    r = W.rng(77)
    X = r.uniform(-1, 1, (16, 100))
    Wm = r.uniform(-0.2, 0.2, (100, 64))
    Y, ref, _, _ = run_case(O, P, X, Wm, None, 16, 64, 8, 30, 3, 78, real="first_upload")
    assert np.abs(Y - ref).max() <= 2e-3


@pytest.mark.parametrize("N1", [1, 4])
def test_real_plaintexts_use_the_palindrome_path(N1):
    """Diagonals with exactly antisymmetric coefficients (real slots): only half of each weight limb is read.
    n = 2048 slots (one run of coefficients per workgroup row), ragged shapes, bias."""
    O, P = make_pair(W.TOY_RING)
    r = W.rng(21)
    X = r.uniform(-1, 1, (16, 100))
    Wm = r.uniform(-0.1, 0.1, (100, 70))
    bias = r.uniform(-0.5, 0.5, 70)
    Y, ref, cnt, slots = run_case(O, P, X, Wm, bias, 16, 64, N1 * 16, 30, 3, 23, real=True)
    assert np.abs(Y - ref).max() <= 1e-3


def test_one_unsymmetric_diagonal_turns_the_palindrome_path_off():
    B = _B()
    O, P = make_pair(W.TOY_RING)
    r = W.rng(22)
    X = r.uniform(-1, 1, (16, 64))
    Wm = r.uniform(-0.1, 0.1, (64, 64))
    Y, ref, cnt, _ = run_case(O, P, X, Wm, None, 16, 64, 16, 30, 3, 25, real=False)
    assert np.abs(Y - ref).max() <= 1e-3


@pytest.mark.parametrize("ring,N1", [("toy", 16), ("toy", 4), ("small", 2), ("small", 16)])
def test_merged_giant_step(ring, N1):
    """CKKS_MATMUL_MERGED_GIANT: one ModDown per output block for the whole giant step, bit for bit against the
    oracle's merged variant (N1 = C: no giant step, the flag changes nothing)."""
    if ring == "toy":
        O, P = make_pair(W.TOY_RING)
        m, C, hw = 16, 64, 64
    else:
        O = helpers.small_oracle(10, L=4, K=2, dnum=2, qbits=40, pbits=45)
        _, P = make_pair(O)
        m, C, hw = 4, 16, 16
    r = W.rng(61)
    X = r.uniform(-1, 1, (m, 2 * C + 3))
    Wm = r.uniform(-0.1, 0.1, (2 * C + 3, C + 5))
    bias = r.uniform(-0.5, 0.5, C + 5)
    Y, ref, cnt, _ = run_case(O, P, X, Wm, bias, m, C, N1, 30, O.L, 63, hw=hw, merged=True, real=(ring == "toy"))
    assert np.abs(Y - ref).max() <= 1e-3
    assert cnt.key_switches == 3 * (N1 - 1) + 2 * (C // N1 - 1)


@pytest.mark.parametrize("merged", [False, True])
def test_more_blocks_than_one_switch_batch(merged):
    """B_out = 36 output blocks: the giant step runs in more than one batch of (32) key switches."""
    O = helpers.small_oracle(10, L=2, K=1, dnum=2, qbits=40, pbits=42)
    _, P = make_pair(O)
    r = W.rng(10)
    X = r.uniform(-1, 1, (64, 8))
    Wm = r.uniform(-0.5, 0.5, (8, 288))
    Y, ref, cnt, _ = run_case(O, P, X, Wm, None, 64, 8, 4, 30, 2, 29, hw=16, merged=merged)
    assert np.abs(Y - ref).max() <= 1e-3


def test_rescale_alone_bit_exact_and_errors():
    B = _B()
    O, P = make_pair(W.BIG_RING)
    r = W.rng(4)
    for level, n_ct in ((24, 2), (2, 1), (7, 3)):
        ct = W.uniform_residues(r, O.q[:level], O.N, lead=(n_ct, 2))
        got = to_host(B.ckks_rescale(P, to_dev(ct), level, n_ct))
        assert (got == O.rescale(ct, level)).all()
    d = torch.zeros((1, 2, 1, O.N), dtype=torch.int64, device="cuda")
    with pytest.raises(B.CkksError) as e:
        B.ckks_rescale(P, d, 1, 1)
    assert e.value.code == -2
    assert B.lib.ckks_rescale(P.h, d.data_ptr(), 25, 1, d.data_ptr(), None) == -2


def test_matmul_errors():
    B = _B()
    O, P = make_pair(W.TOY_RING)
    with pytest.raises(B.CkksError) as e:
        B.ckks_weights_create(P, 3, 16, 48, 1, 1, 16)          # C does not divide the 128 segments
    assert e.value.code == -1
    with pytest.raises(B.CkksError) as e:
        B.ckks_weights_create(P, 4, 16, 64, 1, 1, 64)          # level > L
    assert e.value.code == -2
    w = B.ckks_weights_create(P, 3, 16, 64, 1, 1, 32)
    with pytest.raises(B.CkksError) as e:
        B.ckks_weights_set_diagonals(w, 60, torch.zeros((8, O.N), dtype=torch.int64, device="cuda"))
    assert e.value.code == -1
    x = torch.zeros((1, 2, 3, O.N), dtype=torch.int64, device="cuda")
    with pytest.raises(B.CkksError) as e:
        B.ckks_ctpt_matmul(P, w, x, [None] * 31, [None])
    assert e.value.code == -3


@pytest.mark.parametrize("d_in,spec,real_tail", [(40, "small", False), (100, "toy", False), (40, "small", True),
                                                 (170, "toy", True)])
def test_complex_pair_compression_with_decomplexification(d_in, spec, real_tail):
    """Complexified inputs x^(2u) + i x^(2u+1), complex weights (times 1/2), y + conj(y) per output block:
    residues bit for bit against the oracle, decrypted result against X @ W + b.
    real_tail: an odd number of real groups, so the last complexified input has imaginary part zero and its
    weights real slots; with exactly antisymmetric encodings the library keeps that group as half records and sums
    it in a second launch onto the accumulators of the complex groups."""
    B = _B()
    if spec == "small":
        O = helpers.small_oracle(10, L=3, K=1, dnum=3, qbits=40, pbits=42)
        _, P = make_pair(O)
        m, C, N1, d_out, hw = 4, 16, 4, 20, 16
    else:
        O, P = make_pair(W.TOY_RING)
        m, C, N1, d_out, hw = 16, 64, 16, 70, 64
    N, n, level = O.N, O.n, 3
    r = W.rng(d_in)
    X = r.uniform(-1, 1, (m, d_in))
    Wm = r.uniform(-0.1, 0.1, (d_in, d_out))
    bias = r.uniform(-0.5, 0.5, d_out)
    G, B_out, N2 = -(-d_in // C), -(-d_out // C), C // N1
    U = -(-G // 2)
    cl = helpers.Client(O, 41, hamming_weight=hw)
    sc = 2.0**30
    mx = E.encode(E.pack_columns_complex(X, n, C), sc, N)
    ct_x = np.stack([cl.encrypt_coeffs(mx[u], level) for u in range(U)])
    diag = E.encode_diagonals_complex(Wm, m, N, C, N1, sc, half=True)
    if real_tail:
        assert G % 2 == 1 and U >= 2
        diag[:, :, U - 1] = make_real(diag[:, :, U - 1])
    bias_c = np.stack([E.encode(E.bias_slots(bias, m, n, C, b) + 0j, sc, N) for b in range(B_out)])
    baby_np, baby_h = load_keys(P, O, cl, [q * m for q in range(1, N1)])
    giant_np, giant_h = load_keys(P, O, cl, [p * N1 * m for p in range(1, N2)])
    (conj_np,), (conj_h,) = load_keys(P, O, cl, ["conj"])
    w = B.ckks_weights_create(P, level, m, C, U, B_out, N1)
    B.ckks_weights_set_diagonals(w, 0, to_dev(diag.reshape(-1, N)))
    B.ckks_weights_set_bias(w, to_dev(bias_c), int(sc))
    y_dev, cnt = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h, conj_key=conj_h)
    y_res = B.ckks_rescale(P, y_dev, level, B_out)
    torch.cuda.synchronize()
    want = O.ctpt_matmul(level, m, U, B_out, N1, N2, diag, bias_c, int(sc), ct_x, baby_np, giant_np, conj_key=conj_np)
    assert (to_host(y_dev) == want).all()
    assert (to_host(y_res) == O.rescale(want, level)).all()
    assert cnt.key_switches == U * (N1 - 1) + B_out * (N2 - 1) + B_out
    got = to_host(y_res)
    slots = np.stack([cl.decrypt_slots(got[b], 2, sc * sc / O.q[2], nlimbs=2) for b in range(B_out)])
    assert np.abs(E.unpack_columns(slots.real, m, C, d_out) - (X @ Wm + bias)).max() <= 1e-3
    assert np.abs(slots.imag).max() <= 1e-3
    # the order Sec. 3.2 displays: the real part of every giant-step accumulator before the fold (N2 conjugations
    # per block), with either giant-step order after it; other residues, the same values
    for merged in (False, True):
        fl = B.MATMUL_CONJ_PER_ACC | (B.MATMUL_MERGED_GIANT if merged else 0)
        y2, cnt2 = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h, conj_key=conj_h, flags=fl)
        y2r, _ = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h, conj_key=conj_h, flags=fl | B.MATMUL_RESCALE)
        torch.cuda.synchronize()
        want2 = O.ctpt_matmul(level, m, U, B_out, N1, N2, diag, bias_c, int(sc), ct_x, baby_np, giant_np,
                              conj_key=conj_np, merged=merged, conj_per_acc=True)
        assert not (want2 == want).all()
        assert (to_host(y2) == want2).all()
        assert (to_host(y2r) == O.rescale(want2, level)).all()
        assert cnt2.key_switches == U * (N1 - 1) + B_out * (N2 - 1) + B_out * N2
        got2 = to_host(y2r)
        slots2 = np.stack([cl.decrypt_slots(got2[b], 2, sc * sc / O.q[2], nlimbs=2) for b in range(B_out)])
        assert np.abs(E.unpack_columns(slots2.real, m, C, d_out) - (X @ Wm + bias)).max() <= 1e-3
    with pytest.raises(B.CkksError) as e:
        B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h, flags=B.MATMUL_CONJ_PER_ACC)
    assert e.value.code == -3                  # CKKS_E_NOKEY: the flag without a conjugation key


def test_fused_qk_projection():
    """Weights W_Q + i W_K on a real-packed input: one projection, Q in the real and K in the imaginary parts."""
    B = _B()
    O, P = make_pair(W.TOY_RING)
    m, C, N1, level = 16, 64, 16, 3
    N, n = O.N, O.n
    r = W.rng(55)
    X = r.uniform(-1, 1, (m, 128))
    WQ, WK = r.uniform(-0.1, 0.1, (128, 64)), r.uniform(-0.1, 0.1, (128, 64))
    G, B_out, N2 = 2, 1, C // N1
    cl = helpers.Client(O, 43)
    sc = 2.0**30
    mx = E.encode(E.pack_columns(X, n, C) + 0j, sc, N)
    ct_x = np.stack([cl.encrypt_coeffs(mx[g], level) for g in range(G)])
    diag = E.encode_diagonals_fused(WQ, WK, m, N, C, N1, sc)
    baby_np, baby_h = load_keys(P, O, cl, [q * m for q in range(1, N1)])
    giant_np, giant_h = load_keys(P, O, cl, [p * N1 * m for p in range(1, N2)])
    w = B.ckks_weights_create(P, level, m, C, G, B_out, N1)
    B.ckks_weights_set_diagonals(w, 0, to_dev(diag.reshape(-1, N)))
    y_dev, _ = B.ckks_ctpt_matmul(P, w, to_dev(ct_x), baby_h, giant_h)
    y_res = to_host(B.ckks_rescale(P, y_dev, level, B_out))
    want = O.ctpt_matmul(level, m, G, B_out, N1, N2, diag, None, 0, ct_x, baby_np, giant_np)
    assert (to_host(y_dev) == want).all()
    slots = cl.decrypt_slots(y_res[0], 2, sc * sc / O.q[2], nlimbs=2)[None]
    assert np.abs(E.unpack_columns(slots.real, m, C, 64) - X @ WQ).max() <= 1e-3
    assert np.abs(E.unpack_columns(slots.imag, m, C, 64) - X @ WK).max() <= 1e-3


def test_conj_key_must_be_a_conjugation_key():
    B = _B()
    O, P = make_pair(W.TOY_RING)
    cl = helpers.Client(O, 44)
    _, (k1,) = load_keys(P, O, cl, [1])
    w = B.ckks_weights_create(P, 3, 16, 64, 1, 1, 1)
    x = torch.zeros((1, 2, 3, O.N), dtype=torch.int64, device="cuda")
    _, giant = load_keys(P, O, cl, [p * 16 for p in range(1, 64)])
    with pytest.raises(B.CkksError) as e:
        B.ckks_ctpt_matmul(P, w, x, [], giant, conj_key=k1)
    assert e.value.code == -1


def test_weights_load_in_one_call_equals_streamed_upload():
    """ckks_weights_load = create + set_diagonals (in pieces) + set_bias: same output ciphertexts, bit for bit."""
    B = _B()
    O = helpers.small_oracle(10, L=3, K=1, dnum=3, qbits=40, pbits=42)
    _, P = make_pair(O)
    r = W.rng(77)
    m, C, N1, level = 4, 16, 4, 3
    X, Wm, bias = r.uniform(-1, 1, (m, 40)), r.uniform(-0.5, 0.5, (40, 20)), r.uniform(-0.5, 0.5, 20)
    G, B_out, N2 = 3, 2, C // N1
    sc = 2.0**30
    cl = helpers.Client(O, 78, hamming_weight=16)
    mx = E.encode(E.pack_columns(X, O.n, C) + 0j, sc, O.N)
    ct_x = to_dev(np.stack([cl.encrypt_coeffs(mx[g], level) for g in range(G)]))
    diag = to_dev(E.encode_diagonals(Wm, m, O.N, C, N1, sc).reshape(-1, O.N))
    bias_c = to_dev(np.stack([E.encode(E.bias_slots(bias, m, O.n, C, b) + 0j, sc, O.N) for b in range(B_out)]))
    _, baby = load_keys(P, O, cl, [q * m for q in range(1, N1)])
    _, giant = load_keys(P, O, cl, [p * N1 * m for p in range(1, N2)])
    w1 = B.ckks_weights_create(P, level, m, C, G, B_out, N1)
    B.ckks_weights_set_diagonals(w1, 0, diag)
    B.ckks_weights_set_bias(w1, bias_c, int(sc))
    w2 = B.ckks_weights_load(P, level, m, C, G, B_out, N1, diag, bias_c, int(sc))
    y1, _ = B.ckks_ctpt_matmul(P, w1, ct_x, baby, giant)
    y2, _ = B.ckks_ctpt_matmul(P, w2, ct_x, baby, giant)
    assert bool((y1 == y2).all())
    w3 = B.ckks_weights_load(P, level, m, C, G, B_out, N1, diag)            # no bias
    y3, _ = B.ckks_ctpt_matmul(P, w3, ct_x, baby, giant)
    assert not bool((y3 == y1).all())
    with pytest.raises(ValueError):
        B.ckks_weights_load(P, level, m, C, G, B_out, N1, diag[:-1])
    with pytest.raises(B.CkksError):
        B.ckks_weights_load(P, level + 1, m, C, G, B_out, N1, diag)
    assert B.lib.ckks_weights_load(P.h, level, m, C, G, B_out, N1, None, None, 0, None, None) == -1


@pytest.mark.parametrize("N1,merged", [(4, False), (8, True)])
def test_ring_2_13_xcd_unfolded_tile_order(N1, merged):
    """N = 2^13 is the smallest ring whose coefficient runs divide over the 8 XCDs, which switches the
    multiply-accumulate kernels to their unfolded workgroup order (the one every N = 2^16 launch uses).  Real
    diagonals on a sub-2^50 chain (packed half records), 10 output blocks: N1 = 4 gives 40 (b,p) pairs, five full
    tiles; N1 = 8 gives 20, two full tiles and a ragged one.  Every residue of every block against the oracle."""
    O = helpers.small_oracle(13, L=3, K=1, dnum=3, qbits=45, pbits=50)
    _, P = make_pair(O)
    r = W.rng(1313)
    X = r.uniform(-1, 1, (8, 40))
    Wm = r.uniform(-0.5, 0.5, (40, 150))
    bias = r.uniform(-0.5, 0.5, 150)
    Y, ref, cnt, slots = run_case(O, P, X, Wm, bias, 8, 16, N1, 35, 3, 77, hw=16, real=True, merged=merged)
    assert np.abs(Y - ref).max() <= 1e-3
    assert np.abs(slots.imag).max() <= 1e-3


def test_argument_checks_enqueue_nothing():
    """A weight set with diagonals missing, unknown flag bits and an output that overlaps the input are refused
    with CKKS_E_INVAL before anything is enqueued; so are overlapping buffers of rescale and the hoisted rotation."""
    B = _B()
    O = helpers.small_oracle(10, L=3, K=1, dnum=3, qbits=40, pbits=42)
    _, P = make_pair(O)
    N, level, m, C, N1 = O.N, 3, 4, 16, 4
    w = B.ckks_weights_create(P, level, m, C, 1, 1, N1)
    x = torch.zeros((1, 2, level, N), dtype=torch.int64, device="cuda")
    cl = helpers.Client(O, 5, hamming_weight=16)
    _, baby = load_keys(P, O, cl, [q * m for q in range(1, N1)])
    _, giant = load_keys(P, O, cl, [p * N1 * m for p in range(1, C // N1)])
    with pytest.raises(B.CkksError) as e:                       # nothing loaded
        B.ckks_ctpt_matmul(P, w, x, baby, giant)
    assert e.value.code == -1 and "diagonal 0 of 16 was never loaded" in str(e.value)
    B.ckks_weights_set_diagonals(w, 0, torch.zeros((5, N), dtype=torch.int64, device="cuda"))
    with pytest.raises(B.CkksError) as e:                       # partly loaded
        B.ckks_ctpt_matmul(P, w, x, baby, giant)
    assert "diagonal 5 of 16" in str(e.value)
    B.ckks_weights_set_diagonals(w, 5, torch.zeros((11, N), dtype=torch.int64, device="cuda"))
    with pytest.raises(B.CkksError) as e:
        B.ckks_ctpt_matmul(P, w, x, baby, giant, flags=8)
    assert e.value.code == -1 and "flags" in str(e.value)
    with pytest.raises(B.CkksError) as e:
        B.ckks_ctpt_matmul(P, w, x, baby, giant, d_ct_y=x)
    assert e.value.code == -1 and "overlaps" in str(e.value)
    y, _ = B.ckks_ctpt_matmul(P, w, x, baby, giant)             # complete and well-formed: runs
    torch.cuda.synchronize()
    assert int(y.abs().max()) == 0
    with pytest.raises(B.CkksError) as e:
        B.ckks_rescale(P, x, level, 1, d_ct_out=x.view(-1)[:2 * (level - 1) * N])
    assert "overlaps" in str(e.value)
    with pytest.raises(B.CkksError) as e:
        B.ckks_rotate_hoisted(P, x, level, [1], [None], d_ct_out=x)
    assert "overlaps" in str(e.value)
    # the scratch arena was sized by the create calls: the projection did not grow it, and a reservation does
    before = B.ckks_params_scratch_bytes(P)
    B.ckks_params_reserve(P, before + 4096)
    assert B.ckks_params_scratch_bytes(P) == before + 4096


def test_adopted_key_gives_the_same_rotation():
    """ckks_galois_key_adopt (the library converts the caller's buffer in place and borrows it) against
    ckks_galois_key_load (the library keeps a copy): identical outputs of a hoisted rotation."""
    B = _B()
    O = helpers.small_oracle(11, L=4, K=2, dnum=2, qbits=45, pbits=50)
    _, P = make_pair(O)
    cl = helpers.Client(O, 77, hamming_weight=16)
    ct = to_dev(cl.encrypt_slots(W.unit_disk_slots(W.rng(3), O.n), 2.0 ** 35, 4))
    g = O.galois_elt(3)
    key = cl.galois_key(g)
    k_copy = B.ckks_galois_key_load(P, g, to_dev(key))
    buf = to_dev(key)
    k_adopt = B.ckks_galois_key_adopt(P, g, buf)
    a = B.ckks_rotate_hoisted(P, ct, 4, [3], [k_copy])
    b = B.ckks_rotate_hoisted(P, ct, 4, [3], [k_adopt])
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert (to_host(a)[0] == O.rotate_hoisted(to_host(ct), 4, [g], [key])[0]).all()


@pytest.mark.parametrize("C,d_in,d_out", [(16, 16, 40), (2, 3, 80), (16, 5, 16)])
def test_separate_giant_step_over_several_batches(C, d_in, d_out):
    """Every giant rotation a complete switch: 45 rotations of three blocks, 40 blocks of one rotation (more than a batch
    holds, batches that end inside a rotation, sums that go on from what the last batch left) and 15 of one block."""
    O = helpers.small_oracle(12, L=3, K=1, dnum=3, qbits=40, pbits=42)
    _, P = make_pair(O)
    r = W.rng(64)
    X, Wm = r.uniform(-1, 1, (4, d_in)), r.uniform(-0.5, 0.5, (d_in, d_out))
    Y, ref, cnt, _ = run_case(O, P, X, Wm, r.uniform(-0.5, 0.5, d_out), 4, C, 1, 30, 3, 65, hw=16, real=True)
    assert np.abs(Y - ref).max() <= 1e-3
    assert cnt.key_switches == -(-d_out // C) * (C - 1)


@pytest.mark.parametrize("L,dnum,C,N1,G,B_out", [(3, 3, 128, 8, 1, 1), (3, 3, 128, 128, 2, 1), (12, 12, 64, 2, 1, 1),
                                                 (3, 3, 32, 1, 2, 40), (12, 4, 64, 4, 2, 2)])
def test_arena_of_a_projection(L, dnum, C, N1, G, B_out):
    """ckks_weights_create reserves what either giant-step order needs with one rotation of up to 32 blocks (or 32 inputs) per
    batch; that the separate order takes several rotations into a batch costs at most a quarter more, or 256 MiB."""
    B = _B()
    O = helpers.small_oracle(13, L=L, K=1, dnum=dnum, qbits=50, pbits=60)
    _, P = make_pair(O)
    level, K, N, N2 = L, 1, O.N, C // N1
    before = B.ckks_params_scratch_bytes(P)
    w = B.ckks_weights_create(P, level, 4, C, G, B_out, N1)
    ctw, digits = 2 * level * N, dnum * (level + K) * N
    batch = min(32, max(G, B_out))
    words = batch * (digits + level * N) + 32 * 2 * (2 * level + K) * N        # key switch
    words += (G * N1 + B_out * N2) * ctw                                       # bank, accumulators
    words += B_out * ctw + 64 * 2 * N                                          # blocks and dropped limbs of the rescale
    if N2 > 1:
        words += B_out * 2 * (level + K) * N + min(8, N2 - 1) * min(batch, B_out) * digits     # merged order
    one = max(before, 8 * words)
    got = B.ckks_params_scratch_bytes(P)
    assert one <= got <= max(one * 5 // 4, one + (256 << 20))
    assert N2 > 1 or got == one
    w.close()


@pytest.mark.parametrize("logN,level,C,G,B_out,N1,kinds", [(14, 5, 4, 3, 6, 2, "r"), (14, 5, 4, 3, 5, 2, "r"), (14, 4, 4, 5, 13, 2, "r"),
                                                            (14, 5, 4, 3, 7, 2, "gr"),          # general inputs, then a real one
                                                            (16, 4, 2, 66, 4, 1, "g"), (16, 4, 2, 66, 6, 1, "g"),
                                                            (16, 4, 2, 67, 5, 1, "g"),
                                                            # the border of the two kinds inside a record of four steps
                                                            (14, 5, 4, 4, 3, 1, "gr"), (14, 5, 4, 4, 7, 1, "rg"),
                                                            (16, 4, 2, 72, 4, 1, "gr"), (16, 4, 2, 72, 6, 1, "gr"),
                                                            # half records: 24 steps and more, or 12 where no wavefront is idle
                                                            (14, 5, 4, 12, 6, 2, "r"), (14, 5, 4, 13, 5, 2, "r"), (14, 4, 4, 27, 7, 1, "r"),
                                                            (14, 5, 4, 27, 7, 1, "rg"), (14, 5, 4, 6, 8, 2, "r"), (14, 5, 4, 15, 4, 1, "rg")])
def test_wavefronts_that_share_the_bank(logN, level, C, G, B_out, N1, kinds):
    """Launches of 256 workgroups and more whose wavefronts share bank residues by four (three and seven tiles, the last ones short,
    steps behind the last whole record) and by two; kinds of the input groups, the first letter for all but the last of two, where
    either launch masks the other's steps of a record they share.  Every output block: each wavefront of a workgroup takes a tile."""
    import oracle
    B = _B()
    O = oracle.Oracle(logN, oracle.find_primes(50, logN, level), oracle.find_primes(60, logN, 2), 1 if level > 8 else level)
    P = B.ckks_params_create(O.logN, O.q, O.p, O.dnum)
    r = W.rng(logN + G + B_out)
    m, N2 = O.n // 8, C // N1
    diag = r.integers(-1 << 40, 1 << 40, (B_out, N2, G, N1, O.N))
    for g in range(G):
        if kinds[0 if g + 1 < G or len(kinds) == 1 else 1] == "r":
            diag[:, :, g] = make_real(diag[:, :, g])
    top = np.array(O.q, dtype=np.uint64)[:, None] - np.uint64(1)
    x = W.uniform_residues(r, O.q, O.N, lead=(G, 2))
    x = np.where(r.integers(0, 5, x.shape) == 0, top, x)
    steps = [q * m for q in range(1, N1)], [p * N1 * m for p in range(1, N2)]
    keys = [[W.uniform_residues(r, O.moduli, O.N, lead=(O.dnum, 2)) for _ in s] for s in steps]
    baby, giant = [[B.ckks_galois_key_load(P, O.galois_elt(s), to_dev(k)) for s, k in zip(ss, kk)] for ss, kk in zip(steps, keys)]
    w = B.ckks_weights_create(P, level, m, C, G, B_out, N1)
    B.ckks_weights_set_diagonals(w, 0, to_dev(diag.reshape(-1, O.N)))
    got = to_host(B.ckks_ctpt_matmul(P, w, to_dev(x), baby, giant)[0])
    want = O.ctpt_matmul(level, m, G, B_out, N1, N2, diag, None, 0, x, keys[0], keys[1])
    for b in range(B_out):
        assert (got[b] == want[b]).all(), b
