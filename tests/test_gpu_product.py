"""Rings of 1024 to 8192 coefficients: the transform kernel that stops two stages early (moduli from 2^34 to
2^59) and the full one (a modulus outside that), every number of stages a round at both ends of the batch sizes
that take it, against the oracle's schoolbook product, bit for bit."""
import numpy as np
import pytest

import cop_inputs as ci
from test_gpu_rlwe import _gpu_phase, _primes, _tables

pytestmark = pytest.mark.gpu

# N, ciphertexts, limbs, bits of the moduli: 256 | 257 and 1023 | 1024 polynomials are where the
# number of stages a round changes
CASES = [
    (1024, 1, 1, 35), (1024, 257, 1, 58), (1024, 512, 2, 59),
    (2048, 256, 1, 58), (2048, 257, 1, 58), (2048, 129, 2, 59),
    (4096, 128, 2, 58), (4096, 257, 1, 58), (4096, 341, 3, 35), (4096, 1024, 1, 58), (4096, 512, 2, 59),
    (8192, 1, 1, 35), (8192, 65, 4, 58), (8192, 2, 2, 59),
]


@pytest.mark.parametrize("N,T,L,q_bits", CASES)
def test_phase_at_the_ends_of_each_kind_of_batch(oracle, N, T, L, q_bits):
    """uniform ciphertexts, the first of them with c1 = q - 1 everywhere; a secret of the largest coefficients"""
    moduli = _primes(q_bits, 16, N, L)
    rng = np.random.default_rng(N + T)
    s = rng.choice(np.array([-128, -127, -1, 0, 1, 126, 127], dtype=np.int8), size=N)
    ct = ci.uniform_residues(N + T, 43, (T, 2), moduli, N)
    for l, q in enumerate(moduli):
        ct[0, 1, l] = q - 1
    print(f"[product] N={N} T={T} L={L} q_bits={q_bits}", flush=True)
    got = _gpu_phase(ct, moduli, _tables(N, moduli, s))
    for r in sorted({0, T // 2, T - 1}):
        assert np.array_equal(got[r], oracle.phase(ct[r], s, moduli)), f"ciphertext {r}"


# N, ciphertexts, bits of each limb: one modulus below 2^34 or from 2^59 on takes all limbs to the full transform, in
# rounds of min(4, log N - 10) stages (2 at least) below 1024 polynomials and min(4, log N - 8) from there on
FULL = [
    (1024, 3, [34]), (1024, 1024, [60]), (2048, 3, [33, 62]), (2048, 1024, [61]),
    (4096, 1, [62]), (4096, 511, [60, 54]), (4096, 512, [62, 60]), (4096, 1024, [34]), (4096, 341, [54, 60, 34]),
    (8192, 2, [61, 59]), (8192, 341, [62, 55, 34]), (8192, 512, [60, 62]), (8192, 1024, [33]),
]


def _limbs(bits, N, t_bits):
    return tuple(ci.limb_primes(b, max(t_bits, N.bit_length()), 1)[0] for b in bits)


@pytest.mark.parametrize("N,T,bits", FULL)
def test_phase_with_moduli_of_the_full_transform(oracle, N, T, bits):
    moduli = _limbs(bits, N, 16)
    rng = np.random.default_rng(N + T)
    s = rng.choice(np.array([-128, -127, -1, 0, 1, 126, 127], dtype=np.int8), size=N)
    ct = ci.uniform_residues(N + T, 44, (T, 2), moduli, N)
    for l, q in enumerate(moduli):
        ct[0, 1, l] = q - 1
    print(f"[full] N={N} T={T} bits={bits}", flush=True)
    got = _gpu_phase(ct, moduli, _tables(N, moduli, s))
    for r in sorted({0, T // 2, T - 1}):
        assert np.array_equal(got[r], oracle.phase(ct[r], s, moduli)), f"ciphertext {r}"


# N, weight rows, bits of each limb: of either transform every number of stages a round (rows times limbs are the polynomials)
ENCRYPT = [
    (1024, 300, [58]), (2048, 256, [59]), (2048, 150, [58, 57]), (2048, 257, [59]),
    (4096, 256, [59]), (4096, 150, [58, 54]), (4096, 257, [59]), (4096, 515, [58, 35]), (4096, 1030, [59]),
    (8192, 300, [58]), (8192, 150, [59, 55]),
    (1024, 3, [60]), (2048, 1030, [62]), (4096, 3, [62]), (4096, 515, [60, 54]), (8192, 3, [34, 61]), (8192, 1030, [60]),
]


@pytest.mark.parametrize("N,rows,bits", ENCRYPT)
def test_encryption_with_a_secret_of_every_coefficient(oracle, N, rows, bits):
    """uniform a (q - 1 everywhere in the first row), errors and weights at the ends of their ranges among them"""
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    t_bits, L = 16, len(bits)
    moduli = _limbs(bits, N, t_bits)
    rng = np.random.default_rng(N + rows)
    s = rng.integers(-128, 128, N).astype(np.int8)
    W = rng.integers(0, 1 << t_bits, (rows, N)).astype(np.uint64)
    e = rng.integers(-128, 128, (rows, N)).astype(np.int8)
    W[:, :2], W[:, -2:] = (1 << t_bits) - 1, 0
    a = ci.uniform_residues(N + rows, 45, (rows,), moduli, N)
    for l, q in enumerate(moduli):
        a[0, l] = q - 1
    print(f"[encrypt] N={N} rows={rows} bits={bits}", flush=True)
    ctW = torch.full((rows, 1, 2, L, N), -1, dtype=torch.int64, device="cuda")
    nc.nimbus_rlwe_encrypt(gu.dev(W), rows, N, t_bits, N, L, moduli, _tables(N, moduli, s), gu.dev(a),
                           torch.from_numpy(e).cuda(), ctW)
    got = gu.host(ctW)[:, 0]
    assert np.array_equal(got[:, 1], a)
    for r in sorted({0, rows // 2, rows - 1}):
        want = oracle.encrypt_rns(W[r:r + 1], s, a[r:r + 1], e[r:r + 1], moduli, t_bits)[0]
        assert np.array_equal(got[r], want), f"row {r}: " + gu.first_mismatch(got[r], want)
