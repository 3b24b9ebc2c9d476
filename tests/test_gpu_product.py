"""The transform kernel that stops two stages early (rings of 1024 to 8192 coefficients, moduli from 2^34 to
2^59): every number of stages a round at both ends of the batch sizes that take it, against the oracle's
schoolbook product, bit for bit."""
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
