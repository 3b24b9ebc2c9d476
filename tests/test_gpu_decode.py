"""Decoding of phases whose limbs differ widely in size, and of scalings so small that every quotient
lies on an integer, against the formula on Python integers."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

N = 64


def prime_above(start):
    """the first prime from `start` on that is 1 modulo 2 N"""
    q = -(-(start - 1) // (2 * N)) * 2 * N + 1
    while not ci.is_prime(q):
        q += 2 * N
    return q


# starts of the moduli, t_bits
CASES = [
    ([2**61 + 2**60, 2**33], 32), ([2**33, 2**61 + 2**60], 32), ([2**61, 2**20, 2**55], 16),
    ([2**17, 2**61, 2**45, 2**61 + 2**59], 16), ([2**61 + 2**60, 2**61 + 2**59, 2**61, 2**17], 8),
    ([2**16], 16), ([2**32], 32), ([2**33], 32), ([2**58, 2**54], 32), ([2**55, 2**54, 2**53], 24),
]


@pytest.mark.parametrize("starts,t_bits", CASES)
def test_decode_against_python_integers(starts, t_bits):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli = tuple(prime_above(s + 1) for s in starts)
    L, Q = len(moduli), 1
    for q in moduli:
        Q *= q
    delta = Q >> t_bits
    rng = np.random.default_rng(len(starts) + t_bits)
    values = [0, 1, Q - 1, Q // 2, delta // 2, delta]
    for mm in (1, 3, (1 << t_bits) - 1):
        # on a boundary, next to it, and at distances around 2^-14 of a step, where the estimate is settled
        for d in (-1, 0, 1, -(delta >> 14) - 1, -(delta >> 14), delta >> 14, (delta >> 14) + 1, delta >> 13):
            values.append((delta * mm + delta // 2 + d) % Q)
    while len(values) < 40 * N or len(values) % N:
        values.append(int.from_bytes(rng.bytes(40), "little") % Q)
    T = len(values) // N
    phi = np.array([[[values[t * N + c] % q for c in range(N)] for q in moduli] for t in range(T)], dtype=np.uint64)
    print(f"[decode] L={L} t_bits={t_bits} moduli of {[q.bit_length() for q in moduli]} bits", flush=True)
    out = torch.full((T, N), -1, dtype=torch.int64, device="cuda")
    nc.nimbus_rlwe_decode(gu.dev(phi), T, N, L, moduli, t_bits, out)
    want = np.array([((v + delta // 2) // delta) % (1 << t_bits) for v in values], dtype=np.uint64).reshape(T, N)
    got = gu.host(out)
    assert np.array_equal(got, want), gu.first_mismatch(got, want)
