"""Encryption where its last step wraps: the secret 1 makes a s the polynomial a itself, so that
q - a s + e and Delta w + (q - a s + e) take their smallest and largest values."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu


def prime_below(end, step):
    """the largest prime below `end` that is 1 modulo `step`"""
    q = (end - 2) // step * step + 1
    while not ci.is_prime(q):
        q -= step
    return q


# ring, ends of the moduli, t_bits: the smallest modulus there is (193, where |e| is most of it), the
# largest, each kind of transform (moduli from 2^34, from 2^58, from 2^59), limbs of unequal size,
# and the ring that is joined from two halves
CASES = [
    (32, [194], 7), (32, [258, 194], 7), (64, [2**30], 16), (64, [2**62], 32), (1024, [2**40, 2**62], 32),
    (2048, [2**59], 32), (4096, [2**54, 2**54 - 2**40], 20), (32768, [2**55], 20), (32768, [2**62, 2**59], 32),
]


@pytest.mark.parametrize("N,ends,t_bits", CASES)
def test_encryption_at_the_ends_of_its_last_step(N, ends, t_bits):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli = tuple(prime_below(e, 2 * N) for e in ends)
    L, t, k = len(moduli), 1 << t_bits, 3
    rng = np.random.default_rng(N + t_bits)
    pick = lambda values, size: np.array(values, dtype=object)[rng.integers(0, len(values), size)]
    a = np.empty((k, L, N), dtype=object)
    for l, q in enumerate(moduli):
        a[:, l] = pick([0, 1, 2, 126, 127, 128, q - 129, q - 128, q - 127, q - 2, q - 1, q // 2], (k, N))
    e = pick([-128, -127, -1, 0, 1, 126, 127], (k, N))
    w = pick([0, 1, t - 1, t // 2, *(int(v) for v in rng.integers(0, t, 40))], (k, N))
    s = np.zeros(N, dtype=np.int8)
    s[0] = 1
    Q = 1
    for q in moduli:
        Q *= q
    delta = Q >> t_bits
    want = np.empty((k, 1, 2, L, N), dtype=np.uint64)
    for l, q in enumerate(moduli):
        want[:, 0, 0, l] = ((delta % q) * w + e - a[:, l]) % q
        want[:, 0, 1, l] = a[:, l]
    print(f"[encrypt] N={N} moduli of {[q.bit_length() for q in moduli]} bits t_bits={t_bits}", flush=True)
    tables = torch.empty(nc.nimbus_rlwe_tables_bytes(N, L), dtype=torch.uint8, device="cuda")
    nc.nimbus_rlwe_setup(N, L, moduli, torch.from_numpy(s).cuda(), tables)
    # both ends of the batch sizes: the kernel for small batches and the one for large ones
    for copies in (1, -(-1024 // (k * L)) if N <= 4096 else 1):
        out = torch.full((copies * k, 1, 2, L, N), -1, dtype=torch.int64, device="cuda")
        nc.nimbus_rlwe_encrypt(gu.dev(np.tile(w.astype(np.uint64), (copies, 1))), copies * k, N, t_bits, N, L, moduli,
                               tables, gu.dev(np.tile(a.astype(np.uint64)[:, None], (copies, 1, 1, 1))),
                               torch.from_numpy(np.tile(e.astype(np.int8), (copies, 1))).cuda(), out)
        got = gu.host(out).reshape(copies, *want.shape)
        for c in range(copies):
            assert np.array_equal(got[c], want), gu.first_mismatch(got[c], want)
