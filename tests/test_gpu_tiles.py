"""The 128 x 64 tile kernel where its loop has a single operand set, at every length of the loop's
ends, against the oracle."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu


def check(oracle, m, k, n, N, L, x_bits, q_bits):
    import gpu_util as gu
    moduli = ci.limb_primes(q_bits, x_bits, L)
    X = ci.gen_X(800 + m + k, m, k, x_bits)
    X[0, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(800 + m + k, k, -(-n // N), moduli, N)
    mask = ci.gen_mask_uniform(800 + m + k, m, -(-n // N), moduli, N)
    for l, q in enumerate(moduli):
        ctW[:, 0, :, l, :4] = q - 1
    print(f"[tiles] m={m} k={k} n={n} N={N} L={L} x_bits={x_bits} q_bits={q_bits}", flush=True)
    prepared = gu.prepare(ctW, moduli, n, N)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, n, N, msk)
        got = gu.run_mfma(X, ctW, moduli, n, N, x_bits, msk, prepared=prepared)
        assert np.array_equal(got, want), gu.first_mismatch(got, want)


# one to seven k-blocks; rows with waves that have none, one and two row blocks
@pytest.mark.parametrize("x_bits,q_bits", [(32, 54), (24, 62), (32, 62)])
@pytest.mark.parametrize("m,k", [(33, 20), (40, 40), (70, 80), (97, 128), (130, 150), (40, 190), (200, 220)])
def test_one_operand_set(oracle, m, k, x_bits, q_bits):
    check(oracle, m, k, 32, 32, 2, x_bits, q_bits)


# no row tests (m a multiple of 128), more tiles than compute units with the second shape
@pytest.mark.parametrize("m,k,N,x_bits,q_bits", [(128, 70, 8192, 32, 54), (128, 170, 16384, 32, 62),
                                                 (256, 40, 4096, 24, 62)])
def test_one_operand_set_full_blocks(oracle, m, k, N, x_bits, q_bits):
    check(oracle, m, k, N, N, 1 if N > 4096 else 2, x_bits, q_bits)
