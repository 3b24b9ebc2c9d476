"""More than 32 rows against the oracle: with ten and eleven accumulators at every length of the tile kernel's
loop's ends; row blocks of 64 rows (few columns) and where they end."""
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


# row blocks of 64 rows: rows on both sides of a block, the last block without its second row tile; one
# and several tiles per XCD; both sides of the line (256 compute units: 16 x 16 blocks, then 17 x 16)
@pytest.mark.parametrize("m,k,N,L,x_bits,q_bits", [
    (65, 33, 32, 1, 20, 54), (96, 100, 64, 2, 20, 54), (128, 450, 64, 1, 20, 54), (129, 70, 256, 2, 16, 50),
    (300, 64, 128, 1, 32, 54), (1024, 40, 512, 1, 20, 54), (1025, 40, 512, 1, 20, 54), (200, 130, 64, 2, 24, 62),
    (100, 200, 32, 1, 12, 62),
])
def test_row_blocks_of_64(oracle, m, k, N, L, x_bits, q_bits):
    check(oracle, m, k, N, N, L, x_bits, q_bits)
