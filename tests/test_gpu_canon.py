"""The kernel on the canonical layout at the edges of its stages and tiles: every output word against the
oracle."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu


# rows on both sides of a 16-row tile, of a wave's second, and of a row block; k on both sides of a stage,
# of eight k and of the loop's ends; every plane count, residues that are centred and that are not;
# limbs that share a 64-column tile
@pytest.mark.parametrize("x_bits,q_bits,L", [(9, 40, 1), (16, 50, 2), (16, 55, 1), (20, 54, 1), (24, 55, 2), (32, 54, 2), (32, 55, 1),
                                            (16, 62, 1), (24, 62, 1)])
@pytest.mark.parametrize("m,k,n,N", [(1, 1, 32, 32), (16, 64, 32, 32), (17, 63, 64, 32), (33, 65, 40, 64), (48, 128, 32, 32),
                                     (64, 129, 64, 64), (65, 200, 512, 512), (113, 192, 32, 32), (128, 71, 96, 32),
                                     (129, 257, 64, 64), (256, 320, 1024, 512), (300, 40, 320, 64)])
def test_canonical_layout(oracle, m, k, n, N, x_bits, q_bits, L):
    import gpu_util as gu
    moduli = ci.limb_primes(q_bits, min(x_bits, 14), L)
    Ch = -(-n // N)
    X = ci.gen_X(4400 + m + k, m, k, x_bits)
    X[0, :] = X[-1, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(4400 + m + k, k, Ch, moduli, N)
    mask = ci.gen_mask_uniform(4400 + m + k, m, Ch, moduli, N)
    for l, q in enumerate(moduli):
        ctW[:, 0, :, l, :2] = q - 1
        ctW[:, 0, :, l, 2:4] = (q - 1) // 2
        ctW[:, 0, :, l, 4:6] = (q + 1) // 2
        mask[0, 0, :, l, :4] = q - 1
    print(f"[canon] m={m} k={k} n={n} N={N} L={L} x_bits={x_bits} q_bits={q_bits}", flush=True)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, n, N, msk)
        got = gu.run_canon(X, ctW, moduli, n, N, x_bits, msk)
        assert np.array_equal(got, want), gu.first_mismatch(got, want)


# the choice between 32 and 64 k a stage: one to eight k-blocks, row blocks on both sides of 96 rows, without
# row tests and with them, several row blocks; every plane count, centred and not
@pytest.mark.parametrize("x_bits,q_bits", [(16, 50), (16, 55), (20, 54), (24, 55), (32, 54), (32, 55), (16, 62), (24, 62)])
@pytest.mark.parametrize("m,k", [(96, 70), (97, 20), (97, 96), (100, 160), (128, 30), (128, 64), (128, 90), (128, 150),
                                 (128, 220), (128, 230), (113, 220), (200, 150), (256, 90), (256, 224), (512, 33)])
def test_few_stages(oracle, m, k, x_bits, q_bits):
    import gpu_util as gu
    n, N = 96, 64
    moduli = ci.limb_primes(q_bits, min(x_bits, 14), 1)
    X = ci.gen_X(4600 + m + k, m, k, x_bits)
    X[0, :] = X[-1, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(4600 + m + k, k, 2, moduli, N)
    mask = ci.gen_mask_uniform(4600 + m + k, m, 2, moduli, N)
    q = moduli[0]
    for col, value in enumerate((q - 1, (q - 1) // 2, (q + 1) // 2, 0)):
        ctW[:, 0, :, 0, col] = value
    mask[0, 0, :, 0, :4] = q - 1
    print(f"[canon] few stages: m={m} k={k} x_bits={x_bits} q_bits={q_bits}", flush=True)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, n, N, msk)
        got = gu.run_canon(X, ctW, moduli, n, N, x_bits, msk)
        assert np.array_equal(got, want), gu.first_mismatch(got, want)
