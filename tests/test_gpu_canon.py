"""The kernel on the canonical layout at the edges of its stages and tiles: every output word against the
oracle."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu


# rows on both sides of a 16-row tile, of a wave's second, and of a row block; k on both sides of a stage,
# of eight k and of the loop's ends; every plane count, residues that are centred and that are not;
# limbs that share a 64-column tile
@pytest.mark.parametrize("x_bits,q_bits,L", [(9, 40, 1), (16, 50, 2), (20, 54, 1), (24, 55, 2), (32, 54, 2), (32, 55, 1),
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
