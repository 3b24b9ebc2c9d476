"""Staging of shares wider than 32 bits: the planes of both halves, byte for byte those that the halves
get as shares of their own."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu


# rows and k on both sides of a tile; every plane count of the upper half, widths that do and do not
# end with a byte
@pytest.mark.parametrize("m,k", [(1, 1), (31, 33), (32, 32), (33, 31), (128, 768), (130, 97)])
@pytest.mark.parametrize("x_bits", [33, 40, 48, 50, 56, 63, 64])
def test_both_halves_in_one_launch(m, k, x_bits):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    X = ci.gen_X(5100 + m + k, m, k, x_bits)
    X[0, 0] = (1 << x_bits) - 1
    X[-1, -1] = (1 << x_bits) - 1
    print(f"[stage wide] m={m} k={k} x_bits={x_bits}", flush=True)

    def staged(words, bits):
        # (sixteen bytes behind the planes show a store past the end)
        size = nc.nimbus_cop_workspace_bytes(m, k, bits)
        buf = torch.full((size + 16,), 85, dtype=torch.uint8, device="cuda")
        nc.nimbus_cop_stage_shares(gu.dev(words), m, k, bits, buf[:size])
        got = buf.cpu().numpy()
        assert (got[size:] == 85).all()
        return got[:size]

    want = np.concatenate([staged(X & np.uint64(0xffffffff), 32), staged(X >> np.uint64(32), x_bits - 32)])
    assert np.array_equal(staged(X, x_bits), want)
