"""The kernel for few rows where its slices are about as long as the stages in flight, from the shares
themselves with one and two 16-row tiles, and on more columns than one descriptor holds of the mask."""
import re

import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

# m, k, n, N, L, x_bits, q_bits: one to nine stages of 64 k in one, two, four and eight slices (up to four are
# in flight of a wave, two with wide operands), slices of unequal length, a last k-block alone and in a
# pair; both sides of a 16-row tile; elements finished in pairs and one by one; every plane count
SHAPES = [
    (1, 20, 64, 64, 1, 20, 54), (16, 64, 2048, 1024, 1, 16, 50), (3, 128, 512, 512, 1, 32, 62), (16, 200, 8192, 8192, 2, 24, 62),
    (5, 256, 5120, 1024, 1, 20, 54), (16, 270, 2048, 2048, 2, 32, 54), (2, 330, 8192, 8192, 2, 16, 62), (9, 545, 64, 32, 1, 20, 55),
    (17, 70, 2048, 2048, 1, 20, 54), (32, 130, 2048, 2048, 1, 16, 50), (31, 200, 512, 512, 1, 32, 62), (24, 280, 2048, 2048, 2, 24, 62),
    (32, 300, 64, 64, 1, 32, 54), (18, 545, 32, 32, 1, 16, 62), (32, 520, 4096, 4096, 1, 20, 54),
]


@pytest.mark.parametrize("m,k,n,N,L,x_bits,q_bits", SHAPES)
def test_short_slices_from_the_shares(oracle, m, k, n, N, L, x_bits, q_bits):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli, Ch = ci.limb_primes(q_bits, 14, L), -(-n // N)
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, L, moduli)
    assert len(route) == 1 and re.match(rf"cop_thin_kernel<\d, \d, {-(-m // 16)}, \(nimbus::ThinShares\)2, 1> ", route[0]), route
    print(f"[thin short] m={m} k={k} n={n} N={N} x_bits={x_bits} q_bits={q_bits}: {route[0]}", flush=True)
    X = ci.gen_X(700 + m + k, m, k, x_bits)
    X[0, :] = X[-1, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(700 + m + k, k, Ch, moduli, N)
    mask = ci.gen_mask_uniform(700 + m + k, m, Ch, moduli, N)
    for l, q in enumerate(moduli):
        ctW[:, 0, :, l, :4] = q - 1
        mask[0, 0, :, l, :4] = mask[-1, -1, :, l, -4:] = q - 1
    prepared = gu.prepare(ctW, moduli, n, N)
    ws_bytes = nc.nimbus_cop_workspace_bytes(m, k, x_bits)
    planes = torch.full((ws_bytes,), 85, dtype=torch.uint8, device="cuda")
    nc.nimbus_cop_stage_shares(gu.dev(X), m, k, x_bits, planes)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, n, N, msk)
        ws = torch.full((ws_bytes,), 170, dtype=torch.uint8, device="cuda")
        out = torch.full((m + 1, Ch, 2, L, N), -1, dtype=torch.int64, device="cuda")   # a row behind the last one
        nc.nimbus_cop_matmul_prepared(gu.dev(X), m, k, x_bits, prepared, n, N, L, moduli,
                                      gu.dev(msk) if msk is not None else None, out[:m], ws)
        got = gu.host(out)
        assert np.array_equal(got[:m], want), gu.first_mismatch(got[:m], want)
        assert (got[m] == np.uint64(2**64 - 1)).all() and torch.equal(ws, planes)


def test_masks_on_more_columns_than_a_descriptor_holds():
    """2^23 columns, against the vector-ALU kernel on the canonical layout"""
    import torch
    import paper_2411_15707_amd as nc
    m, k, N, Ch, x_bits = 2, 40, 65536, 64, 20
    n, moduli = Ch * N, ci.limb_primes(54, 20, 1)
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, 1, moduli)
    assert len(route) == 1 and route[0].startswith("cop_thin_kernel"), route
    print(f"[thin short] 2^23 columns: {route[0]}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    draw = lambda shape, bound: torch.randint(0, bound, shape, dtype=torch.int64, device="cuda", generator=gen)
    X, ctW, mask = draw((m, k), 1 << x_bits), draw((k, Ch, 2, 1, N), moduli[0]), draw((m, Ch, 2, 1, N), moduli[0])
    prepared = torch.empty(nc.nimbus_cop_prepared_bytes(k, n, N, 1, moduli), dtype=torch.uint8, device="cuda")
    nc.nimbus_cop_prepare(ctW, k, n, N, 1, moduli, prepared)
    ws = torch.empty(nc.nimbus_cop_workspace_bytes(m, k, x_bits), dtype=torch.uint8, device="cuda")
    for msk in (mask, None):
        want, out = torch.empty_like(mask), torch.full_like(mask, -1)
        nc.nimbus_cop_matmul_valu(X, m, k, x_bits, ctW, n, N, 1, moduli, msk, want)
        nc.nimbus_cop_matmul_prepared(X, m, k, x_bits, prepared, n, N, 1, moduli, msk, out, ws)
        assert torch.equal(out, want)
