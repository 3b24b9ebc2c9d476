"""The kernel for few rows (m <= 32) at the edges of its tiles, slices and routes: every output word
against the oracle, through the call that stages and multiplies (up to 16 rows: from the shares
themselves), the staged call and the batch; and the workspace that the first one leaves behind.
(From staged shares the short inner dimensions among SHAPES are faster with the tile kernel, and go
there; ROUTED holds sizes that do not, and the instance that each is there for.)"""
import re

import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

# rows on both sides of a 16-row tile; k on both sides of a k-block, a 64-wide stage, the stages in
# flight and the eight slices of k; columns for 8, 4, 2 and 1 slices; every plane count; shares of
# two halves; weights of two limbs in one workgroup; shares whose planes do not fit the LDS
SHAPES = [
    (1, 1, 32, 32, 1, 16, [50]), (1, 31, 32, 32, 2, 20, [54, 54]), (15, 33, 64, 64, 1, 32, [54]),
    (16, 64, 64, 1024, 1, 16, [50]), (17, 65, 40, 64, 2, 20, [54, 54]), (31, 96, 64, 64, 1, 24, [62]),
    (32, 129, 32, 32, 1, 32, [62]), (4, 257, 64, 64, 2, 9, [40, 40]), (16, 513, 64, 32, 1, 20, [55]),
    (7, 1025, 32, 32, 1, 32, [54]), (3, 2337, 32, 32, 1, 32, [54]), (2, 100, 2048, 2048, 2, 20, [54, 54]),
    (20, 70, 4096, 4096, 2, 16, [50, 50]), (5, 449, 8192, 8192, 2, 24, [55, 55]), (9, 321, 8192, 8192, 2, 20, [54, 54]),
    (17, 64, 8192, 8192, 2, 20, [54, 54]), (32, 90, 8192, 8192, 2, 32, [62, 62]), (32, 2000, 32, 32, 1, 32, [54]),
    (33, 64, 32, 32, 1, 20, [54]),
    (6, 20, 24576, 8192, 2, 16, [62, 62]),              # three rounds of tiles: staged, then the tiles
    (16, 300, 64, 64, 2, 64, [59, 55]), (27, 130, 64, 64, 1, 40, [59]), (1, 70, 32, 32, 1, 48, [50]),
]


@pytest.mark.parametrize("m,k,n,N,L,x_bits,q_bits", SHAPES)
def test_few_rows(oracle, m, k, n, N, L, x_bits, q_bits):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    t_bits = min(x_bits, 32)
    moduli = ci.limb_primes(q_bits[0], 14 if x_bits > 32 else t_bits, L)
    if len(set(q_bits)) > 1:
        moduli = tuple(ci.limb_primes(b, 14, 1)[0] for b in q_bits)
    Ch = -(-n // N)
    X = ci.gen_X(600 + m + k, m, k, x_bits)
    X[0, 0] = X[-1, -1] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(600 + m + k, k, Ch, moduli, N)
    mask = ci.gen_mask_uniform(600 + m + k, m, Ch, moduli, N)
    for l, q in enumerate(moduli):
        ctW[:, 0, :, l, :4] = q - 1
        mask[0, 0, :, l, :4] = q - 1
    print(f"[thin] m={m} k={k} n={n} N={N} x_bits={x_bits} q_bits={q_bits}", flush=True)
    prepared = gu.prepare(ctW, moduli, n, N)
    ws_bytes = nc.nimbus_cop_workspace_bytes(m, k, x_bits)
    dX = gu.dev(X)
    staged = torch.full((ws_bytes,), 85, dtype=torch.uint8, device="cuda")
    nc.nimbus_cop_stage_shares(dX, m, k, x_bits, staged)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, n, N, msk, wide=x_bits > 32)
        dM = gu.dev(msk) if msk is not None else None
        ws = torch.full((ws_bytes,), 170, dtype=torch.uint8, device="cuda")
        out = torch.full((m, Ch, 2, L, N), -1, dtype=torch.int64, device="cuda")
        nc.nimbus_cop_matmul_prepared(dX, m, k, x_bits, prepared, n, N, L, moduli, dM, out, ws)
        got = gu.host(out)
        assert np.array_equal(got, want), "prepared: " + gu.first_mismatch(got, want)
        assert torch.equal(ws, staged)                      # the planes, whichever way was taken
        out.fill_(-1)
        nc.nimbus_cop_matmul_staged(staged, m, k, x_bits, prepared, n, N, L, moduli, dM, out)
        got = gu.host(out)
        assert np.array_equal(got, want), "staged: " + gu.first_mismatch(got, want)
    if x_bits <= 32:
        outs = [torch.full((m, Ch, 2, L, N), -1, dtype=torch.int64, device="cuda") for _ in range(2)]
        nc.nimbus_cop_matmul_staged_batch([staged, staged], m, k, x_bits, [prepared, prepared], n, N, L, moduli,
                                          None, outs)
        for out in outs:
            got = gu.host(out)
            assert np.array_equal(got, want), "batch: " + gu.first_mismatch(got, want)


# m, k, n, N, L, x_bits, q_bits, problems: 16-row tiles, where the shares come from (0 staged planes per
# wave, 1 copied to LDS once), slices of k.  One k-block to several stages in one slice, the last
# column group alone in its workgroup; two, four and eight slices with and without a remainder;
# every plane count; the last shape's planes do not fit the LDS
ROUTED = [
    (1, 193, 5120, 1024, 2, 20, 54, 1, (1, 0, 1)), (16, 255, 5120, 1024, 2, 16, 50, 1, (1, 0, 1)),
    (15, 128, 10272, 32, 1, 32, 62, 1, (1, 0, 1)), (16, 161, 6144, 1024, 2, 24, 62, 1, (1, 0, 1)),
    (9, 225, 5120, 1024, 2, 16, 62, 1, (1, 0, 1)), (7, 865, 3072, 1024, 2, 20, 54, 1, (1, 0, 2)),
    (16, 417, 32, 32, 1, 32, 54, 1, (1, 0, 4)), (2, 379, 32, 32, 1, 32, 62, 1, (1, 0, 4)),
    (16, 513, 64, 32, 1, 20, 55, 1, (1, 0, 8)), (16, 1025, 32, 32, 1, 32, 62, 1, (1, 0, 8)),
    (17, 1256, 5120, 1024, 2, 20, 54, 1, (2, 1, 1)), (32, 545, 6144, 1024, 2, 32, 62, 1, (2, 1, 1)),
    (31, 1121, 5120, 1024, 2, 24, 62, 1, (2, 1, 1)), (20, 1364, 5120, 1024, 2, 32, 54, 1, (2, 0, 1)),
    (17, 441, 32, 32, 1, 32, 62, 1, (2, 0, 4)), (32, 448, 32, 32, 2, 32, 62, 1, (2, 0, 4)),
    (25, 513, 32, 32, 2, 24, 62, 1, (2, 0, 8)), (32, 1025, 32, 32, 1, 32, 62, 1, (2, 0, 8)),
    # batches: problems with shares, weights and masks of their own
    (16, 168, 2048, 1024, 2, 20, 54, 3, (1, 0, 1)), (5, 364, 64, 64, 1, 32, 62, 3, (1, 0, 4)),
    (17, 751, 2048, 1024, 2, 32, 54, 3, (2, 1, 1)), (32, 565, 2048, 1024, 2, 32, 62, 3, (2, 1, 1)),
    (32, 441, 32, 32, 2, 32, 62, 3, (2, 0, 4)), (24, 600, 64, 64, 2, 24, 62, 4, (2, 0, 8)),
]


@pytest.mark.parametrize("m,k,n,N,L,x_bits,q_bits,problems,instance", ROUTED)
def test_few_rows_from_staged_shares(oracle, m, k, n, N, L, x_bits, q_bits, problems, instance):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli = ci.limb_primes(q_bits, 14, L)
    Ch = -(-n // N)
    tiles, source, slices = instance
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, L, moduli, staged=True, count=problems)
    line = re.match(r"cop_thin_kernel<\d, \d, (\d), \(nimbus::ThinShares\)(\d), (\d+)> grid=(\d+),(\d+) ", route[0])
    assert line, route
    rt, src, room, blocks, count = map(int, line.groups())
    assert (rt, src, count) == (tiles, source, problems) and room == (1 if problems == 1 else 16)
    assert blocks == -(-Ch * 2 * L * N // 16 * slices // 8), route
    print(f"[thin] m={m} k={k} n={n} N={N} x_bits={x_bits} q_bits={q_bits} problems={problems}: {route[0]}", flush=True)
    staged, prepared, masks, outs, wants = [], [], [], [], []
    for b in range(problems):
        seed = 3000 + 10 * (m + k) + b
        X = ci.gen_X(seed, m, k, x_bits)
        X[0, 0] = X[-1, -1] = (1 << x_bits) - 1
        ctW = ci.gen_ctW_uniform(seed, k, Ch, moduli, N)
        mask = ci.gen_mask_uniform(seed, m, Ch, moduli, N)
        for l, q in enumerate(moduli):
            ctW[:, 0, :, l, :4] = q - 1
            mask[0, 0, :, l, :4] = q - 1
        wants.append([oracle.cop_ref(X, ctW, moduli, n, N, msk)[0] for msk in (mask, None)])
        staged.append(torch.full((nc.nimbus_cop_workspace_bytes(m, k, x_bits),), 85, dtype=torch.uint8, device="cuda"))
        nc.nimbus_cop_stage_shares(gu.dev(X), m, k, x_bits, staged[-1])
        prepared.append(gu.prepare(ctW, moduli, n, N))
        masks.append(gu.dev(mask))
        outs.append(torch.empty((m, Ch, 2, L, N), dtype=torch.int64, device="cuda"))
    for which, msks in enumerate((masks, None)):
        for out in outs:
            out.fill_(-1)
        if problems == 1:
            nc.nimbus_cop_matmul_staged(staged[0], m, k, x_bits, prepared[0], n, N, L, moduli,
                                        msks[0] if msks else None, outs[0])
        else:
            nc.nimbus_cop_matmul_staged_batch(staged, m, k, x_bits, prepared, n, N, L, moduli, msks, outs)
        for b in range(problems):
            got = gu.host(outs[b])
            assert np.array_equal(got, wants[b][which]), f"problem {b}: " + gu.first_mismatch(got, wants[b][which])
