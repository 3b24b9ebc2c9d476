"""More than 32 rows on few columns: the kernel for few rows, 32 rows at a time.  Its route by name, then
every output word against the oracle."""
import re

import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

# m, k, n, N, L, x_bits, q_bits, problems, slices of k: rows on both sides of a row tile, the last
# one with a single row; sixteen k-blocks, an odd number of them, a last one that is not full; column
# groups that are and that are not whole rounds of the XCDs; every plane count; a batch
SHAPES = [
    (33, 512, 32, 32, 1, 20, 54, 1, 8), (64, 513, 64, 32, 1, 16, 50, 1, 8), (65, 545, 64, 64, 2, 32, 54, 1, 8),
    (97, 700, 96, 32, 1, 24, 62, 1, 8), (128, 1000, 320, 64, 1, 20, 54, 1, 8), (200, 600, 160, 32, 1, 32, 62, 1, 8),
    (40, 520, 2048, 1024, 1, 16, 62, 1, 4), (70, 1600, 1536, 128, 1, 20, 54, 1, 2), (513, 512, 32, 32, 1, 9, 40, 1, 8),
    (50, 640, 64, 64, 1, 20, 54, 3, 8),
    # seven to nine k-blocks: slices of one stage and of two, the last k-block alone in its stage or short of
    # rows, a last row tile of one row to 32, columns that are not whole groups of a workgroup, batches
    (33, 221, 127, 128, 2, 20, 54, 3, 4), (34, 215, 300, 512, 2, 20, 54, 1, 4), (63, 193, 707, 512, 1, 32, 54, 1, 4),
    (64, 224, 64, 32, 1, 16, 50, 1, 4), (65, 225, 128, 512, 2, 24, 40, 1, 4), (97, 248, 131, 512, 1, 20, 62, 1, 4),
    (128, 256, 29, 256, 1, 32, 54, 1, 4), (130, 257, 160, 32, 1, 32, 62, 1, 4), (161, 275, 23, 128, 1, 24, 40, 1, 4),
    (193, 255, 121, 128, 1, 9, 54, 2, 4), (255, 288, 30, 128, 1, 32, 54, 2, 4), (48, 283, 35, 64, 2, 20, 62, 2, 4),
]


@pytest.mark.parametrize("m,k,n,N,L,x_bits,q_bits,problems,slices", SHAPES)
def test_more_rows_on_few_columns(oracle, m, k, n, N, L, x_bits, q_bits, problems, slices):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli = ci.limb_primes(q_bits, 14, L)
    Ch = -(-n // N)
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, L, moduli, staged=True, count=problems)
    line = re.match(r"cop_thin_kernel<\d, \d, 2, \(nimbus::ThinShares\)3, (\d+)> grid=(\d+),(\d+) ", route[0])
    assert line, route
    room, blocks, count = map(int, line.groups())
    assert count == problems and room == (1 if problems == 1 else 16)
    assert blocks == -(-Ch * 2 * L * N // 16 * slices // 8) * -(-m // 32), route
    print(f"[thin rows] m={m} k={k} n={n} N={N} x_bits={x_bits} q_bits={q_bits} problems={problems}: {route[0]}", flush=True)
    staged, prepared, masks, outs, wants = [], [], [], [], []
    for b in range(problems):
        seed = 9000 + 10 * (m + k) + b
        X = ci.gen_X(seed, m, k, x_bits)
        X[0, :] = X[-1, :] = (1 << x_bits) - 1
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
        # (a row behind the last one shows a store past the end)
        outs.append(torch.empty((m + 1, Ch, 2, L, N), dtype=torch.int64, device="cuda"))
    for which, msks in enumerate((masks, None)):
        for out in outs:
            out.fill_(-1)
        if problems == 1:
            nc.nimbus_cop_matmul_staged(staged[0], m, k, x_bits, prepared[0], n, N, L, moduli,
                                        msks[0] if msks else None, outs[0][:m])
        else:
            nc.nimbus_cop_matmul_staged_batch(staged, m, k, x_bits, prepared, n, N, L, moduli, msks,
                                              [out[:m] for out in outs])
        for b in range(problems):
            got = gu.host(outs[b])
            assert np.array_equal(got[:m], wants[b][which]), f"problem {b}: " + gu.first_mismatch(got[:m], wants[b][which])
            assert (got[m] == np.uint64(2**64 - 1)).all()
