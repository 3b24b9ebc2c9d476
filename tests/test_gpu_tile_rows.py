"""The tile kernel with row tests: waves of one to four 16-row tiles through whole turns of the operand
rings, with the last k-block alone and in a pair, several tiles per workgroup, one and several problems.
The longest inner dimension on the same kernel.  Routes by name, then every output word against the
oracle."""
import re

import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

# share and ciphertext planes: the widths that give them
PLANES = {(2, 7): (16, 50), (3, 7): (20, 54), (4, 7): (32, 54), (2, 8): (16, 62), (3, 8): (24, 62), (4, 8): (32, 62)}
# rows, inner dimension, columns, problems.  More than 256 tiles in all.  16-row tiles of the two halves of
# a workgroup: 77 rows 3 and 2, 97 and 100 rows 4 and 3, 113 rows 4 and 4, 130 rows 3 and 3 then 2 and 1.
# k-blocks: 1, 3, 4, 6, 14 and 15.
SHAPES = [
    (77, 450, 16512, 1), (97, 100, 16512, 1), (100, 417, 16512, 1), (113, 450, 16512, 1), (120, 30, 16512, 1),
    (113, 70, 16512, 1), (130, 417, 8320, 1), (130, 450, 8320, 1), (40, 190, 16512, 1),
    (77, 450, 5504, 3), (113, 417, 5504, 3),
]


def _tile_route(nc, m, k, x_bits, n, N, moduli, masked, problems, planes, full):
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, 1, moduli, masked=masked, staged=True, count=problems)
    flag = "true" if full else "false"
    assert len(route) == 1 and re.match(
        rf"cop_mfma_kernel<{planes[0]}, {planes[1]}, {flag}, (true|false), (true|false), "
        rf"{1 if problems == 1 else 16}> grid=256,1 ", route[0]), route
    return route[0]


@pytest.mark.parametrize("planes", PLANES)
@pytest.mark.parametrize("m,k,C,problems", SHAPES)
def test_rows_of_every_number(oracle, m, k, C, problems, planes):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    x_bits, q_bits = PLANES[planes]
    N = 64
    Ch, n = C // (2 * N), C // 2
    moduli = ci.limb_primes(q_bits, 14, 1)
    q = np.uint64(moduli[0])
    for masked in (True, False):
        route = _tile_route(nc, m, k, x_bits, n, N, moduli, masked, problems, planes, False)
        print(f"[tile rows] m={m} k={k} masked={masked}: {route}", flush=True)
    # (the problems share weights, not shares and masks)
    ctW = ci.gen_ctW_uniform(6100 + m + k, k, Ch, moduli, N)
    ctW[:, 0, :, 0, :4] = q - np.uint64(1)
    prepared = gu.prepare(ctW, moduli, n, N)
    staged, masks, outs, wants = [], [], [], []
    for b in range(problems):
        X = ci.gen_X(6200 + m + k + b, m, k, x_bits)
        X[0, :] = X[-1, :] = (1 << x_bits) - 1
        mask = ci.gen_mask_uniform(6300 + m + k + b, m, Ch, moduli, N)
        mask[0, 0, :, 0, :4] = mask[-1, -1, :, 0, -4:] = q - np.uint64(1)
        plain = oracle.cop_ref(X, ctW, moduli, n, N, None)[0]
        wants.append(((plain + mask) % q, plain))
        staged.append(torch.empty(nc.nimbus_cop_workspace_bytes(m, k, x_bits), dtype=torch.uint8, device="cuda"))
        nc.nimbus_cop_stage_shares(gu.dev(X), m, k, x_bits, staged[-1])
        masks.append(gu.dev(mask))
        # (a row behind the last one shows a store past the end)
        outs.append(torch.empty((m + 1, Ch, 2, 1, N), dtype=torch.int64, device="cuda"))
    for which, msks in enumerate((masks, None)):
        for out in outs:
            out.fill_(-1)
        if problems == 1:
            nc.nimbus_cop_matmul_staged(staged[0], m, k, x_bits, prepared, n, N, 1, moduli,
                                        msks[0] if msks else None, outs[0][:m])
        else:
            nc.nimbus_cop_matmul_staged_batch(staged, m, k, x_bits, [prepared] * problems, n, N, 1, moduli, msks,
                                              [out[:m] for out in outs])
        torch.cuda.synchronize()
        for b in range(problems):
            got = gu.host(outs[b])
            assert np.array_equal(got[:m], wants[b][which]), \
                f"problem {b}: " + gu.first_mismatch(got[:m], wants[b][which])
            assert (got[m] == np.uint64(2**64 - 1)).all()


@pytest.mark.parametrize("planes,m,k", [((3, 7), 128, 16383), ((3, 7), 40, 16352), ((4, 8), 40, 16383),
                                        ((4, 8), 128, 16352), ((2, 7), 113, 16383), ((2, 7), 128, 16352)])
def test_longest_inner_dimension_on_the_tile_kernel(oracle, planes, m, k):
    """512 and 511 k-blocks, the int32 accumulators closest to their bound: shares 0 and t-1 and residues
    around q/2 give digits of the largest magnitude.  Sixteen problems, so that the tiles win."""
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    x_bits, q_bits = PLANES[planes]
    N, Ch, problems = 64, 9, 16
    n = Ch * N
    moduli = ci.limb_primes(q_bits, 14, 1)
    q = moduli[0]
    route = _tile_route(nc, m, k, x_bits, n, N, moduli, True, problems, planes, m == 128)
    print(f"[tile rows] m={m} k={k}: {route}", flush=True)
    X = ci.gen_X(6400 + m, m, k, x_bits)
    X[0, :] = 0
    X[1, :] = X[-1, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(6400 + m, k, Ch, moduli, N)
    for col, value in enumerate(((q - 1) // 2, (q - 1) // 2 + 1, q - 1, 0)):
        ctW[:, 0, :, 0, col] = value
        ctW[:, -1, :, 0, N - 1 - col] = value
    plain = oracle.cop_ref(X, ctW, moduli, n, N, None)[0]
    prepared = gu.prepare(ctW, moduli, n, N)
    staged = torch.empty(nc.nimbus_cop_workspace_bytes(m, k, x_bits), dtype=torch.uint8, device="cuda")
    nc.nimbus_cop_stage_shares(gu.dev(X), m, k, x_bits, staged)
    masks = [ci.gen_mask_uniform(6500 + m + b, m, Ch, moduli, N) for b in range(problems)]
    outs = [torch.full((m, Ch, 2, 1, N), -1, dtype=torch.int64, device="cuda") for _ in range(problems)]
    nc.nimbus_cop_matmul_staged_batch([staged] * problems, m, k, x_bits, [prepared] * problems, n, N, 1, moduli,
                                      [gu.dev(mask) for mask in masks], outs)
    torch.cuda.synchronize()
    for b in range(problems):
        got, want = gu.host(outs[b]), (plain + masks[b]) % np.uint64(q)
        assert np.array_equal(got, want), f"problem {b}: " + gu.first_mismatch(got, want)
