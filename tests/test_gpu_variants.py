"""Every instance of the tile kernel by name: the route of the call is asked first, so that a change of the
dispatch cannot take a size away from the instance it is there for.  Every output word against the
oracle."""
import numpy as np
import pytest

import cop_inputs as ci

pytestmark = pytest.mark.gpu

# share and ciphertext planes: the widths that give them
PLANES = {(2, 7): (16, 50), (3, 7): (20, 54), (4, 7): (32, 54), (2, 8): (16, 62), (3, 8): (24, 62), (4, 8): (32, 62)}
MASK_AHEAD = [(2, 7), (3, 7), (2, 8)]           # nine accumulators at most: the mask words fit next to them
# rows, columns of one problem and of each of two, inner dimension, mask; (no row tests, mask words ahead,
# several row blocks) and rows of a block.  More than 256 blocks of 64 rows, but for the last form.
FORMS = {
    "full": (128, 8320, 4224, 70, True, (True, True, False), 128),
    "full, no mask": (128, 8320, 4224, 417, False, (True, False, False), 128),
    "full, long": (128, 8320, 4224, 417, True, (True, True, False), 128),
    "full, long, odd": (128, 8320, 4224, 450, True, (True, True, False), 128),
    "two full blocks": (256, 4224, 2176, 70, True, (True, True, True), 128),
    "two full blocks, no mask": (256, 4224, 2176, 70, False, (True, False, True), 128),
    "two full blocks, long": (256, 4224, 2176, 448, True, (True, True, True), 128),
    "rows": (40, 256, 256, 100, True, (False, False, False), 128),
    "rows, two blocks": (130, 5504, 2816, 100, True, (False, False, True), 128),
    "blocks of 64": (128, 1024, 1024, 270, True, (False, False, True), 64),
}
CASES = [(form, planes, problems) for form in FORMS for planes in PLANES for problems in (1, 2)]


@pytest.mark.parametrize("form,planes,problems", CASES)
def test_every_instance_of_the_tile_kernel(oracle, form, planes, problems):
    import torch
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    m, alone, each, k, masked, flags, block = FORMS[form]
    C = alone if problems == 1 else each
    x_bits, q_bits = PLANES[planes]
    full, ahead, shared = flags
    ahead = ahead and planes in MASK_AHEAD
    N, L = 64, 1
    n = C // (2 * N) * N
    moduli = ci.limb_primes(q_bits, 14, L)
    route = nc.nimbus_route_matmul(m, k, x_bits, n, N, L, moduli, masked=masked, staged=True, count=problems)
    flag = lambda b: "true" if b else "false"
    tiles = C // 64 * -(-m // block) * problems
    assert route == [f"cop_mfma_kernel<{planes[0]}, {planes[1]}, {flag(full)}, {flag(ahead)}, {flag(shared)}, "
                     f"{1 if problems == 1 else 16}> grid={min(tiles, 256)},1 block=512"]
    print(f"[variants] {form} x {problems}: {route[0]}", flush=True)
    staged, prepared, masks, outs, wants = [], [], [], [], []
    for b in range(problems):
        seed = 5000 + 10 * (m + k + sum(planes)) + b
        X = ci.gen_X(seed, m, k, x_bits)
        X[0, :] = X[-1, :] = (1 << x_bits) - 1
        ctW = ci.gen_ctW_uniform(seed, k, C // (2 * N), moduli, N)
        ctW[:, 0, :, 0, :4] = moduli[0] - 1
        mask = ci.gen_mask_uniform(seed, m, C // (2 * N), moduli, N) if masked else None
        if masked:
            mask[0, 0, :, 0, :4] = moduli[0] - 1
        wants.append(oracle.cop_ref(X, ctW, moduli, n, N, mask)[0])
        staged.append(torch.empty(nc.nimbus_cop_workspace_bytes(m, k, x_bits), dtype=torch.uint8, device="cuda"))
        nc.nimbus_cop_stage_shares(gu.dev(X), m, k, x_bits, staged[-1])
        prepared.append(gu.prepare(ctW, moduli, n, N))
        masks.append(gu.dev(mask) if masked else None)
        outs.append(torch.full((m, C), -1, dtype=torch.int64, device="cuda"))
    if problems == 1:
        nc.nimbus_cop_matmul_staged(staged[0], m, k, x_bits, prepared[0], n, N, L, moduli, masks[0], outs[0])
    else:
        nc.nimbus_cop_matmul_staged_batch(staged, m, k, x_bits, prepared, n, N, L, moduli,
                                          masks if masked else None, outs)
    for b in range(problems):
        got = gu.host(outs[b]).reshape(wants[b].shape)
        assert np.array_equal(got, wants[b]), f"problem {b}: " + gu.first_mismatch(got, wants[b])


# m, k, N, x_bits, and the instances of the passes over the upper and the lower halves: full row blocks on
# the paper's ring degree and limbs, the same with an upper half of two planes, with row tests, in
# blocks of 64 rows, and few rows
@pytest.mark.parametrize("m,k,N,x_bits,upper,lower", [
    (128, 70, 8192, 64, "cop_mfma_kernel<4, 8, true, false, false, 1>", "cop_mfma_kernel<4, 8, true, false, false, 1>"),
    (128, 417, 4096, 40, "cop_mfma_kernel<2, 8, true, false, false, 1>", "cop_mfma_kernel<4, 8, true, false, false, 1>"),
    (256, 64, 2048, 56, "cop_mfma_kernel<3, 8, true, false, true, 1>", "cop_mfma_kernel<4, 8, true, false, true, 1>"),
    (200, 100, 2048, 64, "cop_mfma_kernel<4, 8, false, false, true, 1>", "cop_mfma_kernel<4, 8, false, false, true, 1>"),
    (128, 64, 64, 64, "cop_mfma_kernel<4, 8, false, false, true, 1>", "cop_mfma_kernel<4, 8, false, false, true, 1>"),
    (40, 64, 64, 33, "cop_mfma_kernel<2, 8, false, false, false, 1>", "cop_mfma_kernel<4, 8, false, false, false, 1>"),
    (20, 520, 64, 64, "cop_thin_kernel<4, 8, 2, (nimbus::ThinShares)0, 1>", "cop_thin_kernel<4, 8, 2, (nimbus::ThinShares)0, 1>"),
    (16, 64, 64, 48, "cop_thin_kernel<2, 8, 1, (nimbus::ThinShares)2, 1>", "cop_thin_kernel<4, 8, 1, (nimbus::ThinShares)2, 1>"),
])
def test_both_passes_of_wide_shares(oracle, m, k, N, x_bits, upper, lower):
    import gpu_util as gu
    import paper_2411_15707_amd as nc
    moduli = tuple(ci.limb_primes(b, 14, 1)[0] for b in (59, 55))
    route = nc.nimbus_route_matmul(m, k, x_bits, N, N, 2, moduli)
    assert [line.split(" grid")[0] for line in route if "planes" not in line] == [upper, lower]
    print(f"[variants] wide shares m={m} k={k} N={N} x_bits={x_bits}: {route[-1]}", flush=True)
    X = ci.gen_X(7700 + m, m, k, x_bits)
    X[0, :] = X[-1, :] = (1 << x_bits) - 1
    ctW = ci.gen_ctW_uniform(7700 + m, k, 1, moduli, N)
    mask = ci.gen_mask_uniform(7700 + m, m, 1, moduli, N)
    for l, q in enumerate(moduli):
        ctW[:, 0, :, l, :4] = q - 1
        mask[0, 0, :, l, :4] = q - 1
    prepared = gu.prepare(ctW, moduli, N, N)
    for msk in (mask, None):
        want, _ = oracle.cop_ref(X, ctW, moduli, N, N, msk, wide=True)
        got = gu.run_mfma(X, ctW, moduli, N, N, x_bits, msk, prepared=prepared)
        assert np.array_equal(got, want), gu.first_mismatch(got, want)
