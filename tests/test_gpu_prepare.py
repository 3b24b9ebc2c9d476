"""nimbus_cop_prepare against the layout its header states, word for word."""
import numpy as np
import pytest

import cop_inputs as ci
import paper_2411_15707_amd as nc

pytestmark = pytest.mark.gpu


def prepared_reference(ctW, moduli, N):
    """signed base-256 digits of the centred residues, [column tile][k block][plane][64 lanes][16],
    and the column sums (Python integers)"""
    k = ctW.shape[0]
    flat = ctW.reshape(k, -1)
    C = flat.shape[1]
    DQ = max(7, -(-(max(q.bit_length() for q in moduli) + 1) // 8))
    KB = -(-k // 32)
    q_of_col = np.array([moduli[(c // N) % len(moduli)] for c in range(C)], dtype=np.int64)
    r = np.zeros((KB * 32, C), dtype=np.int64)
    r[:k] = flat.astype(np.int64)
    r = np.where(r > (q_of_col - 1) // 2, r - q_of_col, r)
    planes = np.empty((DQ, KB * 32, C), dtype=np.int8)
    for d in range(DQ):
        digit = ((r + 128) & 255) - 128
        planes[d] = digit.astype(np.int8)
        r = (r - digit) >> 8
    assert not r.any()
    # k = 32 kb + 16 h + b, column = 32 ct + c  ->  [ct][kb][d][h][c][b]
    tiles = planes.reshape(DQ, KB, 2, 16, C // 32, 32).transpose(4, 1, 0, 2, 5, 3)
    sums = np.array([int(sum(int(v) for v in flat[:, c])) % int(q_of_col[c]) for c in range(C)], dtype=np.uint64)
    return np.ascontiguousarray(tiles).reshape(-1).view(np.uint8), sums


# k on both sides of a k-block (one wave per tile below it), of the sixteen k-blocks from which
# sixteen waves share a tile, and of two rounds of them; one column tile and several; both plane
# counts; tiles of two limbs
@pytest.mark.parametrize("k,n,N,L,q_bits", [
    (32, 96, 32, 2, 54), (17, 2048, 1024, 2, 59), (1, 32, 32, 1, 50), (31, 40, 32, 2, 54), (33, 64, 64, 1, 62), (480, 32, 32, 1, 54),
    (481, 32, 32, 2, 59), (512, 100, 64, 1, 50), (545, 32, 32, 1, 55), (1025, 64, 64, 1, 62),
])
def test_prepared_weights_have_the_documented_layout(k, n, N, L, q_bits):
    import gpu_util as gu
    moduli = ci.limb_primes(q_bits, 16, L)
    Ch = -(-n // N)
    ctW = ci.gen_ctW_uniform(900 + k, k, Ch, moduli, N)
    ctW[0, 0, 0, :, :4] = np.array([[0, (q - 1) // 2, (q - 1) // 2 + 1, q - 1] for q in moduli], dtype=np.uint64)
    ctW[:, 0, 1, :, 0] = np.array([q - 1 for q in moduli], dtype=np.uint64)      # largest column sum
    got = gu.prepare(ctW, moduli, n, N).cpu().numpy()
    tiles, sums = prepared_reference(ctW, moduli, N)
    assert got.size == tiles.size + 8 * sums.size
    assert np.array_equal(got[tiles.size:].view(np.uint64), sums)
    assert np.array_equal(got[:tiles.size], tiles)


# where the waves per tile and the columns per workgroup change: 4 / 5, 8 / 9, 16 / 17 k-blocks and an
# odd number of them (a workgroup of half a tile takes pairs); 128 column tiles, 132, 256, 264 and 1024
@pytest.mark.parametrize("k,n,N,L,q_bits", [
    (128, 32, 32, 1, 54), (129, 32, 32, 1, 62), (250, 64, 64, 2, 59), (257, 2048, 1024, 1, 54),
    (530, 33, 32, 1, 54), (1100, 64, 32, 2, 62), (160, 2048, 2048, 1, 54), (161, 2080, 32, 1, 54),
    (192, 4096, 4096, 1, 62), (200, 4200, 64, 1, 54), (300, 4096, 4096, 1, 59), (257, 16384, 8192, 1, 54),
])
def test_prepared_weights_where_the_split_changes(k, n, N, L, q_bits):
    test_prepared_weights_have_the_documented_layout(k, n, N, L, q_bits)
