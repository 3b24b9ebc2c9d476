"""Which kernels a call launches, asked of the dispatch on the host (include/nimbus_route.h)."""
import ctypes
import os
import re

import pytest

import cop_inputs as ci
import paper_2411_15707_amd as nc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LINE = re.compile(r"(\w+)<([^>]*)> grid=(\d+),(\d+) block=(\d+)$")


def moduli_of(q_bits, L):
    return ci.limb_primes(q_bits, 14, L)


def test_header_binding_and_argument_checks():
    text = open(os.path.join(ROOT, "include", "nimbus_route.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = sorted(set(re.findall(r"\b(nimbus_route_\w+)\s*\(", text)))
    assert declared == sorted(nc.ROUTE_SYMBOLS)
    lib = nc.load_library()
    for name in declared:
        assert hasattr(lib, name), name
    mods = moduli_of(54, 1)
    with pytest.raises(nc.NimbusCopError) as e:
        nc.nimbus_route_prepare(0, 32, 32, 1, mods)
    assert e.value.status == -1
    with pytest.raises(nc.NimbusCopError) as e:
        nc.nimbus_route_matmul(4, 50000, 20, 32, 32, 1, mods)       # k beyond the accumulators' bound
    assert e.value.status == -2
    with pytest.raises(nc.NimbusCopError) as e:
        nc.nimbus_route_matmul(4, 64, 20, 32, 32, 1, mods, count=2)     # a batch is staged
    assert e.value.status == -1
    with pytest.raises(nc.NimbusCopError) as e:
        nc.nimbus_route_matmul(4, 64, 40, 32, 32, 1, mods, staged=True, count=2)    # wide shares: no batch
    assert e.value.status == -2
    # a text longer than the buffer is cut off
    text = ctypes.create_string_buffer(b"x" * 40)
    mod = (ctypes.c_uint64 * 1)(*mods)
    assert lib.nimbus_route_matmul(0, 1, 64, 768, 20, 32, 32, 1, mod, 1, 0, text, 20) == 0
    assert len(text.value) == 19 and text.raw[20:40] == b"x" * 20


def test_every_launch_of_a_call_is_named():
    """a BERT-base up-projection: one staging and one product kernel, the second alone when staged"""
    cfg = ci.CONFIGS[3]
    lines = nc.nimbus_route_matmul(cfg.m, cfg.k, cfg.t_bits, cfg.n, cfg.N, cfg.L, cfg.moduli)
    assert [LINE.match(x).group(1) for x in lines] == ["x_planes_kernel", "cop_mfma_kernel"]
    assert lines[1] == "cop_mfma_kernel<3, 7, true, true, false, 1> grid=256,1 block=512"
    assert nc.nimbus_route_matmul(cfg.m, cfg.k, cfg.t_bits, cfg.n, cfg.N, cfg.L, cfg.moduli, staged=True) == lines[1:]
    assert LINE.match(nc.nimbus_route_prepare(cfg.k, cfg.n, cfg.N, cfg.L, cfg.moduli)[0]).group(1) == "prepare_kernel"
    # shares of two halves: a pass for each
    assert len(nc.nimbus_route_matmul(cfg.m, cfg.k, 64, cfg.n, cfg.N, cfg.L, cfg.moduli, staged=True)) == 2


def test_every_launch_of_the_setup_has_fewer_than_2_to_32_threads():
    """the runtime refuses larger ones: 2^29 columns of one row (124 GB of planes) are a size that fits
    the device's memory"""
    for q_bits, k, n, N, L in [(54, 1, 2**28, 65536, 1), (62, 1, 2**28 + 1, 65536, 1), (54, 32, 2**28, 65536, 1),
                               (54, 33, 2**28, 65536, 1), (54, 96, 2**27, 65536, 2), (54, 31, 4096, 4096, 1),
                               (54, 97, 4096, 4096, 1), (54, 511, 4096, 4096, 1), (54, 768, 2**20, 65536, 4)]:
        line = LINE.match(nc.nimbus_route_prepare(k, n, N, L, ci.limb_primes(q_bits, 17, L))[0])
        blocks, threads = int(line.group(3)), int(line.group(5))
        assert blocks * threads < 2**32, (line.group(0), k, n, N, L)
        assert blocks == -(-n // N) * 2 * L * N // 32 and int(line.group(4)) == 1


def test_slices_of_few_rows_follow_the_compute_units():
    """a wave per 16 columns and slice, eight to a workgroup: 512 column groups are four slices on 256
    compute units, eight where there are twice as many, two on half of them and none on a quarter"""
    mods = moduli_of(54, 2)
    for units, blocks in ((64, 64), (128, 128), (256, 256), (512, 512)):
        line = nc.nimbus_route_matmul(1, 3072, 20, 2048, 2048, 2, mods, staged=True, units=units)[0]
        assert line.startswith("cop_thin_kernel") and f"grid={blocks},1 " in line, (units, line)


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("m", [1, 16, 32])
def test_every_launch_of_few_rows_has_fewer_than_2_to_32_threads(m, staged):
    """a row on 2^30 columns: 240 GB of planes, within the device's memory"""
    for n in (2**28, 2**29 - 65536, 2**29, 2**30 - 65536):
        for line in nc.nimbus_route_matmul(m, 1, 20, n, 65536, 1, ci.limb_primes(54, 20, 1), staged=staged):
            line = LINE.match(line)
            assert int(line.group(3)) * int(line.group(5)) < 2**32, (n, line.group(0))


def kernels(lines):
    return [LINE.match(x).group(1) for x in lines]


# m, k, C, x_bits, problems, and the kernel from staged shares (us on 256 compute units, the kernel for few rows /
# the tiles, 54-bit moduli: 5.1 / 4.4, 7.8 / 4.8, 4.7 / 5.0, 9.1 / 5.9, 20.2 / 19.7, 32.4 / 26.3, 23.2 / 17.7, 9.2 / 9.1,
# 8.9 / 5.8, 253 / 197, 6.9 / 8.5, 16.7 / 15.5, 18.7 / 17.7, 19.0 / 18.0; 30.3 / 38.5, 7.9 / 10.3, 89.7 / 75.8,
# 31.6 / 42.5).  Held is what the rule chooses: the faster one but for 1 x 128 x 256 and 16 x 64 x 20480, which its
# margin for a single call of up to 16 rows leaves with the tiles, and 32 x 2032 x 16384 twice, where both
# estimates are off (62-bit moduli, an older tile kernel: 98.1 / 134.0).
@pytest.mark.parametrize("m,k,C,x_bits,count,kernel", [
    (16, 32, 4096, 20, 1, "cop_mfma_kernel"), (32, 32, 4096, 20, 1, "cop_mfma_kernel"),
    (1, 128, 256, 20, 1, "cop_mfma_kernel"), (32, 64, 8192, 20, 1, "cop_mfma_kernel"),
    (16, 32, 131072, 20, 1, "cop_mfma_kernel"), (32, 32, 131072, 20, 1, "cop_mfma_kernel"),
    (32, 128, 49152, 20, 1, "cop_mfma_kernel"), (16, 256, 16384, 20, 1, "cop_mfma_kernel"),
    (24, 32, 4096, 20, 4, "cop_mfma_kernel"), (24, 64, 262144, 20, 4, "cop_mfma_kernel"),
    (16, 64, 20480, 20, 1, "cop_mfma_kernel"), (32, 256, 24576, 20, 1, "cop_mfma_kernel"),
    (1, 768, 16384, 20, 1, "cop_mfma_kernel"), (16, 768, 16384, 20, 1, "cop_mfma_kernel"),
    (1, 3072, 8192, 20, 1, "cop_thin_kernel"),
    (32, 512, 4096, 20, 1, "cop_thin_kernel"), (32, 2032, 16384, 32, 2, "cop_thin_kernel"),
    (4, 2097, 2944, 32, 3, "cop_thin_kernel"),
])
def test_which_kernel_few_rows_take(m, k, C, x_bits, count, kernel):
    n = C // 4                                      # (two limbs)
    N = min(4096, n & -n)                           # the power of two in it
    lines = nc.nimbus_route_matmul(m, k, x_bits, n, N, 2, moduli_of(54, 2), staged=True, count=count, units=256)
    assert kernels(lines) == [kernel]


# 33 rows and more on few columns, k-blocks and the kernel (us, the kernel for few rows / the tiles, 54-bit moduli, 64 x
# 1024 columns and 20-bit shares by k-blocks: 6.3 / 7.0, 6.9 / 7.5, 6.9 / 7.7, 6.4 / 8.8, 6.3 / 9.1, 6.9 / 9.6, 6.5 / 9.8;
# 256 x 2048 and 32-bit shares: 10.0 / 11.0, 10.7 / 11.7).  Under five k-blocks always the tiles, from five to nine only
# where this kernel is well ahead by the estimates
@pytest.mark.parametrize("m,C,x_bits,kernels_at", [
    (64, 1024, 20, {1: "mfma", 4: "mfma", 5: "mfma", 6: "mfma", 7: "thin", 8: "thin", 9: "mfma", 10: "thin", 11: "thin"}),
    (256, 2048, 32, {8: "mfma", 9: "mfma", 10: "thin"}),
    (128, 256, 32, {4: "mfma", 7: "thin", 9: "thin", 10: "thin"}),
])
def test_which_kernel_more_rows_take_by_k_blocks(m, C, x_bits, kernels_at):
    for k_blocks, kernel in kernels_at.items():
        for k in (32 * k_blocks - 31, 32 * k_blocks):
            lines = nc.nimbus_route_matmul(m, k, x_bits, C // 2, C // 2, 1, moduli_of(54, 1), staged=True, units=256)
            assert kernels(lines) == [f"cop_{kernel}_kernel"], (k_blocks, k)


# 17 to 32 rows from the shares themselves: split in the kernel, or staged and one kernel or the other (us, split
# in the kernel / staged: 7.6 / 8.8, 8.2 / 10.6, 23.8 / 19.1; the kernel for few rows / the tiles: 61.8 / 55.7,
# 39.1 / 43.8)
@pytest.mark.parametrize("m,k,C,x_bits,launched", [
    (24, 82, 2048, 32, ["cop_thin_kernel"]), (20, 200, 8192, 20, ["cop_thin_kernel"]),
    (31, 610, 16384, 24, ["x_planes_kernel", "cop_mfma_kernel"]),
    (31, 1329, 32768, 24, ["x_planes_kernel", "cop_mfma_kernel"]),
    (24, 987, 24576, 32, ["x_planes_kernel", "cop_thin_kernel"]),
])
def test_17_to_32_rows_take_the_faster_way(m, k, C, x_bits, launched):
    n = C // 4                                      # (two limbs)
    lines = nc.nimbus_route_matmul(m, k, x_bits, n, n & -n, 2, moduli_of(54, 2), units=256)
    assert kernels(lines) == launched


# m, k, C, and the kernels from the shares themselves (us, split in the kernel / staged and tiles, replayed from
# a graph: 31.7 / 18.1, 52.6 / 44.3; one launch where a call takes little more than that)
@pytest.mark.parametrize("m,k,C,x_bits,q_bits,expected", [
    (6, 16, 107520, 16, 62, ["x_planes_kernel", "cop_mfma_kernel"]),
    (14, 748, 39552, 20, 54, ["x_planes_kernel", "cop_mfma_kernel"]),
    (1, 768, 16384, 20, 54, ["cop_thin_kernel"]), (8, 32, 4096, 20, 54, ["cop_thin_kernel"]),
    (4, 2097, 49152, 32, 62, ["cop_thin_kernel"]),
])
def test_few_rows_from_the_shares_themselves(m, k, C, x_bits, q_bits, expected):
    n = C // 4
    N = min(4096, n & -n)
    assert kernels(nc.nimbus_route_matmul(m, k, x_bits, n, N, 2, moduli_of(q_bits, 2), units=256)) == expected
