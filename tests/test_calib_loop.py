"""The calibration's matrix-core loop holds matrix instructions and next to nothing else: its rate is read as
that of the instruction (compiled for the device only, no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2411_15707_amd import build as hip_build

CSRC = os.path.join(os.path.dirname(os.path.abspath(hip_build.__file__)), "csrc")


def test_matrix_core_loop_copies_nothing(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "calib.asm"
    subprocess.run([hipcc] + hip_build.HIPCC_FLAGS + ["--cuda-device-only", "-S", "-o", str(out),
                                                      os.path.join(CSRC, "calib.hip")],
                   check=True, stderr=subprocess.DEVNULL)
    text = out.read_text()
    start = re.search(r"^\S*calib_mfma_kernel\S*:", text, re.M).end()
    body = text[start:text.index("s_endpgm", start)]
    product = r"^\s*v_mfma_i32_16x16x64_i8\b"
    # basic blocks; the loop is the one with all 42 products
    loops = [b for b in re.split(r"^\.LBB\S+:", body, flags=re.M) if len(re.findall(product, b, re.M)) >= 42]
    assert len(loops) == 1
    loop = loops[0][:re.search(r"^\s*s_cbranch\S+", loops[0], re.M).start()]
    products = len(re.findall(product, loop, re.M))
    others = len(re.findall(r"^\s*v_(?!mfma)\w+", loop, re.M))
    assert products == 42
    assert others <= 4, f"{others} other vector instructions next to {products} products"
