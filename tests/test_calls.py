"""The entry points called without ctypes (csrc/calls.cpp): they answer None for every call that is not the
ordinary one, before anything is launched, and the binding then refuses or accepts it as ever."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2411_15707_amd as nc
from paper_2411_15707_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _arguments():
    import torch
    words = lambda count: torch.zeros(count, dtype=torch.int64)
    raw = torch.zeros(1 << 20, dtype=torch.uint8)
    m, k, n, N, L, mod = 4, 64, 32, 32, 1, (ci_prime(),)
    C = 2 * L * N
    return {
        "matmul": (words(m * k), m, k, 20, words(k * C), n, N, L, mod, words(m * C), words(m * C), None),
        "prepare": (words(k * C), k, n, N, L, mod, raw, None),
        "matmul_prepared": (words(m * k), m, k, 20, raw, n, N, L, mod, None, words(m * C), raw, None),
        "stage_shares_batch": ([words(m * k)], m, k, 20, [raw], None),
        "matmul_staged_batch": ([raw], m, k, 20, [raw], n, N, L, mod, None, [words(m * C)], None),
        "pack": (words(m * C), m, 8, N, L, mod, words(C), words(C), None),
        "decrypt": (words(m * C), m, N, L, mod, 20, raw, words(m * N), words(m * N), None),
        "encrypt": (words(k * n), k, n, 20, N, L, mod, raw, words(k * N), torch.zeros(k * N, dtype=torch.int8), words(k * C), None),
    }


def ci_prime():
    import cop_inputs as ci
    return ci.limb_primes(54, 20, 1)[0]


@pytest.mark.parametrize("name", sorted(_arguments()))
def test_what_is_not_ordinary_is_left_to_the_binding(name):
    """tensors in host memory, other types and other numbers of arguments; every argument in turn replaced"""
    nc.load_library()
    call = getattr(binding._calls, name)
    args = _arguments()[name]
    assert call(*args) is None                          # (host memory)
    assert call() is None and call(*args[:-1]) is None and call(*args, None) is None
    for i in range(len(args)):
        for other in (None, 0, -1, 1 << 40, 2.5, "x", np.int64(4), True, [], [None] * 20, object()):
            assert call(*args[:i], other, *args[i + 1:]) is None, (i, other)


@pytest.mark.gpu
def test_the_binding_refuses_what_it_refused():
    import torch
    m, k, n, N, L, mod = 4, 64, 32, 32, 1, (ci_prime(),)
    C = 2 * L * N
    words = lambda count: torch.zeros(count, dtype=torch.int64, device="cuda")
    raw = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    good = dict(X=words(m * k), m=m, k=k, x_bits=20, prepared=raw, n=n, N=N, L=L, moduli=mod, mask=None, out=words(m * C),
                workspace=raw.clone())
    nc.nimbus_cop_matmul_prepared(**good)
    nc.nimbus_cop_matmul_prepared(**{**good, "moduli": [np.uint64(mod[0])]})    # not an int: the other way, accepted
    for change, error, text in (
            ({"X": words(m * k + 1)}, ValueError, "words, expected"), ({"X": words(2 * m * k)[::2]}, ValueError, "contiguous"),
            ({"out": words(m * C).to(torch.int32)}, ValueError, "64-bit"), ({"prepared": raw.cpu()}, ValueError, "on the GPU"),
            ({"X": None}, AttributeError, None), ({"k": 64.0}, Exception, None), ({"moduli": (4,)}, nc.NimbusCopError, "nimbus_cop_matmul_prepared"),
            ({"workspace": raw[:64]}, nc.NimbusCopError, "status -4"), ({"out": good["X"]}, nc.NimbusCopError, "status -1")):
        with pytest.raises(error, match=text):
            nc.nimbus_cop_matmul_prepared(**{**good, **change})
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        nc.nimbus_cop_matmul_prepared(**good)
    nc.nimbus_cop_matmul_prepared(**good, stream=side)
    nc.nimbus_cop_matmul_prepared(**good, stream=side.cuda_stream)
    torch.cuda.synchronize()


@pytest.mark.parametrize("missing", ["sys.modules['paper_2411_15707_amd._calls'] = None",
                                     "import types; sys.modules['paper_2411_15707_amd._calls'] = types.ModuleType('_calls')",
                                     "import torch; torch.__version__ = '1.0'"])
def test_without_the_native_module_calls_go_through_ctypes(missing):
    """not built, another file of that name, built for another torch: the library loads all the same, with a warning"""
    code = f"""
import sys, warnings
sys.path.insert(0, {ROOT!r})
import paper_2411_15707_amd as nc
from paper_2411_15707_amd import binding
{missing}
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    nc.load_library()
assert any("ctypes" in str(w.message) for w in seen), seen
assert nc.nimbus_cop_packed_count(8, 64, 1024) == 1
for name in {sorted(_arguments())!r}:
    assert getattr(binding._calls, name)() is None
import torch
try:
    nc.nimbus_cop_prepare(torch.zeros(4096, dtype=torch.int64), 64, 32, 32, 1, ({ci_prime()},), torch.zeros(1 << 20, dtype=torch.uint8))
except ValueError as e:
    assert "on the GPU" in str(e)
else:
    raise AssertionError("host memory accepted")
"""
    done = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr


def test_the_native_module_is_there():
    """built with the library, for this interpreter and this torch"""
    import torch
    nc.load_library()
    assert not isinstance(binding._calls, binding._NoCalls)
    assert binding._calls.torch_version == torch.__version__
