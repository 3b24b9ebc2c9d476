"""The entry points called without ctypes (csrc/calls.cpp): they answer None for every call that is not the
ordinary one, before anything is launched, and the binding then refuses or accepts it as ever."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import cop_inputs as ci
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


# ---- every check of every call, with tensors on the GPU; the entry points behind it are callbacks here, which
# note their arguments and launch nothing ----
NOTED = 77                                              # their status
ENTRIES = ("nimbus_cop_matmul", "nimbus_cop_prepare", "nimbus_cop_workspace_bytes", "nimbus_cop_matmul_prepared",
           "nimbus_cop_stage_shares_batch", "nimbus_cop_matmul_staged_batch", "nimbus_cop_packed_count",
           "nimbus_cop_pack", "nimbus_rlwe_decrypt", "nimbus_rlwe_encrypt")
# arguments that are arrays of 64-bit words on the host: their places and lengths
ARRAYS = {"nimbus_cop_matmul": {8: 2}, "nimbus_cop_prepare": {5: 2}, "nimbus_cop_matmul_prepared": {8: 2},
          "nimbus_cop_stage_shares_batch": {1: 3, 5: 3}, "nimbus_cop_matmul_staged_batch": {1: 3, 5: 3, 9: 2, 10: 3, 11: 3},
          "nimbus_cop_pack": {5: 2}, "nimbus_rlwe_decrypt": {4: 2}, "nimbus_rlwe_encrypt": {6: 2}}
DEVICE = "cuda"


@pytest.fixture
def noted(monkeypatch):
    """a list of (entry point, its arguments) in the place of the launches"""
    lib, calls, keep = nc.load_library(), [], []
    for name in ENTRIES:
        real = getattr(lib, name)
        if name in ("nimbus_cop_workspace_bytes", "nimbus_cop_packed_count"):      # (asked on the host)
            keep.append(real)
            continue

        def note(*args, name=name):
            calls.append([name] + [list((ctypes.c_uint64 * ARRAYS[name][i]).from_address(arg)) if arg and i in ARRAYS[name] else arg
                                   for i, arg in enumerate(args)])
            return NOTED
        keep.append(ctypes.CFUNCTYPE(ctypes.c_int, *real.argtypes)(note))
    binding._calls.bind(tuple(ctypes.cast(f, ctypes.c_void_p).value for f in keep), lambda: 0, lambda device: 4321)
    yield calls
    monkeypatch.setattr(binding, "_lib", None)
    nc.load_library()                                   # (the library's own addresses again)


def _gpu_arguments(name):
    """(arguments, places of the tensors: 'words', 'bytes' or 'error'; lists of them too); two limbs, three problems"""
    import torch
    words = lambda count: torch.zeros(count, dtype=torch.int64, device=DEVICE)
    raw = lambda: torch.zeros(1 << 14, dtype=torch.uint8, device=DEVICE)
    m, k, n, N, L, q = 4, 64, 40, 32, 2, ci.limb_primes(54, 20, 2)
    Ch = 2
    C = Ch * 2 * L * N
    return {
        "matmul": ([words(m * k), m, k, 20, words(k * C), n, N, L, q, words(m * C), words(m * C), 0],
                   {0: "words", 4: "words", 9: "words", 10: "words"}),
        "prepare": ([words(k * C), k, n, N, L, q, raw(), 0], {0: "words", 6: "bytes"}),
        "matmul_prepared": ([words(m * k), m, k, 20, raw(), n, N, L, q, words(m * C), words(m * C), raw(), 0],
                            {0: "words", 4: "bytes", 9: "words", 10: "words", 11: "bytes"}),
        "stage_shares_batch": ([[words(m * k) for _ in range(3)], m, k, 20, [raw() for _ in range(3)], 0],
                               {0: "words", 4: "bytes"}),
        "matmul_staged_batch": ([[raw() for _ in range(3)], m, k, 20, [raw() for _ in range(3)], n, N, L, q,
                                 [words(m * C) for _ in range(3)], [words(m * C) for _ in range(3)], 0],
                                {0: "bytes", 4: "bytes", 9: "words", 10: "words"}),
        "pack": ([words(m * 2 * L * N), m, 8, N, L, q, words(2 * L * N), words(2 * L * N), 0],
                 {0: "words", 6: "words", 7: "words"}),
        "decrypt": ([words(m * 2 * L * N), m, N, L, q, 20, raw(), words(m * L * N), words(m * N), 0],
                    {0: "words", 6: "bytes", 7: "words", 8: "words"}),
        "encrypt": ([words(k * n), k, n, 20, N, L, q, raw(), words(k * Ch * L * N),
                     torch.zeros(k * Ch * N, dtype=torch.int8, device=DEVICE), words(k * C), 0],
                    {0: "words", 7: "bytes", 8: "words", 9: "error", 10: "words"}),
    }[name]


def _unfit(t, kind):
    """tensors that may not stand in the place of t"""
    import torch
    yield "strided", torch.zeros(2 * t.numel(), dtype=t.dtype, device=t.device)[::2]
    yield "transposed", torch.zeros(2, t.numel() // 2, dtype=t.dtype, device=t.device).t()
    yield "in host memory", torch.zeros(t.numel(), dtype=t.dtype)
    if kind == "bytes":                                 # (any number of any size)
        return
    for count in (t.numel() - 1, t.numel() + 1, 2 * t.numel()):
        yield f"{count} elements", torch.zeros(count, dtype=t.dtype, device=t.device)
    for dtype in (torch.int32, torch.int16, torch.float32) + ((torch.int64,) if kind == "error" else (torch.uint8,)):
        yield str(dtype), torch.zeros(t.numel(), dtype=dtype, device=t.device)
        # as many bytes
        yield f"bytes as {dtype}", torch.zeros(t.numel() * t.element_size() // dtype.itemsize, dtype=dtype, device=t.device)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(_arguments()))
def test_no_unfit_tensor_reaches_an_entry_point(name, noted):
    call = getattr(binding._calls, name)
    args, tensors = _gpu_arguments(name)
    assert call(*args) == NOTED and len(noted) == 1     # (what is refused below is refused for the one change)

    def refused(i, other, what):
        assert call(*args[:i], other, *args[i + 1:]) is None, f"argument {i}: {what}"

    for i, kind in tensors.items():
        if not isinstance(args[i], list):
            for what, other in _unfit(args[i], kind):
                refused(i, other, what)
            continue
        for at in (0, 2):
            for what, other in _unfit(args[i][at], kind):
                refused(i, args[i][:at] + [other] + args[i][at + 1:], f"item {at}: {what}")
            refused(i, args[i][:at] + [None] + args[i][at + 1:], f"item {at}: None")
        for items in (args[i][:2], args[i] + args[i][:1], [], args[i] * 6):
            refused(i, items, f"{len(items)} items")
    for i, arg in enumerate(args):
        if isinstance(arg, int) and i < len(args) - 1:  # (the last one is the stream)
            for other in (0, -arg, 1 << 31, 1 << 70, float(arg), True, np.int64(arg), None):
                refused(i, other, other)
        if isinstance(arg, tuple):                      # the moduli, a word each of two limbs
            for other in ((), arg[:1], arg * 5, (arg[0], -1), (arg[0], 1 << 64), (arg[0], 2.0), (arg[0], np.uint64(arg[1])), None):
                refused(i, other, other)
    for other in (-1 << 70, 1 << 70, 1.0, "0", object()):
        refused(len(args) - 1, other, other)
    if name.endswith("_batch"):                         # more problems than a launch takes
        assert call(*[arg * 6 if isinstance(arg, list) else arg for arg in args]) is None
    if name == "matmul_staged_batch":                   # staged shares that cannot be of this shape
        room = nc.nimbus_cop_workspace_bytes(*args[1:4])
        for at in (0, 2):
            refused(0, args[0][:at] + [args[0][at][:room - 1]] + args[0][at + 1:], "a short item")
        assert call([t[:room] for t in args[0]], *args[1:]) == NOTED
        noted.pop()
    assert len(noted) == 1, noted


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(_arguments()))
def test_an_entry_point_receives_the_arguments(name, noted):
    """every address, size and number in its place; the current stream where none is given; no mask"""
    call = getattr(binding._calls, name)
    args, tensors = _gpu_arguments(name)
    masks = {"matmul": 9, "matmul_prepared": 9, "matmul_staged_batch": 9, "pack": 6}
    for stream, masked in ((5, True), (None, True), (0, False)):
        given = args[:-1] + [stream]
        if not masked and name in masks:
            given[masks[name]] = None
        assert call(*given) == NOTED
        want = [3] if name.endswith("_batch") else []   # (the number of problems comes first)
        for i, arg in enumerate(given[:-1]):
            if isinstance(arg, (list, tuple)):
                want.append([t if isinstance(t, int) else t.data_ptr() for t in arg])
            else:
                want.append(arg.data_ptr() if i in tensors and arg is not None else arg)
            if (name, i) in (("prepare", 6), ("matmul_prepared", 11), ("stage_shares_batch", 4)):
                want.append(1 << 14)                    # its size
        entry, *got = noted.pop()
        assert entry.endswith(name) and got == want + [4321 if stream is None else stream or None]


@pytest.mark.gpu
def test_the_smallest_workspace_of_a_batch_counts(noted):
    args, _ = _gpu_arguments("stage_shares_batch")
    for at in range(3):
        workspaces = [t[:100] if i == at else t for i, t in enumerate(args[4])]
        assert binding._calls.stage_shares_batch(*args[:4], workspaces, 0) == NOTED
        assert noted.pop()[1 + 6] == 100
