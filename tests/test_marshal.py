"""The native marshalling of binding.py's calls: what it takes runs as the general path does, anything else is left to that."""
import ctypes
import importlib.util
import subprocess

import numpy as np
import pytest
import torch

from paper_2502_08145_amd import binding as B

M, N, K = 96, 72, 136


I64, INT, PTR = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p
GEMM_T = ctypes.CFUNCTYPE(INT, I64, I64, I64, INT, PTR, PTR, PTR, INT, PTR)
TUNED_T = ctypes.CFUNCTYPE(INT, INT, I64, I64, I64, PTR, PTR, PTR, PTR, PTR, ctypes.c_size_t, INT, PTR, ctypes.POINTER(INT))
TRANSPOSE_T = ctypes.CFUNCTYPE(INT, I64, I64, PTR, PTR, PTR)
# what one place takes no other of: (place's kind, values that are left to the general path)
LEFT = {"entry": [0, None, 1.0], "size": [8.0, np.int64(8), True, 1 << 70, "8"], "name": ["XX", b"NN", 1 << 40, None, 1.0],
        "flag": [True, 1.0, 1 << 40], "stream": ["stream", 1 << 80, True, 1.0]}


def test_tensors_off_the_device_are_left_to_the_general_path():
    """Nothing runs: the entry points' addresses are not followed."""
    B.lib()
    cpu = torch.zeros(8, 8, dtype=torch.bfloat16)
    assert B._gemm(B._fwd_at, 8, 8, 8, "NN", cpu, cpu, cpu, 1, 0) is None
    assert B._tuned(B._tuned_at, "fwd", 8, 8, 8, cpu, cpu, cpu, None, 1, 0) is None
    assert B._transpose(B._transpose_at, 8, 8, cpu, cpu, 0) is None


class Tagged(torch.Tensor):
    pass


def _calls(t, entry):
    """(function, its C type, arguments that it takes, the kind of each, what the entry point then gets)."""
    x, y, z = (t[i] for i in range(3))
    p, q, r = (i.data_ptr() for i in (x, y, z))
    return [(B._gemm, GEMM_T, [entry, 8, 9, 10, "NT", x, y, z, 1, 77], "entry size size size name tensor tensor tensor flag stream", (8, 9, 10, 1, p, q, r, 1, 77)),
            (B._tuned, TUNED_T, [entry, "bwd_weight", 8, 9, 10, x, y, z, x, 1, 77], "entry name size size size tensor tensor tensor tensor flag stream",
             (2, 8, 9, 10, p, q, r, p, None, 0, 1, 77)),
            (B._transpose, TRANSPOSE_T, [entry, 8, 9, x, y, 77], "entry size size tensor tensor stream", (8, 9, p, q, 77))]


@pytest.mark.gpu
@pytest.mark.parametrize("which", [0, 1, 2])
def test_only_plain_arguments_reach_the_entry_point(which):
    """With an entry point that records its calls: the arguments as they stand reach it, and not with any one of them of another kind."""
    B.lib()
    seen = []
    t = torch.zeros(3, 8, 8, dtype=torch.bfloat16, device="cuda")
    _, ctype, *_ = _calls(t, 1)[which]
    record = ctype(lambda *args: seen.append(args) or -7)
    call, _, args, kinds, want = _calls(t, ctypes.cast(record, PTR).value)[which]
    assert call(*args) == -7 and len(seen) == 1 and seen[0][:len(want)] == want
    left = {**LEFT, "tensor": [4096, t[0].cpu(), t[0].float(), t[0].as_subclass(Tagged), t[0].t()[:, :4], "x"] + ([] if which == 1 else [None])}
    for i, kind in enumerate(kinds.split()):
        for value in left[kind]:
            assert call(*args[:i], value, *args[i + 1:]) is None, (i, value)
    assert call(*args[:-1]) is None and call(*args, 0) is None
    if which == 1:
        for i in (5, 6, 7):
            assert call(*args[:i], None, *args[i + 1:]) is None
    assert len(seen) == 1
    i = kinds.split().index("tensor")   # a parameter is a plain tensor
    assert call(*args[:i], torch.nn.Parameter(args[i]), *args[i + 1:]) == -7 and seen[-1][:len(want)] == want
    # no stream: the current one.  Names and numbers are the same.
    assert call(*args[:-1], None) == -7 and (seen[-1][8 if which == 0 else 11 if which == 1 else 4] or 0) == torch.cuda.current_stream().cuda_stream
    if which < 2:
        i = kinds.split().index("name")
        assert call(*args[:i], want[3 if which == 0 else 0], *args[i + 1:]) == -7 and seen[-1][:len(want)] == want
    if which == 1:   # the re-stored operand is optional
        assert call(*args[:8], None, *args[9:]) == -7 and seen[-1][7] is None


@pytest.mark.gpu
def test_an_exception_out_of_the_entry_point_is_raised_once(tmp_path):
    """It becomes a Python error, with the interpreter held again, and the call does not go the general way a second time."""
    src, so = tmp_path / "throws.cpp", str(tmp_path / "throws.so")
    src.write_text('#include <stdexcept>\n#include <stdint.h>\nstatic int n = 0;\nextern "C" int calls() { return n; }\n'
                   'extern "C" int gemm(int64_t, int64_t, int64_t, int, const void*, const void*, void*, int, void*) { ++n; throw std::runtime_error("no room"); }\n')
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    t = torch.zeros(3, 8, 8, dtype=torch.bfloat16, device="cuda")
    B.lib()
    with pytest.raises(RuntimeError, match="no room"):
        B._gemm(ctypes.cast(lib.gemm, PTR).value, 8, 8, 8, "NN", t[0], t[1], t[2], 1, 0)
    assert lib.calls() == 1


def _operands():
    gen = torch.Generator(device="cuda").manual_seed(3)
    return [torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16) for s in ((M, K), (K, N))] + [torch.empty((M, N), dtype=torch.bfloat16, device="cuda")]


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["axonn_linear_fwd", "axonn_linear_bwd_data", "axonn_linear_bwd_weight", "axonn_linear_gemm_static"])
def test_both_paths_run_the_same_call(entry):
    x, y, c = _operands()
    call = getattr(B, entry)
    call(M, N, K, "NN", x, y, c)
    want = c.clone()
    for args, kw in (((M, N, K, 0, x, y, c), {}), ((np.int64(M), N, K, "NN", x, y, c), {}), ((M, N, K, "NN", x.data_ptr(), y.data_ptr(), c.data_ptr()), {}),
                     ((M, N, K, "NN", x, y, c), dict(fp32_accumulate=0)), ((M, N, K, "NN", x, y, c), dict(stream=torch.cuda.current_stream())),
                     ((M, N, K, "NN", torch.nn.Parameter(x), y, c), {})):
        c.zero_()
        assert call(*args, **kw) == B.AXONN_OK
        torch.cuda.synchronize()
        assert torch.equal(c, want), (args[:4], kw)
    for bad in ((M, N, K, 3, x, y, c), (-1, N, K, "NN", x, y, c)):
        assert call(*bad, check=False) == B.AXONN_ERR_INVALID_ARG
        with pytest.raises(B.AxonnError):
            call(*bad)
    with pytest.raises(TypeError):
        call(M, N, K, "NN", x.t(), y, c)
    with pytest.raises(TypeError):
        call(M, N, K, "NN", x.float(), y, c)


@pytest.mark.gpu
def test_the_current_stream_is_the_one_that_is_current_at_the_call():
    """A product behind a long wait on a side stream: it is not done when the default stream is."""
    x, y, c = _operands()
    B.axonn_linear_fwd(M, N, K, "NN", x, y, c)
    want = c.clone()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)
        c.zero_()
        B.axonn_linear_fwd(M, N, K, "NN", x, y, c)
        done = side.record_event()
    assert not done.query()
    side.synchronize()
    assert torch.equal(c, want)


@pytest.mark.gpu
def test_tuned_calls_and_transposes():
    x, y, c = _operands()
    t = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    assert B.axonn_transpose_bf16(K, N, y, t) == B.AXONN_OK and torch.equal(t, y.t())
    assert B.axonn_transpose_bf16(K, N, y, y, check=False) == B.AXONN_ERR_INVALID_ARG
    B.axonn_linear_fwd(M, N, K, "NN", x, y, c)
    want = c.clone()
    B.axonn_linear_tuned_set("fwd", M, N, K, "NT")
    try:
        for op in ("fwd", 0):
            c.zero_()
            assert B.axonn_linear_tuned_call(op, M, N, K, x, y, c, t) == B.AXONN_NT
            torch.cuda.synchronize()
            assert (c.float() - want.float()).norm() <= 4e-3 * want.float().norm()   # two roundings to bf16 apart at most
        # no room to re-store the operand: the natural mode
        assert B.axonn_linear_tuned_call("fwd", M, N, K, x, y, c) == B.AXONN_NN
    finally:
        B.axonn_linear_tune_reset()
    assert B.axonn_linear_tuned_call("fwd", M, -1, K, x, y, c, check=False) == B.AXONN_ERR_INVALID_ARG


def test_the_extension_is_there():
    B.lib()
    assert type(B._gemm) is type(B._tuned) is type(B._transpose) is type(len)


@pytest.mark.parametrize("why", ["missing", "unreadable", "another torch"])
def test_without_the_extension_every_call_takes_the_general_path(why, tmp_path, monkeypatch):
    """Queries, addresses and errors as with it, and a warning."""
    spec = importlib.util.spec_from_file_location("binding_alone", B.__file__)
    alone = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(alone)
    if why == "another torch":
        monkeypatch.setattr(torch, "__version__", "0.0")
    else:
        alone.MARSHAL_PATH = str(tmp_path / "axonn_marshal.so")
    if why == "unreadable":
        (tmp_path / "axonn_marshal.so").write_bytes(b"not a library")
    with pytest.warns(RuntimeWarning, match="in Python"):
        alone.lib()
    assert alone.kernel_name(1024, 3072, 3072, "NT") == B.kernel_name(1024, 3072, 3072, "NT")
    assert alone.axonn_linear_fwd(0, 8, 8, "NT", 0, 0, 0, stream=0) == B.AXONN_OK
    with pytest.raises(alone.AxonnError):
        alone.axonn_linear_fwd(8, 8, 8, "NN", 0, 0, 0, stream=0)
    with pytest.raises(TypeError):
        alone.axonn_linear_fwd(8, 8, 8, "NN", torch.zeros(8, 8), 0, 0, stream=0)
