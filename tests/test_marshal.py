"""The native marshalling of binding.py's calls: what it takes runs as the general path does, anything else is left to that."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

from paper_2502_08145_amd import binding as B

M, N, K = 96, 72, 136


def _is_left(call, *args):
    B.lib()
    return call(*args) is None


@pytest.mark.parametrize("at,value", [(0, 0), (0, None), (1, 8.0), (1, np.int64(8)), (1, True), (1, 1 << 70), (4, "XX"), (4, b"NN"), (4, 1 << 40),
                                      (5, None), (5, 4096), (5, torch.zeros(8, 8)), (5, torch.zeros(8, 8, dtype=torch.bfloat16)),
                                      (5, torch.nn.Parameter(torch.zeros(8, 8, dtype=torch.bfloat16))), (8, True), (8, 1.0), (9, "stream"), (9, 1 << 80)])
def test_other_arguments_are_left_to_the_general_path(at, value):
    """Nothing runs: the entry point's address is not followed (the tensors are not on a device)."""
    cpu = torch.zeros(8, 8, dtype=torch.bfloat16)
    args = [B._fwd_at, 8, 8, 8, "NN", cpu, cpu, cpu, 1, 0]
    args[at] = value
    assert _is_left(B._gemm, *args) and _is_left(B._gemm, *args[:-1]) and _is_left(B._gemm, *args, 0)
    assert _is_left(B._transpose, B._transpose_at, 8, 8, cpu, cpu, 0) and _is_left(B._tuned, B._tuned_at, "fwd", 8, 8, 8, cpu, cpu, cpu, None, 1, 0)


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
        B._gemm(ctypes.cast(lib.gemm, ctypes.c_void_p).value, 8, 8, 8, "NN", t[0], t[1], t[2], 1, 0)
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
