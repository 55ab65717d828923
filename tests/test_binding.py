"""The native way through the binding (csrc/fa_binding.cpp) against the Python way: the same results, refusals and errors."""
import math
import os
import subprocess
import sys
import sysconfig

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2407_08608_amd import binding, build


def _both(monkeypatch, call):
    """What `call` returns or raises with the native part and without it."""
    seen = []
    for native in (binding._native, None):
        monkeypatch.setattr(binding, "_native", native)
        try:
            seen.append(call())
        except Exception as e:  # noqa: BLE001 - compared below
            seen.append(e)
    return seen


def _same_error(a, b):
    assert isinstance(a, Exception) and type(a) is type(b) and str(a) == str(b), (a, b)


@pytest.mark.skipif(not os.path.exists(build.BINDING), reason="the native part has not been built")
def test_the_native_part_is_taken_where_it_is_built():
    assert binding._native is not None


def test_the_library_is_built_without_a_compiler_for_the_native_part(monkeypatch, tmp_path, capsys):
    linked = []

    def run(command, **_):
        if command[0] == "no-such-compiler":
            raise FileNotFoundError(command[0])
        linked.append(command[-1])

    monkeypatch.setenv("CXX", "no-such-compiler")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build, "_check_hazards", lambda name: name)
    monkeypatch.setattr(build.subprocess, "run", run)
    assert build.build(verbose=False) == build.LIB
    assert linked and linked[0].endswith(".hip.o") and "no-such-compiler" in capsys.readouterr().err


@pytest.mark.skipif(binding._native is None, reason="the native part has not been built")
def test_the_native_part_is_for_this_python_and_this_torch_only():
    assert binding._native.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    code = ("import torch; torch.__version__ = '0.0'\n"
            "from paper_2407_08608_amd import binding; assert binding._native is None\n"
            "try:\n    from paper_2407_08608_amd import _fa_binding\n"
            "except ImportError as e:\n    assert 'not for 0.0' in str(e)\n"
            "else:\n    raise SystemExit(1)\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_arguments_that_no_way_takes(monkeypatch):
    # no GPU needed: everything here is refused before the library is called
    x = torch.zeros(1, 2, 16, 64)
    for bad in (x, x[..., :32], None, "q", 3):
        for call in (lambda: binding.fa_fwd(bad, x, x, 0.125, False), lambda: binding.fa_fwd_gqa(bad, x, x, 0.125, True),
                     lambda: binding.fa_bwd(bad, x, x, x, x, x, 0.125, False), lambda: binding.fa_fp8_quant_hadamard(bad),
                     lambda: binding.fa_fwd_fp8(bad, x, x, x, x, x, 0.125, False)):
            _same_error(*_both(monkeypatch, call))


def _device_typed(*size, dtype=torch.bfloat16):
    # a plain tensor that says it is on the device, over no memory at all: for calls that end before any is touched
    device, nbytes = torch.device("cuda", 0), math.prod(size) * dtype.itemsize
    stride = [math.prod(size[i + 1:]) for i in range(len(size))]
    storage = torch._C._construct_storage_from_data_pointer(4096, device, nbytes)
    return torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(
        {"nbytes": nbytes, "data_ptr": 4096, "size": size, "stride": stride, "dtype": dtype, "device": device,
         "storage_offset": 0}, storage)


def _allocating_calls():
    # one of every kind that allocates its outputs
    x, c, s = _device_typed(1, 2, 16, 64), _device_typed(1, 2, 16, 64, dtype=torch.uint8), _device_typed(1, 2, 1, dtype=torch.float32)
    lse, ws = _device_typed(1, 2, 16, dtype=torch.float32), _device_typed(4096, dtype=torch.uint8)
    return [lambda: binding.fa_fwd(x, x, x, 0.125, False), lambda: binding.fa_fwd_gqa(x, x, x, 0.125, True),
            lambda: binding.fa_fp8_quant_hadamard(x), lambda: binding.fa_fwd_fp8(c, c, c, s, s, s, 0.125, False),
            lambda: binding.fa_fwd_fp8_gqa(c, c, c, s, s, s, 0.125, True), lambda: binding.fa_bwd(x, x, x, x, lse, x, 0.125, False, workspace=ws),
            lambda: binding.fa_bwd_gqa(x, x, x, x, lse, x, 0.125, True, workspace=ws)]


def test_an_exception_of_a_dispatch_mode_reaches_the_caller(monkeypatch):
    class Refuse(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise LookupError(f"no {func}")

    binding.lib()
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    for call in _allocating_calls():
        with Refuse():
            a, b = _both(monkeypatch, call)
        assert type(a) is LookupError
        _same_error(a, b)


@pytest.mark.skipif(binding._native is None, reason="the native part has not been built")
def test_an_interrupt_in_the_middle_of_a_call_is_not_lost(monkeypatch):
    binding.lib()
    for call in _allocating_calls():
        raised = []

        def stream():  # a key press comes once; should the call go on, it ends here
            raised.append(KeyboardInterrupt() if not raised else LookupError())
            raise raised[-1]

        monkeypatch.setattr(binding, "_stream", stream)
        with pytest.raises(KeyboardInterrupt):
            call()


def _tensors(dtype=torch.bfloat16, H=4, H_kv=2, N=70, d=64):
    g = torch.Generator(device="cuda").manual_seed(7)
    mk = lambda h: torch.randn((2, h, N, d), generator=g, device="cuda").to(dtype)  # noqa: E731
    return mk(H), mk(H_kv), mk(H_kv), mk(H)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("scale,causal", [(0.125, False), (0.125, True), (1, 1)])
def test_both_ways_give_the_same(monkeypatch, dtype, scale, causal):
    q, k, v, do = _tensors(dtype)
    full = _tensors(dtype, H_kv=4)[1:3]
    o, lse = binding.fa_fwd_gqa(q, k, v, scale, causal)
    signs = torch.ones(64, dtype=torch.int8, device="cuda")
    codes = [binding.fa_fp8_quant_hadamard(t) for t in (q, k, v)]
    codes_full = [codes[0]] + [binding.fa_fp8_quant_hadamard(t) for t in full]
    calls = [lambda: binding.fa_fwd(q, *full, scale, causal), lambda: binding.fa_fwd_gqa(q, k, v, scale, causal),
             lambda: binding.fa_fp8_quant_hadamard(q, signs), lambda: binding.fa_fp8_quant_hadamard(q, per_tensor=True),
             lambda: binding.fa_fwd_fp8(*(c[0] for c in codes_full), *(c[1] for c in codes_full), scale, causal),
             lambda: binding.fa_fwd_fp8_gqa(*(c[0] for c in codes), *(c[1] for c in codes), scale, causal)]
    if dtype != torch.float32:
        calls += [lambda: binding.fa_bwd_gqa(q, k, v, o, lse, do, scale, causal),
                  lambda: binding.fa_bwd(q, *full, o, lse, do, scale, causal)]
    for call in calls:
        native, python = _both(monkeypatch, call)
        assert type(native) is tuple and type(python) is tuple and len(native) == len(python)
        for a, b in zip(native, python):
            assert type(a) is torch.Tensor and a.dtype == b.dtype and a.device == b.device and a.stride() == b.stride()
            assert not a.requires_grad and torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_given_outputs_are_the_ones_returned_and_inputs_keep_their_graph(monkeypatch):
    q, k, v, do = _tensors()
    q = q.requires_grad_()
    # a contiguous tensor whose strides are not the ordinary ones (a dimension of size 1)
    one = torch.empty_strided((1, 4, 70, 64), (7, 70 * 64, 64, 1), dtype=torch.bfloat16, device="cuda").normal_()
    for native in (binding._native, None):
        monkeypatch.setattr(binding, "_native", native)
        o, lse = torch.empty_like(do), torch.empty((2, 4, 70), device="cuda")
        got = binding.fa_fwd_gqa(q, k, v, 0.125, True, o=o, lse=lse)
        assert got[0] is o and got[1] is lse and q.requires_grad and not o.requires_grad
        dk = torch.empty_like(k)
        grads = binding.fa_bwd_gqa(q, k, v, o, lse, do, 0.125, True, dk=dk)
        assert grads[1] is dk and not grads[0].requires_grad
        o1, l1 = binding.fa_fwd(one, one, one, 0.125, False)
        assert o1.stride() == (4 * 70 * 64, 70 * 64, 64, 1)
        assert binding.fa_bwd(one, one, one, o1, l1, one, 0.125, False)[0].stride() == one.stride()


@pytest.mark.gpu
def test_both_ways_refuse_the_same(monkeypatch):
    q, k, v, do = _tensors()
    lse = torch.empty((2, 4, 70), device="cuda")
    codes, scales = binding.fa_fp8_quant_hadamard(q)
    small = torch.empty((16,), dtype=torch.uint8, device="cuda")
    f32 = q.float()
    for call in (lambda: binding.fa_fwd(q, k, v, -1.0, False), lambda: binding.fa_fwd(q, k, v, float("nan"), False),
                 lambda: binding.fa_fwd(q[..., :32].contiguous(), k, v, 0.125, False), lambda: binding.fa_fwd(q.double(), k, v, 0.125, False),
                 lambda: binding.fa_fwd(q[0], k, v, 0.125, False), lambda: binding.fa_fwd(q.transpose(1, 2), k, v, 0.125, False),
                 lambda: binding.fa_fwd_gqa(q, q[:, :3].contiguous(), q[:, :3].contiguous(), 0.125, False),
                 lambda: binding.fa_fwd_gqa(q, k.reshape(-1), v, 0.125, False), lambda: binding.fa_fwd(q, k, v.cpu(), 0.125, False),
                 lambda: binding.fa_bwd(q, q, q, q, lse, do, 0.125, False, workspace=small),
                 lambda: binding.fa_bwd(f32, f32, f32, f32, lse, f32, 0.125, False),
                 lambda: binding.fa_fp8_quant_hadamard(codes), lambda: binding.fa_fp8_quant_hadamard(q, block_rows=64),
                 lambda: binding.fa_fwd_fp8(codes, codes, codes, scales, scales, scales, 0.0, False),
                 lambda: binding.fa_fwd(q, k, v, "scale", False)):
        _same_error(*_both(monkeypatch, call))
