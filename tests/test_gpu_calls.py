"""The compiled form of the binding's calls against its Python form: the same outputs for what both take, and everything else handed on."""
import pytest
import torch

from paper_2509_23202_amd import binding as fp4

G = fp4.A_LAYOUT_GEMM | fp4.W_LAYOUT_GEMM


def flat(out):
    return [out] if isinstance(out, torch.Tensor) else [t for t in out if t is not None]


def operands(fmt, rows, K, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(rows, K, device="cuda", generator=g).bfloat16()


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [fp4.MXFP4, fp4.NVFP4])
@pytest.mark.parametrize("M,N,K", [(1, 16, 128), (3, 264, 512), (129, 2048, 1024)])
def test_compiled_calls_equal_the_python_ones(monkeypatch, fmt, M, N, K):
    assert fp4._calls is not None
    x, w = operands(fmt, M, K, M), operands(fmt, N, K, N)
    rot = torch.linalg.qr(torch.randn(64, 64))[0].bfloat16().cuda().contiguous()
    qx, qw = fp4.fp4_rotate_quantize(x, 16, fmt, flags=fp4.LAYOUT_GEMM), fp4.fp4_quantize_weights(w, 16, fmt, flags=fp4.LAYOUT_GEMM)
    # (canonical layouts: in GEMM order the rows behind the last are not written)
    calls = [lambda: fp4.fp4_rotate_quantize(x, 16, fmt), lambda: fp4.fp4_rotate_quantize(x, 32, fmt, flags=fp4.SCALE_MSE),
             lambda: fp4.fp4_quantize_weights(w, 16, fmt), lambda: fp4.fp4_rotate_quantize_dense(x, rot, fmt),
             lambda: fp4.fp4_gemm(*qx, *qw, M, N, K, fmt, flags=G), lambda: fp4.fp4_gemm(*qx, *qw, M, N, K, fmt, flags=G | fp4.OUT_F32)]
    if fmt == fp4.MXFP4 and M <= 4:
        calls += [lambda: fp4.fp4_fused_linear(x, 16, qw[0], qw[1], N), lambda: fp4.fp4_w4a16_linear(x, 16, qw[0], qw[1], N, flags=fp4.OUT_F32)]
    got = [call() for call in calls]
    monkeypatch.setattr(fp4, "_calls", None)
    for a, call in zip(got, calls):
        b = call()
        assert type(a) is type(b) and len(flat(a)) == len(flat(b))
        for s, t in zip(flat(a), flat(b)):
            assert type(s) is torch.Tensor and s.dtype == t.dtype and s.shape == t.shape and torch.equal(s, t)


@pytest.mark.gpu
def test_other_calls_are_handed_on():
    x, w = operands(fp4.MXFP4, 2, 256, 1), operands(fp4.MXFP4, 32, 256, 2)
    qw = fp4.fp4_quantize_weights(w, 32, fp4.MXFP4, flags=fp4.LAYOUT_GEMM)
    want = fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32)
    out = torch.empty_like(want)
    assert fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32, out=out) is out and torch.equal(out, want)
    sub = fp4.fp4_fused_linear(torch.nn.Parameter(x, requires_grad=False), 32, qw[0], qw[1], 32)
    assert type(sub) is torch.Tensor and torch.equal(sub, want)
    f32 = fp4.fp4_rotate_quantize(x.float(), 1, fp4.MXFP4)
    assert torch.equal(f32[0], fp4.fp4_rotate_quantize(x, 1, fp4.MXFP4)[0])
    with pytest.raises(TypeError):
        fp4.fp4_rotate_quantize(x.half(), 32, fp4.MXFP4)
    with pytest.raises(AssertionError):
        fp4.fp4_rotate_quantize(x.t(), 32, fp4.MXFP4)
    for refused in (lambda: fp4.fp4_rotate_quantize(x, 33, fp4.MXFP4), lambda: fp4.fp4_rotate_quantize(x, 32, 7),
                    lambda: fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32, fp4.NVFP4), lambda: fp4.fp4_gemm(qw[0], qw[1], None, qw[0], qw[1], None, 2, 32, 250, fp4.MXFP4)):
        with pytest.raises(fp4.Fp4mrError):
            refused()


@pytest.mark.gpu
def test_an_error_of_the_device_is_raised_at_once(monkeypatch):
    """Entry points that report one without having touched the device: each is called once, and the calls raise."""
    import ctypes
    names = ["fp4_rotate_quantize", "fp4_quantize_weights", "fp4_rotate_quantize_dense", "fp4_gemm", "fp4_fused_linear", "fp4_w4a16_linear",
             "fp4_workspace_bytes", "fp4_packed_bytes"]
    functions = [getattr(fp4.lib, name) for name in names]
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    called, device = [], 7

    def stub(name):
        f = getattr(fp4.lib, name)
        return ctypes.CFUNCTYPE(f.restype, *f.argtypes)(lambda *args: called.append(name) or device)

    stubs = [stub(name) for name in names[:6]]
    assert fp4.lib.fp4_status_string(device).decode().startswith("HIP runtime error")
    x, w = operands(fp4.MXFP4, 2, 256, 1), operands(fp4.MXFP4, 32, 256, 2)
    rot = torch.eye(64).bfloat16().cuda()
    qx, qw = fp4.fp4_rotate_quantize(x, 32, fp4.MXFP4, flags=fp4.LAYOUT_GEMM), fp4.fp4_quantize_weights(w, 32, fp4.MXFP4, flags=fp4.LAYOUT_GEMM)
    torch.cuda.synchronize()
    calls = [lambda: fp4.fp4_rotate_quantize(x, 32, fp4.MXFP4), lambda: fp4.fp4_quantize_weights(w, 32, fp4.MXFP4),
             lambda: fp4.fp4_rotate_quantize_dense(x, rot, fp4.MXFP4), lambda: fp4.fp4_gemm(*qx, *qw, 2, 32, 256, fp4.MXFP4, flags=G),
             lambda: fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32), lambda: fp4.fp4_w4a16_linear(x, 32, qw[0], qw[1], 32)]
    try:
        fp4._calls.bind(*map(address, stubs + functions[6:]), fp4.Fp4mrError)
        for call in calls:
            with pytest.raises(fp4.Fp4mrError) as raised:
                call()
            assert raised.value.status == device
    finally:
        fp4._calls.bind(*map(address, functions), fp4.Fp4mrError)
    assert called == names[:6]
    assert fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32).shape == (2, 32)


@pytest.mark.gpu
def test_calls_under_a_function_mode_are_handed_on():
    """A mode sees the tensor functions of the Python form, and the results are the same."""
    class Mode(torch.overrides.TorchFunctionMode):
        def __init__(self):
            super().__init__()
            self.seen = set()

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.seen.add(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))

    x, w = operands(fp4.MXFP4, 2, 256, 1), operands(fp4.MXFP4, 32, 256, 2)
    qw = fp4.fp4_quantize_weights(w, 32, fp4.MXFP4, flags=fp4.LAYOUT_GEMM)
    for call in (lambda: fp4.fp4_rotate_quantize(x, 32, fp4.MXFP4), lambda: fp4.fp4_fused_linear(x, 32, qw[0], qw[1], 32)):
        want = flat(call())
        with Mode() as mode:
            got = flat(call())
        assert {"data_ptr", "new_empty"} <= mode.seen
        assert all(torch.equal(s, t) for s, t in zip(got, want))


def test_cpu_tensors_are_refused():
    x = torch.zeros(2, 256, dtype=torch.bfloat16)
    for call in (lambda: fp4.fp4_rotate_quantize(x, 32, fp4.MXFP4), lambda: fp4.fp4_fused_linear(x, 32, x, x, 32)):
        with pytest.raises(AssertionError):
            call()
