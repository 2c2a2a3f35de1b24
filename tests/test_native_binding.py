"""The native half of the Python binding (_tqpy.so) takes exactly the calls that the Python
path takes, and leaves every other to it."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2608_08910_amd import _tqpy as fast  # (built with the library: its absence is a failure)
from paper_2608_08910_amd import tq


def test_native_functions_leave_what_they_do_not_take():
    x = torch.zeros((2, 512))
    q, d, b = torch.zeros((2, 512), dtype=torch.int8), torch.zeros((2, 2)), torch.zeros((2, 2), dtype=torch.int32)
    # CPU tensors, no tensors, a wrong count, ints that are not plain or out of range
    assert fast.quantize_act(x, q, d, b, 0) is None
    assert fast.quantize_act(None, q, d, b, 0) is None
    assert fast.quantize_act(x, q, d, b) is None
    assert fast.gemv_f32(2 ** 40, 512, q, q, x, x, q, d, b, 0) is None
    assert fast.gemv_f32(True, 512, q, q, x, x, q, d, b, 0) is None
    assert fast.moe_grouped(1, 256, 256, [q] * 3, (q,) * 3, x, b, d, x, q, 0, 0) is None
    # tensors without storage, and subclasses
    meta = torch.zeros((2, 512), device="meta")
    assert fast.quantize_act(meta, q, d, b, 0) is None
    with pytest.raises(TypeError):
        tq.tq_quantize_act(x, q, d, b)


def test_weights_objects_that_describe_themselves_keep_the_python_path(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    m = tq.TqMatrix(1, 256, None, None)
    assert tq._native(None, m, tq.TqMatrix) and tq._native(None) and not tq._native(0, m, tq.TqMatrix)
    assert not tq._native(None, type("Own", (tq.TqMatrix,), {})(1, 256, None, None), tq.TqMatrix)
    assert not tq._native(None, tq.TqExpertRecords(1, 256, 256, None), tq.TqExperts)


def test_missing_native_half_is_reported():
    code = ("import sys, warnings; sys.modules['paper_2608_08910_amd._tqpy'] = None; warnings.simplefilter('error')\n"
            "try:\n    from paper_2608_08910_amd import tq\nexcept RuntimeWarning as e:\n    print(e)")
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(tq.__file__)), capture_output=True, text=True)
    assert "_tqpy.so is not built" in r.stdout, r.stdout + r.stderr


GPU_CALLS = ["quantize_act", "gemv", "gemv_f32", "gemv2", "gemv_mx", "moe_grouped"]


def moe(*a):
    """tq_moe_grouped on the plain tensors of a TqExperts (codes, scales) and the call's own."""
    tq.tq_moe_grouped(tq.TqExperts(4, 512, 256, a[:3], a[3:6]), *a[6:])
    a[-1].zero_()  # (the workspace's contents are nobody's)


def args_of(name):
    n, k, t = 64, 512, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    codes = torch.randint(0, 256, (n, 2, 128), dtype=torch.uint8, device="cuda", generator=g) & 0x33
    q = torch.randint(-127, 128, (t, k), dtype=torch.int8, device="cuda", generator=g)
    d = torch.rand((t, 2), device="cuda", generator=g)
    b = torch.zeros((t, 2), dtype=torch.int32, device="cuda")
    s = torch.full((n, 2), 0x2C00, dtype=torch.int16, device="cuda")
    x, y = torch.randn((t, k), device="cuda", generator=g), torch.zeros((t, n), device="cuda")
    if name == "quantize_act":
        return tq.tq_quantize_act, [x, q, d, b]
    if name == "gemv":
        return tq.tq_gemv, [tq.TqMatrix(n, k, codes, s), q, d, b, y]
    if name == "gemv_f32":
        return tq.tq_gemv_f32, [tq.TqMatrix(n, k, codes, s), x, y, q, d, b]
    if name == "moe_grouped":
        experts = 4
        shapes = [(256, 2), (256, 2), (512, 1)]
        codes = [torch.randint(0, 256, (experts, r, kb, 128), dtype=torch.uint8, device="cuda", generator=g) & 0x33 for r, kb in shapes]
        scales = [torch.full((experts, r, kb), 0x2C00, dtype=torch.int16, device="cuda") for r, kb in shapes]
        idx = torch.tensor([[0, 2], [3, 2]], dtype=torch.int32, device="cuda")
        ws = tq.moe_workspace(tq.TqExperts(experts, 512, 256, tuple(codes), tuple(scales)), t, 2)
        return moe, [*codes, *scales, x, idx, torch.rand((t, 2), device="cuda", generator=g), torch.zeros_like(x), ws]
    if name == "gemv2":
        return tq.tq_gemv2, [tq.TqMatrix2(n, k, codes, s[:, :, None].repeat(1, 1, 2).contiguous()), q, d, y]
    return tq.tq_gemv_mx, [tq.TqMatrixMx(n, k, codes, torch.full((n, 16), 120, dtype=torch.uint8, device="cuda")), q, d, y]


def outcome(fn, args):
    try:
        fn(*args)
        torch.cuda.synchronize()
        return [a.clone() for a in args if isinstance(a, torch.Tensor)]
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)


@pytest.mark.gpu
@pytest.mark.parametrize("name", GPU_CALLS)
def test_native_and_python_paths_agree(name, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()
    fn, args = args_of(name)
    variants = [lambda a: a]
    for i, v in enumerate(args):
        if isinstance(v, torch.Tensor):
            variants += [lambda a, i=i: a[:i] + [a[i].double()] + a[i + 1:],      # type
                         lambda a, i=i: a[:i] + [a[i].narrow(-1, 0, 1)] + a[i + 1:],  # shape, and strides where wider
                         lambda a, i=i: a[:i] + [a[i].transpose(0, -1)] + a[i + 1:],
                         lambda a, i=i: a[:i] + [a[i].cpu()] + a[i + 1:],
                         lambda a, i=i: a[:i] + [a[i][None]] + a[i + 1:],
                         lambda a, i=i: a[:i] + [None] + a[i + 1:]]
    for j, v in enumerate(variants):
        res = []
        for native in (True, False):
            monkeypatch.setattr(tq, "_fast", fast if native else None)
            fn, args = args_of(name)
            res.append(outcome(fn, v(list(args))))
        if isinstance(res[0], list):
            assert all(torch.equal(p, r) for p, r in zip(*res)), f"{name} variant {j}"
        else:
            assert res[0] == res[1], f"{name} variant {j}"
    monkeypatch.setattr(tq, "_fast", fast)
    fn, args = args_of(name)
    calls = []
    real = getattr(fast, name)
    class Spy:
        def __getattr__(self, a):
            def f(*x):
                calls.append(real(*x))
                return calls[-1]
            return f
    monkeypatch.setattr(tq, "_fast", Spy())
    fn(*args)
    assert calls == [0], "a plain call takes the native path"
