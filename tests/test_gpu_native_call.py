"""The native call path of the binding (csrc/host/call.cpp) against the Python code it stands in for: results, returned
objects and errors of the calls it takes, and the calls it leaves to Python."""
import numpy as np
import pytest

from tests.test_gpu_parity import P2, P43, gpu  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def both(gpu, f):
    """Result of f() on the native path and in Python: values, or the error's type and text."""
    import torch

    def run():
        try:
            r = f()
            torch.cuda.synchronize()
            return r if isinstance(r, tuple) else (r,)
        except Exception as e:                       # noqa: BLE001  (compared, not handled)
            return type(e), str(e)

    native = run()
    keep, gpu._call = gpu._call, None
    try:
        plain = run()
    finally:
        gpu._call = keep
    assert len(native) == len(plain)
    for a, b in zip(native, plain):
        if isinstance(a, torch.Tensor):
            assert a.dtype == b.dtype and a.shape == b.shape and not a.requires_grad and torch.equal(a, b)
        else:
            assert a == b or a is b, (a, b)
    return native


# rows of one wavefront, of one workgroup, and rows that need the workspace
@pytest.mark.parametrize("rows,n", [(0, 16), (64, 16), (5, 1500), (2, 40000)])
def test_results_and_errors(gpu, rows, n):
    import torch
    assert gpu._call is not None, "the native call path was not built"
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((rows, n), generator=g, device="cuda")
    t = torch.randn((rows, n), generator=g, device="cuda")
    k, lam = max(1, n // 10), 0.1
    for p in (P2, P43, 2):
        both(gpu, lambda: gpu.topk_mask_fwd(x, k, p, lam))
        both(gpu, lambda: gpu.topkmag_fwd(x, k, p, lam))
        both(gpu, lambda: gpu.topk_signed_mask_fwd(x, k, p, lam))
        both(gpu, lambda: gpu.topk_masked_value_fwd(x, k, p, lam))
        both(gpu, lambda: gpu.topk_mask_loss(x, t, k, p, lam))
        both(gpu, lambda: gpu.topk_mask_sparse_fwd(x, k, p, lam, min(n, 2 * k)))
        for f in (gpu.topk_mask_jvp, gpu.topk_mask_vjp, gpu.topkmag_jvp, gpu.topkmag_vjp, gpu.topk_signed_mask_jvp,
                  gpu.topk_masked_value_jvp):
            both(gpu, lambda: f(x, t, k, p, lam))
    both(gpu, lambda: gpu.topk_mask_jvp(x, t, k, P2, lam, want_out=False))
    out, d = torch.empty_like(x), torch.empty_like(x)
    r = gpu.topk_mask_jvp(x, t, k, P2, lam, out=out, jvp_out=d)
    assert r[0] is out and r[1] is d
    both(gpu, lambda: gpu.topk_mask_jvp(x, t, k, P2, lam, out=out, jvp_out=d))
    both(gpu, lambda: gpu.topk_mask_fwd(x.clone().requires_grad_(), k, P2, lam))
    both(gpu, lambda: gpu.topk_mask_fwd(torch.nn.Parameter(x), k, P2, lam))
    both(gpu, lambda: gpu.topk_mask_fwd(x, np.int64(k), P2, np.float64(lam)))
    both(gpu, lambda: gpu.topk_mask_fwd(x, str(k), P2, lam))
    # (the side stream's call is waited for in both())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    both(gpu, lambda: gpu.topk_mask_fwd(x, k, P2, lam, stream=s))
    # what is refused stays refused, in the same words
    bad = [lambda: gpu.topk_mask_fwd(x, n + 1, P2, lam), lambda: gpu.topk_mask_fwd(x, k, 3.0, lam),
           lambda: gpu.topk_mask_fwd(x, k, P2, -1.0), lambda: gpu.topk_mask_fwd(x.cpu(), k, P2, lam),
           lambda: gpu.topk_mask_fwd(x.double(), k, P2, lam), lambda: gpu.topk_mask_fwd(x[0] if rows else x[:, 0], k, P2, lam),
           lambda: gpu.topk_mask_jvp(x, t[:, 1:], k, P2, lam), lambda: gpu.topk_mask_sparse_fwd(x, k, P2, lam, n + 1),
           lambda: gpu.topk_mask_fwd(None, k, P2, lam), lambda: gpu.topk_mask_fwd(x, "one", P2, lam),
           lambda: gpu.topk_mask_loss(x, t.cpu(), k, P2, lam)]
    if rows > 1:
        bad += [lambda: gpu.topk_mask_fwd(x, k, P2, lam, out=x), lambda: gpu.topk_mask_jvp(x, t, k, P2, lam, jvp_out=t),
                lambda: gpu.topk_mask_jvp(x, t, k, P2, lam, out=out, jvp_out=out),
                lambda: gpu.topk_mask_fwd(x.t().contiguous().t(), k, P2, lam)]
    for f in bad:
        r = both(gpu, f)
        assert rows == 0 or (isinstance(r[0], type) and issubclass(r[0], Exception)), r


def test_modes_that_watch_tensor_calls_are_left_to_python(gpu):
    import torch
    from torch.overrides import TorchFunctionMode
    x = torch.randn((8, 32), device="cuda")
    seen = []

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))

    with Watch():
        gpu.topk_mask_fwd(x, 2, P2, 0.5)
    assert "empty_like" in seen
    torch.cuda.synchronize()
