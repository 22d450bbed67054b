"""New outputs of the Python entry points are ordinary tensors of torch's allocator: device, grad and inference flags, memory
accounting, storages of their own, and a dispatch mode sees them being made."""
import pytest

from test_gpu_binding import _gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_new_outputs_are_ordinary_tensors():
    R = _gpu()
    x = torch.randn(300, 256, device="cuda")
    R.rtopk_rowwise_exact(x, 32)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    v, i = R.rtopk_rowwise_exact(x, 32)
    assert torch.cuda.memory_allocated() - before == 2 * ((300 * 32 * 4 + 511) // 512 * 512)
    for t, dtype in ((v, torch.float32), (i, torch.int32)):
        assert t.device == x.device and t.dtype == dtype and tuple(t.shape) == (300, 32) and t.is_contiguous()
        assert not t.requires_grad and not t.is_inference() and t.is_leaf and type(t) is torch.Tensor
        assert t.untyped_storage().nbytes() == 300 * 32 * 4 and t.storage_offset() == 0
    assert v.untyped_storage().data_ptr() != i.untyped_storage().data_ptr()
    v.requires_grad_().mul(2).sum().backward()  # a leaf like any other
    assert bool((v.grad == 2).all())
    with torch.inference_mode():
        assert R.rtopk_rowwise_exact(x, 32)[0].is_inference()
    assert tuple(R.rtopk_rowwise_exact(torch.empty(0, 256, device="cuda"), 32)[0].shape) == (0, 32)


def test_a_dispatch_mode_sees_new_outputs():
    R = _gpu()
    from torch.utils._python_dispatch import TorchDispatchMode

    seen = []

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    x = torch.randn(30, 256, device="cuda")
    with Watch():
        v, i = R.rtopk_rowwise_exact(x, 32)
    assert seen.count(torch.ops.aten.empty.memory_format) == 2
    w, j = R.rtopk_rowwise_exact(x, 32)
    assert torch.equal(v, w) and torch.equal(i, j)


def test_a_trace_and_a_profiler_see_new_outputs():
    R = _gpu()
    x = torch.randn(30, 256, device="cuda")
    R.rtopk_rowwise_exact(x, 32)
    traced = torch.jit.trace(lambda t: R.rtopk_rowwise_exact(t, 32), (x,), check_trace=False)
    assert str(traced.graph).count("aten::empty") == 2
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as p:
        R.rtopk_rowwise_exact(x, 32)
    assert sum(e.count for e in p.key_averages() if e.key == "aten::empty") == 2


def test_new_outputs_are_filled_where_memory_is_to_be():
    R = _gpu()
    x = torch.randn(30, 256, device="cuda")
    seen = []
    was = torch.are_deterministic_algorithms_enabled()
    try:
        torch.use_deterministic_algorithms(True)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as p:
            v, i = R.rtopk_rowwise_exact(x, 32)
        seen = [e.key for e in p.key_averages()]
    finally:
        torch.use_deterministic_algorithms(was)
    assert "aten::fill_" in seen
    w, j = R.rtopk_rowwise_exact(x, 32)
    assert torch.equal(v, w) and torch.equal(i, j)
