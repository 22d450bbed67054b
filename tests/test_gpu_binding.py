"""The Python entry points through the native module: the caller's outputs come back as they are, new ones are new, what
was refused is refused by the Python code with the same exceptions, and calls follow the current stream and threads."""
import gc
import threading

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_00822_amd as R

    R.load_library()
    return R


def test_given_outputs_come_back_and_new_ones_are_new():
    R = _gpu()
    x = torch.randn(50, 100, device="cuda")
    v = torch.empty(50, 7, device="cuda")
    i = torch.empty(50, 7, dtype=torch.int32, device="cuda")
    t = torch.empty(50, dtype=torch.int32, device="cuda")
    a = R.rtopk_rowwise_exact(x, 7, v, i)
    assert a[0] is v and a[1] is i
    b = R.rtopk_rowwise_exact(x, 7, out_idx=i)
    assert b[0] is not v and b[1] is i
    c = R.rtopk_rowwise_eps(x, 7, 0, v, i, t)  # an int epsilon goes through the Python code
    assert c[0] is v and c[1] is i and c[2] is t
    assert len(R.rtopk_rowwise_eps(x, 7, 0.0)) == 2 and len(R.rtopk_rowwise_eps(x, 7, 0.0, want_iters=True)) == 3
    y = torch.empty_like(x)
    assert R.rtopk_maxk_dense(x, 7, out=y) is y
    g = R.rtopk_maxk_backward(v, i, 100)
    assert R.rtopk_maxk_backward(v, i, 100, g) is g and R.rtopk_maxk_backward_gather(g, i, v) is v


def test_what_was_refused_is_refused():
    R = _gpu()
    x = torch.randn(50, 100, device="cuda")
    for bad in (x.cpu(), x.double(), x[:, ::2], x[0], x.half()):
        with pytest.raises(ValueError):
            R.rtopk_rowwise_exact(bad, 3)
        with pytest.raises(ValueError):
            R.rtopk_maxk_dense(bad, 3)
    with pytest.raises(ValueError):
        R.rtopk_rowwise_exact(x, 3, out_vals=torch.empty(50, 4, device="cuda"))
    with pytest.raises(ValueError):
        R.rtopk_rowwise_eps(x, 3, 0.1, out_iters=torch.empty(49, dtype=torch.int32, device="cuda"))
    for k in (0, 101):
        with pytest.raises(R.RTopKError):
            R.rtopk_rowwise_exact(x, k)
    with pytest.raises(R.RTopKError):
        R.rtopk_rowwise(x, 3, -1)  # not exact mode
    with pytest.raises(R.RTopKError):
        R.rtopk_rowwise_eps(x, 3, -1.0)
    with pytest.raises(TypeError):
        R.rtopk_rowwise_exact(x, 3.0)
    with pytest.raises(ValueError):
        R.rtopk_maxk_backward(x, torch.zeros(50, 3, dtype=torch.int64, device="cuda"), 100)
    with pytest.raises(ValueError):
        R.rtopk_maxk_backward_gather(x, torch.zeros(49, 3, dtype=torch.int32, device="cuda"))


def test_threads_and_streams():
    R = _gpu()
    xs = [workloads.normal(300, 200 + 13 * t, seed=5000 + t) for t in range(4)]
    got = [None] * 4

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            x = torch.from_numpy(xs[t]).cuda()
            for _ in range(50):
                got[t] = R.rtopk_rowwise_exact(x, 20 + t)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for t in range(4):
        ev, ei = oracle.topk_exact(xs[t], 20 + t)
        assert np.array_equal(got[t][1].cpu().numpy(), ei)
        assert np.array_equal(got[t][0].cpu().numpy().view(np.int32), ev.view(np.int32))


def test_without_memory_for_scratch_the_call_does_without_and_for_outputs_it_raises():
    R = _gpu()
    gc.collect()
    torch.cuda.empty_cache()
    x = torch.randn((512, 131072), device="cuda")
    k, scratch = 400, 24 << 20  # 2048 segments of 12 KiB and a head each
    vals, cols = R.rtopk_rowwise_exact(x, k)
    v, i = torch.empty_like(vals), torch.empty_like(cols)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
    hog = []  # whatever is free inside the segments that tests before this one left behind
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):
            while True:
                hog.append(torch.empty(2 << 20, dtype=torch.uint8, device="cuda"))
        with pytest.raises(torch.cuda.OutOfMemoryError):
            torch.empty(scratch, dtype=torch.uint8, device="cuda")
        R.rtopk_rowwise_exact(x, k, v, i)
        with pytest.raises(torch.cuda.OutOfMemoryError):
            R.rtopk_rowwise_exact(x, 20000)
    finally:
        del hog
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(v, vals) and torch.equal(i, cols)


def test_numbers_of_any_kind_take_the_same_path():
    # rows of more than 32768 columns: only the native module lends the scratch memory that splits them
    R = _gpu()
    from paper_2409_00822_amd import rtopk as binding

    fast = binding._native()
    x = torch.randn(3, 40000, device="cuda")
    want = R.rtopk_rowwise_exact(x, 50)
    early = R.rtopk_rowwise(x, 50, 8)
    eps = R.rtopk_rowwise_eps(x, 50, 1.0, want_iters=True)
    for whole in (np.int64, np.int32, np.uint8, lambda v: torch.tensor(v)):
        got = fast.select(binding._F32 | binding._EXACT, x, whole(50), 0, None, None)
        assert got is not None and all(torch.equal(a, b) for a, b in zip(got, want))
        got = fast.select(binding._F32, x, whole(50), whole(8), None, None)
        assert got is not None and all(torch.equal(a, b) for a, b in zip(got, early))
        got = fast.select_eps(x, whole(50), whole(1), None, None, None, 1)
        assert got is not None and all(torch.equal(a, b) for a, b in zip(got, eps))
    assert len(R.rtopk_rowwise_eps(x, np.int64(50), np.float64(1.0), want_iters=np.bool_(False))) == 2
    assert len(R.rtopk_rowwise_eps(x, 50, "1.0")) == 2  # Python's float() takes it, so the call does
    for bad in (3.0, "3", None, np.float32(3.0)):
        assert fast.select(binding._F32 | binding._EXACT, x, bad, 0, None, None) is None
    with pytest.raises(TypeError):
        R.rtopk_rowwise_exact(x, "3")
