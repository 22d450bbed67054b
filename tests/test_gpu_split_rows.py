"""GPU parity of rows spread over several workgroups (fp32, more than 32768 columns): segment counts and tails, k around
the lists' limits, rows whose segments overflow or whose last threshold is below the floor, several batches of rows.

Selections are copies of inputs and their columns: tolerance 0.
"""
import ctypes

import numpy as np
import pytest

import oracle
from test_gpu_filtered_rows import _gpu, _rows, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M", [32769, 40000, 50001, 65536, 65537, 98304, 131075, 400003])
def test_every_mode_on_every_kind_of_row(M):
    R = _gpu()
    x = _rows(M, 6000 + M)
    xd = torch.from_numpy(x).cuda()
    for k in (1, 50, 256, 257, 512, 513):
        tag = f"M={M} k={k}"
        _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
        _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
        for mi in (7, 8, 13, 1 << 30):
            _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, min(mi, 600)), tag + f" early {mi}")
        _same(R.rtopk_rowwise_smallest(xd, k, 10), oracle.topk_earlystop_smallest(x, k, 10), tag + " smallest early")
        for eps in (1e-2, 1e-5):
            ev, ei, et = oracle.alg1(x, k, eps_rel=eps)
            got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
            _same(got, (ev, ei), tag + f" eps {eps}")
            assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"


@pytest.mark.parametrize("N", [1, 3, 130, 700])
def test_few_and_many_rows(N):
    R = _gpu()
    x = np.tile(_rows(34000, 6100), (N // 10 + 1, 1))[:N].copy()
    x[:, 11] = np.arange(N, dtype=np.float32) * 0.01
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, 40), oracle.topk_exact(x, 40), f"N={N}")


def _plain(R, x, k):
    """The entry point without scratch memory."""
    lib = R.load_library()
    v = torch.empty(x.shape[0], k, device="cuda")
    i = torch.empty(x.shape[0], k, dtype=torch.int32, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    assert lib.rtopk_rowwise_exact(x.data_ptr(), x.shape[0], x.shape[1], k, v.data_ptr(), i.data_ptr(), s) == 0
    return v, i


def test_scratch_memory_in_several_batches_and_refusals():
    R = _gpu()
    lib = R.load_library()
    lib.rtopk_workspace_bytes.restype = ctypes.c_int64
    lib.rtopk_workspace_bytes.argtypes = [ctypes.c_int64] + [ctypes.c_int32] * 4
    N, M, k = 9000, 40000, 512
    need = lib.rtopk_workspace_bytes(N, M, k, 1, 0)
    assert 0 < need <= 129 << 20  # bounded: the rows go through it in batches
    assert lib.rtopk_workspace_bytes(N, 32768, k, 1, 0) == 0 and lib.rtopk_workspace_bytes(N, M, 513, 1, 0) == 0
    assert lib.rtopk_workspace_bytes(N, M, k, 3, 0) == 0 and lib.rtopk_workspace_bytes(0, M, k, 1, 0) == 0
    x = torch.randn(N, M, device="cuda")
    v, i = R.rtopk_rowwise_exact(x, k)
    pv, pi = _plain(R, x, k)
    assert torch.equal(i, pi) and torch.equal(v, pv)
    fn = lib.rtopk_select_ws
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64] + [ctypes.c_int32] * 4 + [ctypes.c_float] + [ctypes.c_void_p] * 4 + [
        ctypes.c_int64, ctypes.c_void_p]
    w = torch.empty(need, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    args = lambda variant, ws, nb: (x.data_ptr(), N, M, k, variant, 0, 0.0, v.data_ptr(), i.data_ptr(), None, ws, nb, s)  # noqa: E731
    assert fn(*args(3, w.data_ptr(), need)) == -2 and fn(*args(6, w.data_ptr(), need)) == -2
    assert fn(*args(1, w.data_ptr() + 4, need - 4)) == -5
    assert fn(*args(1, v.data_ptr(), need)) == -8
    v.zero_()
    assert fn(*args(1, w.data_ptr(), need - 1)) == 0  # too little: the plain entry point's launch
    assert torch.equal(v, pv) and torch.equal(i, pi)


def test_graph_replays_with_new_inputs():
    R = _gpu()
    x = torch.randn(20, 70000, device="cuda")
    R.rtopk_rowwise_exact(x, 30)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        R.rtopk_rowwise_exact(x, 30)
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        v, i = R.rtopk_rowwise_exact(x, 30)
    for seed in range(4):
        torch.manual_seed(seed)
        x.copy_(torch.randn(20, 70000, device="cuda"))
        g.replay()
        torch.cuda.synchronize()
        _same((v, i), oracle.topk_exact(x.cpu().numpy(), 30), f"replay {seed}")
        R.rtopk_rowwise_exact(torch.randn(5, 50000, device="cuda"), 9)


def test_threads_and_streams_share_the_allocator():
    import threading

    R = _gpu()
    xs = [_rows(33000 + 4099 * t, 6200 + t) for t in range(4)]
    got = [None] * 4

    def work(t):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            x = torch.from_numpy(xs[t]).cuda()
            got[t] = [R.rtopk_rowwise_exact(x, 20 + 7 * t) for _ in range(30)]  # scratch and outputs come and go
        s.synchronize()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for t in range(4):
        want = oracle.topk_exact(xs[t], 20 + 7 * t)
        for j, pair in enumerate(got[t]):
            _same(pair, want, f"thread {t} call {j}")


def test_few_very_wide_rows_are_split_into_the_longer_segments():
    R = _gpu()
    lib = R.load_library()
    lib.rtopk_workspace_bytes.restype = ctypes.c_int64
    lib.rtopk_workspace_bytes.argtypes = [ctypes.c_int64] + [ctypes.c_int32] * 4
    assert lib.rtopk_workspace_bytes(2, 1 << 20, 200, 1, 0) > 0  # twice the candidates in the shorter ones would not fit
    x = _rows(1 << 20, 6300)[:4]
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, 200), oracle.topk_exact(x, 200), "exact")
    _same(R.rtopk_rowwise(xd, 200, 9), oracle.topk_earlystop(x, 200, 9), "early")


@pytest.mark.parametrize("M, k", [(60 * 16384, 17), (64 * 16384, 10), (65 * 16384 + 5, 9), (50 * 16384, 40)])
def test_many_short_lists(M, k):
    # a register of the merge holds candidates of one list: lists of a few more than 64 take two, more in all than four
    # wavefronts have, and rows of more than 64 lists are numbered through
    R = _gpu()
    g = np.random.default_rng(M + k)
    x = g.standard_normal((3, M)).astype(np.float32)
    x[1] = np.round(x[1] * 64) / 64
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
    _same(R.rtopk_rowwise(xd, k, 14), oracle.topk_earlystop(x, k, 14), f"M={M} k={k} early")
    ev, ei, et = oracle.alg1(x, k, eps_rel=1e-4)
    got = R.rtopk_rowwise_eps(xd, k, 1e-4, want_iters=True)
    _same(got, (ev, ei), f"M={M} k={k} eps")
    assert np.array_equal(got[2].cpu().numpy(), et)


@pytest.mark.parametrize("M, k, most, fewer", [(50000, 64, 1024, (1023, 700, 512, 3)), (80000, 64, 683, (682, 450, 2))])
def test_memory_for_a_batch_serves_smaller_ones(M, k, most, fewer):
    # the shorter segments of fewer rows need more than the longer ones of more: then these are taken, and the memory is used
    R = _gpu()
    lib = R.load_library()
    lib.rtopk_workspace_bytes.restype = ctypes.c_int64
    lib.rtopk_workspace_bytes.argtypes = [ctypes.c_int64] + [ctypes.c_int32] * 4
    fn = lib.rtopk_select_ws
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64] + [ctypes.c_int32] * 4 + [ctypes.c_float] + [ctypes.c_void_p] * 4 + [
        ctypes.c_int64, ctypes.c_void_p]
    lent = lib.rtopk_workspace_bytes(most, M, k, 1, 0)
    assert any(lib.rtopk_workspace_bytes(N, M, k, 1, 0) > lent for N in fewer)
    x = torch.randn(max(fewer), M, device="cuda")
    w = torch.empty(lent, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    for N in fewer:
        v = torch.empty(N, k, device="cuda")
        i = torch.empty(N, k, dtype=torch.int32, device="cuda")
        w.fill_(0xA5)
        assert fn(x.data_ptr(), N, M, k, 1, 0, 0.0, v.data_ptr(), i.data_ptr(), None, w.data_ptr(), lent, s) == 0
        assert not (w == 0xA5).all(), f"N={N}: not split"
        pv, pi = _plain(R, x[:N], k)
        assert torch.equal(v, pv) and torch.equal(i, pi), f"N={N}"


@pytest.mark.parametrize("M, k", [(65 * 32768 + 3, 2), (2200003, 10), (2200003, 20), (3000001, 50), (100 * 32768 - 5, 90), (1 << 20, 8)])
def test_sixteen_merging_wavefronts_with_few_candidates(M, k):
    # rows of more than 64 lists, and early stopping with few steps: 4, 8 or 16 candidates a lane
    R = _gpu()
    g = np.random.default_rng(M + k)
    x = g.standard_normal((2, M)).astype(np.float32)
    x[1] = np.round(x[1] * 64) / 64
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
    _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), f"M={M} k={k} smallest")
    for steps in (4, 9, 14):
        _same(R.rtopk_rowwise(xd, k, steps), oracle.topk_earlystop(x, k, steps), f"M={M} k={k} early {steps}")
    ev, ei, et = oracle.alg1(x, k, eps_rel=1e-4)
    got = R.rtopk_rowwise_eps(xd, k, 1e-4, want_iters=True)
    _same(got, (ev, ei), f"M={M} k={k} eps")
    assert np.array_equal(got[2].cpu().numpy(), et)


@pytest.mark.parametrize("M, k", [(131072, 72), (150000, 45), (262144, 80), (700000, 16), (700000, 128), (1000000, 80), (1000000, 160),
                                  (1000000, 700)])
def test_lists_that_would_fill_more_registers_than_their_candidates(M, k):
    # lists of a few more than 64, 128 ... candidates: by lists or by number, whichever walks fewer registers, row by row
    R = _gpu()
    g = np.random.default_rng(M * 3 + k)
    x = g.standard_normal((6, M)).astype(np.float32)
    x[1] = np.round(x[1] * 256) / 256
    x[2] = g.random(M, dtype=np.float32)
    x[3, : M // 3] += 2  # most candidates in a third of the lists
    x[4] = np.sort(x[4])
    x[5, 7:] = -3e38  # fewer than k keys above the mask
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
    _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), f"M={M} k={k} smallest")
    for steps in (3, 8, 16):
        _same(R.rtopk_rowwise(xd, k, steps), oracle.topk_earlystop(x, k, steps), f"M={M} k={k} early {steps}")
    ev, ei, et = oracle.alg1(x, k, eps_rel=1e-5)
    got = R.rtopk_rowwise_eps(xd, k, 1e-5, want_iters=True)
    _same(got, (ev, ei), f"M={M} k={k} eps")
    assert np.array_equal(got[2].cpu().numpy(), et)
