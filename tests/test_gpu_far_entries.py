"""Rows whose entries lie far apart -- one very low or very high entry, a masked half or tail, heavy tails -- against the
oracle, and what they cost beside rows without such entries: a masked row of logits is as ordinary as any other.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _far_rows(M, seed, far=1e9):
    g = np.random.Generator(np.random.Philox(seed))
    x = workloads.normal(10, M, seed)
    x[0, g.integers(0, M)] = -far
    x[1, g.integers(0, M)] = far
    x[2, g.random(M) < 0.5] = -far
    x[3, 2 * M // 3:] = -far
    x[4, : M // 4] = far
    x[5] = g.standard_cauchy(M).astype(np.float32)
    x[6] = np.exp(4 * x[6])
    x[7, g.integers(0, M, 8)] = -far * 10.0 ** -np.arange(8, dtype=np.float32)
    x[8, g.integers(0, M, 8)] = far * 10.0 ** -np.arange(8, dtype=np.float32)
    x[9] = -far
    x[9, g.integers(0, M, 5)] = np.linspace(-1, 1, 5, dtype=np.float32)
    return x


@pytest.mark.parametrize("M", [769, 1024, 1025, 1536, 2048, 3072, 4095, 6144, 8192, 8193, 16384, 32000, 40003, 65536, 131075])
def test_fp32_rows(M):
    R = _gpu()
    x = _far_rows(M, 9000 + M)
    xd = torch.from_numpy(x).cuda()
    for k in (1, 33, 64, 100, 245) + ((512,) if M > 8192 else ()):
        tag = f"M={M} k={k}"
        _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
        _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
        for mi in (5, 8, 40):
            _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), tag + f" early {mi}")
        _same(R.rtopk_rowwise_smallest(xd, k, 10), oracle.topk_earlystop_smallest(x, k, 10), tag + " smallest early")
        for eps in (0.3, 1e-3):
            ev, ei, et = oracle.alg1(x, k, eps_rel=eps)
            got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
            _same(got, (ev, ei), tag + f" eps {eps}")
            assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"
        if M <= 65536:
            for mi in (-1, 8):
                y = R.rtopk_maxk_dense(xd, k, mi)
                assert np.array_equal(y.cpu().numpy().view(np.int32), oracle.maxk_dense(x, k, mi).view(np.int32)), tag + f" dense {mi}"


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", [513, 1024, 1536, 4096, 8192, 16384, 32000, 50001])
def test_16bit_rows(kind, M):
    R = _gpu()
    x = np.clip(_far_rows(M, 9100 + M), -6e4, 6e4) if kind == "f16" else _far_rows(M, 9100 + M)
    b = workloads.to_bits16(x, kind)
    xd = torch.from_numpy(b.view(np.int16)).cuda().view(torch.float16 if kind == "f16" else torch.bfloat16)
    exact, early = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16)
    for k in (1, 64, 140, 245):
        v, i = exact(xd, k)
        _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k} exact")
        for mi in (5, 8, 40):
            v, i = early(xd, k, mi)
            _same((v.view(torch.int16), i), oracle.topk_earlystop_16(b, kind, k, mi), f"{kind} M={M} k={k} early {mi}")


def _time(fn):
    """Microseconds per call, the best of three stretches of calls."""
    for _ in range(3):
        fn()
    best = float("inf")
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 50.0)
    return best


# The bounds stand between what the lists of candidates cost on such rows (1.0 to 1.3 of the rows without) and what a
# search over the whole row behind them costs: exact mode 2.6, 3.4 and 10 times at these three widths.
@pytest.mark.parametrize("far", ("one", "half", "tail"))
@pytest.mark.parametrize("N,M,k,bound", [(8192, 4096, 64, 1.45), (1048, 32000, 64, 1.6), (671, 50000, 100, 2.0)])
def test_exact_mode_costs_what_it_costs_without_them(N, M, k, bound, far):
    R = _gpu()
    x = torch.randn((N, M), device="cuda")
    y = x.clone()
    if far == "one":
        y[:, 17] = -1e9
    elif far == "half":
        y[torch.rand((N, M), device="cuda") < 0.5] = -1e9
    else:
        y[:, 2 * M // 3:] = -1e9
    for fn, sign in ((R.rtopk_rowwise_exact, 1), (R.rtopk_rowwise_exact_smallest, -1)):
        xs, ys = sign * x, sign * y
        plain, masked = _time(lambda: fn(xs, k)), _time(lambda: fn(ys, k))
        assert masked < bound * plain, f"{masked:.1f} us against {plain:.1f}"


# A search that ends on a minimum below the floor needs no list.  Building them, and searching the whole row behind them, cost
# 3.9 times (early stopping, one far entry) and 3.5 times (precision 0.3) what ordinary rows do at 50000 columns.
@pytest.mark.parametrize("N,M,k,bound", [(8192, 4096, 64, 1.35), (1048, 32000, 64, 1.6), (671, 50000, 100, 2.0)])
def test_a_search_that_ends_early_costs_no_more_than_one_that_goes_on(N, M, k, bound):
    R = _gpu()
    x = torch.randn((N, M), device="cuda")
    y = x.clone()
    y[:, 17] = -1e9
    plain, masked = _time(lambda: R.rtopk_rowwise(x, k, 8)), _time(lambda: R.rtopk_rowwise(y, k, 8))
    assert masked < bound * plain, f"early stopping: {masked:.1f} us against {plain:.1f}"
    fine, coarse = _time(lambda: R.rtopk_rowwise_eps(x, k, 1e-3)), _time(lambda: R.rtopk_rowwise_eps(x, k, 0.3))
    assert coarse < (bound + 0.8) * fine, f"precision: {coarse:.1f} us against {fine:.1f}"
