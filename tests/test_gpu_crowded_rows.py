"""Rows of more than 32768 columns whose winners crowd -- ties by the thousand, sorted rows, masked segments -- against the
oracle, and what they cost: the list of a segment then holds its k + 1 largest keys, found by a full-width search.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_far_entries import _time
from test_gpu_filtered_rows import _gpu, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _crowded(M, seed):
    g = np.random.Generator(np.random.Philox(seed))
    x = workloads.normal(12, M, seed)
    x[0] = g.integers(0, 64, M)
    x[1] = g.integers(0, 3, M)
    x[2] = np.sort(x[2])
    x[3] = -np.sort(-x[3])
    x[4] = 1.0
    x[5, 20000:] = -1e9
    x[6, :-20000] = -1e9
    # the floor, 1.0, is the last minimum as well; the first columns at or above it are ties, the larger keys the last ones
    x[7] = 0.0
    x[7, : M // 2] = 1.0
    x[7, -7:] = 2.0
    x[8] = 0.0
    x[8, 5::3] = 1.0
    x[8, -3:] = 2.0
    x[8, 17000:17004] = 1.5
    x[9] = np.maximum(x[9], 0.0)
    x[10] = np.round(x[10] * 4) / 4
    x[11] = np.repeat(workloads.normal(1, M // 4096 + 1, seed + 1)[0], 4096)[:M]
    return x


@pytest.mark.parametrize("M", [32769, 40000, 65536, 65537, 131075, 300001])
def test_every_mode(M):
    R = _gpu()
    x = _crowded(M, 9500 + M)
    for rows in (x, -x):
        xd = torch.from_numpy(rows).cuda()
        for k in (1, 6, 50, 256, 257, 512):
            tag = f"M={M} k={k}"
            _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(rows, k), tag + " exact")
            _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(rows, k), tag + " smallest")
            for mi in (8, 13, 40):
                _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(rows, k, mi), tag + f" early {mi}")
                _same(R.rtopk_rowwise_smallest(xd, k, mi), oracle.topk_earlystop_smallest(rows, k, mi), tag + f" smallest early {mi}")
            for eps in (0.3, 1e-2, 1e-6):
                ev, ei, et = oracle.alg1(rows, k, eps_rel=eps)
                got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
                _same(got, (ev, ei), tag + f" eps {eps}")
                assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"


# Ordinary rows of these sizes against crowded ones: 1.5 to 2.5 times here, 5 to 20 times where such rows are streamed.
@pytest.mark.parametrize("N,M,k", [(671, 50000, 100), (256, 131072, 50)])
@pytest.mark.parametrize("kind", ("whole numbers", "sorted", "masked tail"))
def test_what_they_cost(N, M, k, kind):
    R = _gpu()
    x = torch.randn((N, M), device="cuda")
    if kind == "sorted":
        y = x.sort(dim=1).values
    elif kind == "masked tail":
        y = x.clone()
        y[:, M // 2:] = -1e9
    else:
        y = torch.randint(0, 64, (N, M), device="cuda").float()
    plain, crowded = _time(lambda: R.rtopk_rowwise_exact(x, k)), _time(lambda: R.rtopk_rowwise_exact(y, k))
    assert crowded < 4.0 * plain, f"{crowded:.1f} us against {plain:.1f}"


def test_columns_stay_inside_the_row_whatever_the_values_are():
    # the selection is unspecified with NaN or infinities, but a column that was never listed must not come out
    R = _gpu()
    M, k = 40000, 50
    g = np.random.Generator(np.random.Philox(9600))
    x = np.full((8, M), np.nan, dtype=np.float32)
    for r in range(8):
        at = g.integers(0, M, 40 * (r + 1))
        x[r, at] = -np.inf if r % 2 == 0 else g.standard_normal(at.size).astype(np.float32)
    x[4:, ::97] = np.inf
    xd = torch.from_numpy(x).cuda()
    for fn in (lambda v, i: R.rtopk_rowwise_exact(xd, k, v, i), lambda v, i: R.rtopk_rowwise(xd, k, 9, v, i),
               lambda v, i: R.rtopk_rowwise_exact_smallest(xd, k, v, i), lambda v, i: R.rtopk_rowwise_eps(xd, k, 1e-3, v, i)):
        torch.full((1 << 20,), 0x7F7F7F7F, dtype=torch.int32, device="cuda")  # what the scratch memory may hold
        v, i = torch.zeros(8, k, device="cuda"), torch.zeros(8, k, dtype=torch.int32, device="cuda")
        fn(v, i)
        assert int(i.min()) >= 0 and int(i.max()) < M
