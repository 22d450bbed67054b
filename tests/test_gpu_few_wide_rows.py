"""GPU parity of rows of 1537 to 8192 columns on both sides of the row counts up to which they take a workgroup each: ordinary
rows, rows with far entries, tied, masked and sorted ones, every mode, type and form.  The rows repeat a base, so the oracle
runs on that only.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_far_entries import _far_rows
from test_gpu_filtered_rows import _gpu
from test_gpu_list_bins import _bins_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(got, want, tag):
    for g, w in zip(got, want):
        w = torch.from_numpy(np.ascontiguousarray(w)).cuda()
        whole = g.shape[0] // w.shape[0] * w.shape[0]
        assert bool((g[:whole].reshape(-1, *w.shape) == w).all()), tag
        assert bool((g[whole:] == w[: g.shape[0] - whole]).all()), tag


def _tiled(base, N):
    return torch.from_numpy(base).cuda().repeat((N + base.shape[0] - 1) // base.shape[0], 1)[:N].contiguous()


@pytest.mark.parametrize("M, counts", [(1600, (90, 1100)), (2049, (90, 1030)), (3001, (90, 1600)), (4096, (90, 2100)),
                                       (4097, (90, 520, 3100)), (6144, (90, 1030)), (6145, (90, 2000)), (8191, (90,)),
                                       (8192, (90, 24600))])
@pytest.mark.parametrize("k", [1, 64, 140, 256, 257])
def test_fp32_rows(M, k, counts):
    R = _gpu()
    base = np.concatenate([_far_rows(M, 7700 + M), _bins_rows(M, min(k, 200), 7800 + M)[::2]])
    base = np.concatenate([base, np.sort(base[2:4], axis=1), np.round(base[3:6] * 2) / 2]).astype(np.float32)
    want = {"exact": oracle.topk_exact(base, k), "smallest": oracle.topk_exact_smallest(base, k),
            "early": oracle.topk_earlystop(base, k, 5), "early smallest": oracle.topk_earlystop_smallest(base, k, 9),
            "eps": oracle.alg1(base, k, eps_rel=1e-4), "coarse": oracle.alg1(base, k, eps_rel=0.2),
            "dense": [oracle.maxk_dense(base, k)], "early dense": [oracle.maxk_dense(base, k, 8)]}
    for N in counts if k in (64, 256) else counts[:1]:
        x = _tiled(base, N)
        got = {"exact": R.rtopk_rowwise_exact(x, k), "smallest": R.rtopk_rowwise_exact_smallest(x, k),
               "early": R.rtopk_rowwise(x, k, 5), "early smallest": R.rtopk_rowwise_smallest(x, k, 9),
               "eps": R.rtopk_rowwise_eps(x, k, 1e-4, want_iters=True),
               "coarse": R.rtopk_rowwise_eps(x, k, 0.2, want_iters=True), "dense": [R.rtopk_maxk_dense(x, k)],
               "early dense": [R.rtopk_maxk_dense(x, k, 8)]}
        for what in want:
            _check(got[what], want[what], f"{what} {N} x {M} k={k}")
        del got


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M, counts", [(2049, (90, 600)), (4095, (90,)), (4104, (90, 1100)), (8191, (90,)), (8192, (90, 6200))])
def test_16bit_rows(kind, M, counts):
    R = _gpu()
    x = _far_rows(M, 7900 + M)
    base = workloads.to_bits16(np.clip(x, -6e4, 6e4) if kind == "f16" else x, kind)
    exact, early, dtype = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16, torch.float16) if kind == "f16" else (
        R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16, torch.bfloat16)
    for k in (1, 64, 140, 256):
        want = oracle.topk_exact_16(base, kind, k), oracle.topk_earlystop_16(base, kind, k, 8)
        for N in counts:
            d = _tiled(base.view(np.int16), N).view(dtype)
            for got, w in zip((exact(d, k), early(d, k, 8)), want):
                _check((got[0].view(torch.int16), got[1]), (w[0].view(np.int16), w[1]), f"{kind} {N} x {M} k={k}")
