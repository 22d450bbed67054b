"""GPU parity of exact mode's longer lists: k on both sides of their limits by width, type and number of rows, tied and heavy-tailed
rows whose k-th key is found in parts of parts, rows that the lists do not hold.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_far_entries import _far_rows
from test_gpu_filtered_rows import _gpu, _same
from test_gpu_list_bins import _bins_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mixed_rows(M, k, seed):
    g = np.random.default_rng(seed)
    x = np.concatenate([_far_rows(M, seed), _bins_rows(M, k, seed)])
    heavy = (g.standard_normal((3, M)) * np.exp(2 * g.standard_normal((3, M)))).astype(np.float32)
    ints = g.integers(0, 64, (3, M)).astype(np.float32) - np.array([[0], [32], [70]], np.float32)
    steps = np.exp(np.round(3 * g.standard_normal((2, M)), 1)).astype(np.float32)  # few values over a wide range
    return np.concatenate([x, heavy, ints, steps, np.sort(x[5:6], axis=1), g.standard_cauchy((1, M))]).astype(np.float32)


@pytest.mark.parametrize("M, k", [(2049, 257), (3000, 375), (4096, 512), (6000, 400), (8192, 257), (8192, 512), (7300, 600), (8192, 700),
                                  (8200, 300), (12288, 512), (15000, 600), (16384, 512), (16384, 700), (24000, 600), (24576, 513),
                                  (32768, 819), (40001, 1000), (50000, 1024), (65536, 1024)])
def test_fp32_rows(M, k):
    R = _gpu()
    x = _mixed_rows(M, k, M + k)
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
    _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), f"M={M} k={k} smallest")
    if M > 32768:  # many rows: the resident workgroups walk them, rows that fail are read again
        many = xd.repeat(20, 1)
        v, i = R.rtopk_rowwise_exact(many, k)
        _same((v[-x.shape[0]:], i[-x.shape[0]:]), oracle.topk_exact(x, k), f"M={M} k={k} last of many")


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M, k", [(2050, 257), (4096, 512), (5000, 600), (8192, 512), (8192, 1000), (12288, 512), (12001, 700),
                                  (24000, 1000), (32768, 1024), (50001, 700), (65536, 1024)])
def test_16bit_rows(kind, M, k):
    R = _gpu()
    x = _mixed_rows(M, k, M + k)
    b = workloads.to_bits16(np.clip(x, -6e4, 6e4) if kind == "f16" else np.clip(x, -3e38, 3e38), kind)
    exact, dtype = (R.rtopk_rowwise_exact_f16, torch.float16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, torch.bfloat16)
    v, i = exact(torch.from_numpy(b.view(np.int16)).cuda().view(dtype), k)
    _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k}")
