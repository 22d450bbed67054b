"""GPU parity of the exact search on lists by bins: the k-th key alone in its bin, tied within its bin, and in bins of more
members than are ranked (64), where the search by thresholds takes over.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bins_rows(M, k, seed):
    """Rows that put the k-th key in bins of every fill."""
    rng = np.random.default_rng(seed)
    rows = []
    for ties in (1, 2, 17, 63, 64, 65, 66, 200):  # values tied at the k-th, the cut in their middle
        x = rng.standard_normal(M).astype(np.float32)
        order = np.argsort(-x, kind="stable")
        first = max(0, k - 1 - ties // 2)
        x[order[first:first + ties]] = x[order[first]]
        rows.append(x)
    x = rng.standard_normal(M).astype(np.float32)
    x[rng.integers(M)] = 1e30  # every other key in the last bin
    rows.append(x)
    x = rng.standard_normal(M).astype(np.float32)
    x[rng.integers(M)] = -3.4e38
    rows.append(x)
    x = np.full(M, -3.4028235e38, np.float32)  # masks of the lowest value: fewer than k keys left, exactly k, more
    for n in (k - 1, k, k + 1, 2 * k):
        y = x.copy()
        y[rng.permutation(M)[:n]] = rng.standard_normal(n).astype(np.float32)
        rows.append(y)
    rows.append(np.zeros(M, np.float32))
    x = rng.standard_normal(M).astype(np.float32)
    x[rng.permutation(M)[: M // 2]] = np.float32(0)
    x[rng.permutation(M)[: M // 4]] = np.float32(-0.0)
    rows.append(np.minimum(x, 0))  # zeros of both signs across the k-th place
    rows.append(np.float32(1) + rng.integers(0, 40, M).astype(np.float32) * np.float32(2.0**-23))  # neighbouring floats
    rows.append(rng.standard_normal(M).astype(np.float32) * np.float32(1e-42))  # subnormals
    return np.stack(rows)


@pytest.mark.parametrize("M", [40001, 65536, 131075, 700001])
@pytest.mark.parametrize("k", [1, 5, 64, 200, 512])
def test_split_rows(M, k):
    R = _gpu()
    x = _bins_rows(M, k, M + k)
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
    _same(R.rtopk_rowwise_exact_smallest(-xd, k), oracle.topk_exact_smallest(-x, k), f"M={M} k={k} smallest")


@pytest.mark.parametrize("M", [900, 1280, 1536, 2048, 4095, 8192, 8200, 16384, 20001, 32768, 40001])
def test_rows_of_one_wavefront_or_workgroup(M):
    R = _gpu()
    lib = R.load_library()
    for k in (1, 5, 33, 64, 140):
        x = _bins_rows(M, k, M + k)
        if M > 32768:  # without scratch memory: one workgroup per row
            xd = torch.from_numpy(x).cuda()
            v, i = torch.empty(x.shape[0], k, device="cuda"), torch.empty(x.shape[0], k, dtype=torch.int32, device="cuda")
            s = torch.cuda.current_stream().cuda_stream
            assert lib.rtopk_rowwise_exact(xd.data_ptr(), x.shape[0], M, k, v.data_ptr(), i.data_ptr(), s) == 0
            _same((v, i), oracle.topk_exact(x, k), f"M={M} k={k}")
        else:
            xd = torch.from_numpy(x).cuda()
            _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
            _same(R.rtopk_rowwise_exact_smallest(-xd, k), oracle.topk_exact_smallest(-x, k), f"M={M} k={k} smallest")
            dense = R.rtopk_maxk_dense(xd, k).cpu().numpy()
            assert np.array_equal(dense.view(np.int32), oracle.maxk_dense(x, k).view(np.int32)), f"M={M} k={k} dense"


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", [1000, 4096, 20001, 50001])
def test_16bit_rows(kind, M):
    R = _gpu()
    exact, dtype = (R.rtopk_rowwise_exact_f16, torch.float16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, torch.bfloat16)
    for k in (1, 33, 64, 140):
        x = _bins_rows(M, k, M + k)
        b = workloads.to_bits16(np.clip(x, -6e4, 6e4) if kind == "f16" else np.clip(x, -3e38, 3e38), kind)
        v, i = exact(torch.from_numpy(b.view(np.int16)).cuda().view(dtype), k)
        _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k}")
