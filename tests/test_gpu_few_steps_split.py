"""GPU parity of early stopping with one to seven steps on rows of more than 65536 columns: the lists of split rows decide the steps, and
the merging workgroup writes what lies below their floor from the row, in chunks of 16384 columns.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
from test_gpu_filtered_rows import _gpu, _rows, _same
from test_gpu_split_large_k import _large_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M, k", [(65537, 1), (65540, 64), (81920, 500), (98303, 1024), (131073, 257), (262144, 16), (400003, 700),
                                  (1 << 20, 900)])
def test_rows_written_from_the_row_and_from_the_lists(M, k):
    R = _gpu()
    x = np.concatenate([_rows(M, M + k)[:6], _large_rows(M, k, M - k)[-5:]])
    late = np.full((1, M), -1.0, np.float32)  # the k-th key at or above the threshold is the row's last column
    late[0, M - k:] = 1.0
    tail = np.full((1, M), np.finfo(np.float32).min, np.float32)  # a masked row whose last threshold is below every key but these
    tail[0, : k + 5] = np.arange(k + 5)
    x = np.concatenate([x, late, tail])
    xd = torch.from_numpy(x).cuda()
    for mi in range(1, 8):
        _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), f"M={M} k={k} early {mi}")
    for mi in (2, 5):
        _same(R.rtopk_rowwise_smallest(xd, k, mi), oracle.topk_earlystop_smallest(x, k, mi), f"M={M} k={k} smallest early {mi}")
