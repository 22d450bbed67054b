"""GPU parity of byte-wide columns at 256 columns, where full rows go four to a wavefront: row counts around its multiples
and around the count from which a wavefront takes more than two rows.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N", [3, 32767, 32768, 32769, 32770, 32771])
def test_full_rows(N):
    R = _gpu()
    x = workloads.normal(N, 256, seed=9900 + N)
    x[N - 1] = np.round(x[N - 1] * 4) / 4
    xd = torch.from_numpy(x).cuda()
    for k in (1, 31, 64, 256):
        v, i = R.rtopk_rowwise_exact_u8(xd, k)
        _same((v, i.int()), oracle.topk_exact(x, k), f"N={N} k={k} exact")
        v, i = R.rtopk_rowwise_u8(xd, k, 8)
        _same((v, i.int()), oracle.topk_earlystop(x, k, 8), f"N={N} k={k} early")
