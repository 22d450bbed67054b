"""GPU parity of the precision-bounded mode at one to eight and at twelve values per lane: rows whose midpoints cannot round onto a bound
(one loop without that guard), and rows on the other side of that line -- precisions at and below it, values near the type's
limits, a maximum far smaller than the minimum's magnitude.

Selections are copies of inputs and their columns, iterations are whole numbers: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rows(M):
    x = workloads.normal(240, M, 9300 + M)
    x[20:40] *= np.float32(1e37)  # sums of two bounds up to and beyond 2^126
    x[40:50] = np.sign(x[40:50]) * np.float32(3e38)
    x[50:70] *= np.float32(1e-30)
    x[70:80] *= np.float32(1e-42)  # subnormal
    x[80:100] = np.round(x[80:100] * 2)  # whole numbers
    x[100:110] = np.float32(-2.5)  # one value
    x[110:120] = 0.0
    x[120:140] = -np.abs(x[120:140]) - np.float32(1e-6)  # the maximum near zero
    x[140:150, 0] = -1e6  # |min| far above |max|
    x[150:160, -1] = 1e6
    x[160:170, : M // 2] = -np.finfo(np.float32).max
    x[170:180, : M // 2] = -np.inf
    x[180:200] = np.float32(1) + x[180:200] * np.float32(2.0**-21)  # a handful of floats between the bounds
    return x


@pytest.mark.parametrize("M", [17, 64, 65, 128, 150, 192, 200, 256, 300, 333, 384, 400, 448, 500, 512, 513, 600, 768])
@pytest.mark.parametrize("eps_rel", [0.0, 1e-7, 2.0**-21, 2.0**-20, 1e-6, 1e-4, 1e-2, 0.3])
def test_iterations_and_selection(M, eps_rel):
    R = _gpu()
    x = _rows(M)
    xd = torch.from_numpy(x).cuda()
    for k in (1, M // 8, M // 2):
        values, columns, iterations = oracle.alg1(x, k, eps_rel=eps_rel)
        got = R.rtopk_rowwise_eps(xd, k, eps_rel, want_iters=True)
        for g, w in zip(got, (values, columns, iterations)):
            g = g.cpu().numpy()
            bad = [r for r in range(len(g)) if not np.array_equal(np.atleast_1d(g[r]), np.atleast_1d(w[r]))]
            assert not bad, (M, k, eps_rel, bad[:5])
