"""GPU parity of rows that a workgroup searches, on both sides of the lines up to which it takes the lists, at widths that leave
wavefronts partly empty: ordinary, tied, masked and sorted rows.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu, _same
from test_gpu_list_bins import _bins_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rows(M, k):
    x = _bins_rows(M, min(k, M // 2 - 1), 8200 + M)
    rng = np.random.default_rng(8300 + M)
    more = rng.standard_normal((4, M)).astype(np.float32)
    more[1] = np.sort(more[1])
    more[2] = -np.sort(more[2])
    more[3, : M // 2] = -1e9
    return np.concatenate([x, more])


@pytest.mark.parametrize("M, ks", [(1541, (192, 193)), (2051, (256, 257, 307, 308)), (3001, (256, 450, 451)), (3411, (511, 512)),
                                   (4099, (255, 256, 257, 307, 308, 512)), (6001, (450, 451)), (7171, (600, 700)),
                                   (14339, (513, 700)), (20001, (512, 513)), (40001, (500, 1000))])
def test_fp32_rows(M, ks):
    R = _gpu()
    for k in ks:
        x = _rows(M, k)
        xd = torch.from_numpy(x).cuda()
        _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), f"M={M} k={k}")
        _same(R.rtopk_rowwise_exact_smallest(-xd, k), oracle.topk_exact_smallest(-x, k), f"M={M} k={k} smallest")


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M, ks", [(2051, (256, 307, 308)), (3501, (256, 437, 512)), (4099, (308, 512, 513, 614, 615)),
                                   (5337, (800, 801)), (8191, (800, 801, 1000)), (6000, (675, 676)), (9001, (675, 676))])
def test_16bit_rows(kind, M, ks):
    R = _gpu()
    exact, dtype = (R.rtopk_rowwise_exact_f16, torch.float16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, torch.bfloat16)
    for k in ks:
        x = _rows(M, k)
        b = workloads.to_bits16(np.clip(x, -6e4, 6e4) if kind == "f16" else np.clip(x, -3e38, 3e38), kind)
        v, i = exact(torch.from_numpy(b.view(np.int16)).cuda().view(dtype), k)
        _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k}")
