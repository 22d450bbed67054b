"""GPU parity of early stopping on rows masked with the type's lowest value, where the sum of the search's two bounds
overflows and a threshold of -inf reaches the registers past the row's end as well: k next to the row's width, so that a
repeated column of the last lane's, or one missing, shows.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LOWEST = -3.4028235e38  # of float; of bfloat16, -3.3895314e38, which this does not round to


def _masked_rows(M, lowest):
    rng = np.random.default_rng(M)
    rows = np.full((6, M), lowest, np.float32)
    rows[1, 0] = lowest / 2  # the rest of the row far below its largest entry, which overflows as well
    rows[2, M - 1] = lowest / 4
    rows[3, rng.permutation(M)[: M // 2]] = lowest / 8
    rows[4, ::3] = lowest * np.float32(0.75)
    rows[5, M // 2:] = rng.standard_normal(M - M // 2)  # and one whose sums do not overflow
    return rows


@pytest.mark.parametrize("M", [3, 62, 126, 190, 254, 333, 382, 446, 510, 766, 1022, 2046, 9001, 70001])
def test_fp32_rows(M):
    R = _gpu()
    x = _masked_rows(M, np.float32(LOWEST))
    xd = torch.from_numpy(x).cuda()
    for k in (M - 2, M - 1, M):
        for steps in (1, 2, 8):
            tag = f"M={M} k={k} steps={steps}"
            want = oracle.topk_earlystop(x, k, steps)
            _same(R.rtopk_rowwise(xd, k, steps), want, tag)
            _same(R.rtopk_rowwise_smallest(-xd, k, steps), oracle.topk_earlystop_smallest(-x, k, steps), tag + " smallest")
            if M <= 65536:
                dense = R.rtopk_maxk_dense(xd, k, steps).cpu().numpy()
                assert np.array_equal(dense.view(np.int32), oracle.maxk_dense(x, k, steps).view(np.int32)), tag + " dense"
            if M <= 256:
                v, i = R.rtopk_rowwise_u8(xd, k, steps)
                _same((v, i.to(torch.int32)), want, tag + " byte columns")


@pytest.mark.parametrize("M", [62, 126, 190, 254, 333, 510, 766, 2046, 9001])
def test_bf16_rows(M):
    R = _gpu()
    b = workloads.to_bits16(_masked_rows(M, np.float32(-3.3895314e38)), "bf16")
    xd = torch.from_numpy(b.view(np.int16)).cuda().view(torch.bfloat16)
    for k in (M - 2, M - 1, M):
        for steps in (1, 2, 8):
            v, i = R.rtopk_rowwise_bf16(xd, k, steps)
            _same((v.view(torch.int16), i), oracle.topk_earlystop_16(b, "bf16", k, steps), f"M={M} k={k} steps={steps}")
