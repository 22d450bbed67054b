"""GPU parity of rows of 16 values per lane (769 to 1024 columns, 16-bit rows from 513) on both sides of the lines up to which a
row alone in its wavefront builds the lists, with few rows and with many: ordinary, tied, masked and sorted ones.  The rows
repeat a base, so the oracle runs on that only.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_few_wide_rows import _check, _tiled
from test_gpu_filtered_rows import _gpu
from test_gpu_list_bins import _bins_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _base(M, k):
    rng = np.random.default_rng(9100 + M + k)
    more = rng.standard_normal((5, M)).astype(np.float32)
    more[1] = np.sort(more[1])
    more[2] = -np.sort(more[2])
    more[3, : M // 2] = -1e9
    more[4] = np.round(more[4] * 4) / 4
    return np.concatenate([_bins_rows(M, min(k, M // 4), 9200 + M)[::2], more])


@pytest.mark.parametrize("M, ks", [(770, (60, 64, 65, 96, 97, 131, 132)), (1000, (83, 84, 111, 112, 125, 126, 140, 141)), (1024, (64, 65, 128, 129, 140))])
@pytest.mark.parametrize("N", [40, 40000])
def test_fp32_rows(M, ks, N):
    R = _gpu()
    for k in ks:
        base = _base(M, k)
        x = _tiled(base, N)
        _check(R.rtopk_rowwise_exact(x, k), oracle.topk_exact(base, k), f"exact {N} x {M} k={k}")
        _check(R.rtopk_rowwise_exact_smallest(x, k), oracle.topk_exact_smallest(base, k), f"smallest {N} x {M} k={k}")
        _check([R.rtopk_maxk_dense(x, k)], [oracle.maxk_dense(base, k)], f"dense {N} x {M} k={k}")
        for steps in (5, 6, 7, 8, 12):
            _check(R.rtopk_rowwise(x, k, steps), oracle.topk_earlystop(base, k, steps), f"early {steps} {N} x {M} k={k}")
        for steps in (7, 8, 12):
            _check([R.rtopk_maxk_dense(x, k, steps)], [oracle.maxk_dense(base, k, steps)], f"dense early {steps} {N} x {M} k={k}")
        del x


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M, ks", [(514, (48, 57, 58, 64, 65, 95, 96, 140)), (600, (56, 57, 75, 76, 111, 112)), (1024, (96, 97, 128, 129, 140, 141))])
@pytest.mark.parametrize("N", [40, 40000])
def test_16bit_rows(kind, M, ks, N):
    R = _gpu()
    exact, early, dtype = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16, torch.float16) if kind == "f16" else (
        R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16, torch.bfloat16)
    for k in ks:
        x = _base(M, k)
        base = workloads.to_bits16(np.clip(x, -6e4, 6e4) if kind == "f16" else np.clip(x, -3e38, 3e38), kind)
        d = _tiled(base.view(np.int16), N).view(dtype)
        wants = [(exact(d, k), oracle.topk_exact_16(base, kind, k), "exact")]
        wants += [(early(d, k, s), oracle.topk_earlystop_16(base, kind, k, s), f"early {s}") for s in (5, 6, 7, 8, 12)]
        for got, w, what in wants:
            _check((got[0].view(torch.int16), got[1]), (w[0].view(np.int16), w[1]), f"{what} {kind} {N} x {M} k={k}")
        del d, wants, got
