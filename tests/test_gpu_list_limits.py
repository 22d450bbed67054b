"""Rows of 769 to 8192 columns at the largest k that takes the lists of candidates, and one beyond, in every mode, at the
narrowest and widest row of each layout: the rules that send a call to the lists depend on k, the layout and the steps.

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


@pytest.mark.parametrize("M,limits", [(769, (64,)), (1024, (64,)), (1025, (100, 140)), (1536, (100, 140)), (1537, (100, 175)),
                                      (2048, (100, 175)), (2049, (175, 245, 280)), (3072, (175, 245, 280)), (3073, (175, 245)),
                                      (3200, (245, 272, 280)), (3840, (245, 280)), (4097, (48, 245)), (6145, (48, 245)), (8192, (48, 245, 280))])
def test_fp32_rows_around_the_limits(M, limits):
    R = _gpu()
    x = workloads.normal(9, M, seed=9700 + M)
    xd = torch.from_numpy(x).cuda()
    for k in sorted({limit + d for limit in limits for d in (-1, 0, 1)}):
        tag = f"M={M} k={k}"
        _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
        _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
        for mi in (0, 4, 5, 6, 7, 8, 16):
            _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), tag + f" early {mi}")
        ev, ei, et = oracle.alg1(x, k, eps_rel=1e-4)
        got = R.rtopk_rowwise_eps(xd, k, 1e-4, want_iters=True)
        _same(got, (ev, ei), tag + " eps")
        assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"
        for mi in (-1, 4, 8):
            y = R.rtopk_maxk_dense(xd, k, mi)
            assert np.array_equal(y.cpu().numpy().view(np.int32), oracle.maxk_dense(x, k, mi).view(np.int32)), tag + f" dense {mi}"


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", [513, 600, 767, 1024])
def test_16bit_rows_around_the_limits(kind, M):
    R = _gpu()
    b = workloads.to_bits16(workloads.normal(9, M, seed=9800 + M), kind)
    xd = torch.from_numpy(b.view(np.int16)).cuda().view(torch.float16 if kind == "f16" else torch.bfloat16)
    exact, early = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16)
    for limit in (24 * M // 256, 35 * M // 256, 64):
        for k in (limit - 1, limit, limit + 1):
            v, i = exact(xd, k)
            _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k} exact")
            for mi in (6, 7, 8):
                v, i = early(xd, k, mi)
                _same((v.view(torch.int16), i), oracle.topk_earlystop_16(b, kind, k, mi), f"{kind} M={M} k={k} early {mi}")


# A k beyond what the lists can hold costs no more than a little larger one, which never takes them: 2.0 times where every
# row built its lists in vain (3072 columns, k = 420; 2050 columns 1.5 times).
@pytest.mark.parametrize("M,k,beyond", [(3072, 420, 440), (2050, 420, 440), (1538, 280, 300), (3074, 280, 300)])
def test_no_lists_that_cannot_hold(M, k, beyond):
    R = _gpu()
    x = torch.randn(((1 << 25) // M, M), device="cuda")
    a, b = _time(lambda: R.rtopk_rowwise_exact(x, k)), _time(lambda: R.rtopk_rowwise_exact(x, beyond))
    assert a < 1.2 * b, f"{a:.1f} us against {b:.1f}"
