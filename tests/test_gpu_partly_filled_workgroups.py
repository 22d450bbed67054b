"""GPU parity of the workgroup layouts of every form at the edges of what they hold: the last columns of one layout and the first of the
next, odd widths, k on both sides of the lists.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
from test_gpu_filtered_rows import _gpu, _rows, _same
from test_gpu_parity_16bit import KINDS, TORCH_DT, assert_parity16

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M", [8193, 12287, 12288, 12289, 16385, 24575, 24576, 24577, 32769, 49151, 49152, 49153])
@pytest.mark.parametrize("k", [7, 200, 600])
def test_every_form(M, k):
    R = _gpu()
    x = _rows(M, M + k)
    xd = torch.from_numpy(x).cuda()
    tag = f"M={M} k={k}"
    _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
    _same(R.rtopk_rowwise_smallest(xd, k, 8), oracle.topk_earlystop_smallest(x, k, 8), tag + " smallest early")
    ev, ei, et = oracle.alg1(x, k, eps_rel=1e-3)
    got = R.rtopk_rowwise_eps(xd, k, 1e-3, want_iters=True)
    _same(got, (ev, ei), tag + " eps")
    assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"
    for mi in (-1, 8):
        y, want = R.rtopk_maxk_dense(xd, k, mi).cpu().numpy(), oracle.maxk_dense(x, k, mi)
        assert np.array_equal(y.view(np.uint32), want.view(np.uint32)), f"{tag} dense {mi}"
    for kind in KINDS:
        h = torch.from_numpy(np.clip(x, -6e4, 6e4)).to(TORCH_DT[kind])
        bits = h.view(torch.int16).numpy().view(np.uint16)
        assert_parity16(R, bits, kind, k, "exact", tag=tag)
        assert_parity16(R, bits, kind, k, "early", 8, tag=tag)
