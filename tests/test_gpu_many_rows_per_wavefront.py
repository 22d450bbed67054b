"""GPU parity around the lines from two to four rows per wavefront of 257 to 512 columns and from four to eight of 129 to 256: row
counts on both sides of them that leave the last wavefront fewer, the widths and k at which the rule changes.  The rows repeat a base of 97.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu
from test_gpu_rows_per_wavefront import BASE, _check, _tiled

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = (61439, 61440, 61441, 61442, 61443)


@pytest.mark.parametrize("M,k", [(257, 1), (257, 42), (257, 43), (320, 32), (321, 33), (384, 64), (385, 40), (416, 69), (417, 30),
                                 (449, 70), (512, 85)])
def test_fp32_rows(M, k):
    R = _gpu()
    base = workloads.normal(BASE, M, 9300 + M)
    base[::7] = np.round(base[::7] * 4) / 4  # tied rows
    base[5] = 1.5
    exact, smallest = oracle.topk_exact(base, k), oracle.topk_exact_smallest(base, k)
    eps = oracle.alg1(base, k, eps_rel=1e-4)
    early = {steps: oracle.topk_earlystop(base, k, steps) for steps in (0, 5, 8)}
    for N in ROWS:
        x, tag = _tiled(base, N), f"{N} x {M} k {k}"
        _check(R.rtopk_rowwise_exact(x, k), exact, tag + " exact")
        _check(R.rtopk_rowwise_exact_smallest(x, k), smallest, tag + " smallest")
        _check(R.rtopk_rowwise_eps(x, k, 1e-4, want_iters=True), eps, tag + " eps")
        for steps, want in early.items():
            _check(R.rtopk_rowwise(x, k, steps), want, f"{tag} steps {steps}")


@pytest.mark.parametrize("M,k", [(257, 1), (333, 128), (333, 129), (512, 64), (512, 127)])
def test_16bit_rows(M, k):
    R = _gpu()
    for kind, dtype in (("f16", torch.float16), ("bf16", torch.bfloat16)):
        base = workloads.to_bits16(workloads.normal(BASE, M, 9400 + M), kind)
        exact, early = getattr(R, f"rtopk_rowwise_exact_{kind}"), getattr(R, f"rtopk_rowwise_{kind}")
        want_exact, want_early = oracle.topk_exact_16(base, kind, k), oracle.topk_earlystop_16(base, kind, k, 6)
        for N in ROWS:
            x, tag = _tiled(base.view(np.int16), N).view(dtype), f"{kind} {N} x {M} k {k}"
            for got, want in ((exact(x, k), want_exact), (early(x, k, 6), want_early)):
                _check((got[0].view(torch.int16), got[1]), (want[0].view(np.int16), want[1]), tag)


@pytest.mark.parametrize("M,k", [(129, 21), (160, 26), (192, 27), (193, 7), (240, 40), (241, 40), (256, 32)])
def test_narrower_fp32_rows(M, k):
    R = _gpu()
    base = workloads.normal(BASE, M, 9500 + M)
    base[::7] = np.round(base[::7] * 4) / 4
    base[5] = 1.5
    exact, smallest = oracle.topk_exact(base, k), oracle.topk_exact_smallest(base, k)
    eps, early = oracle.alg1(base, k, eps_rel=1e-4), oracle.topk_earlystop(base, k, 8)
    for N in (196607, 196608, 196611, 196613, 262143, 262145, 262150):
        x, tag = _tiled(base, N), f"{N} x {M} k {k}"
        _check(R.rtopk_rowwise_exact(x, k), exact, tag + " exact")
        _check(R.rtopk_rowwise_exact_smallest(x, k), smallest, tag + " smallest")
        _check(R.rtopk_rowwise(x, k, 8), early, tag + " early")
        _check(R.rtopk_rowwise_eps(x, k, 1e-4, want_iters=True), eps, tag + " eps")
