"""GPU parity for every number of rows that a wavefront takes: row counts on both sides of the lines between them, the last
wavefront's batch incomplete.  The rows repeat a base of 97, so the oracle runs on those only.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_filtered_rows import _gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BASE = 97
ROWS = (4095, 4097, 8191, 12289, 16385, 24575, 32769, 49151, 98305, 147457, 196609, 393217)


def _tiled(base, N):
    return torch.from_numpy(base).cuda().repeat((N + BASE - 1) // BASE, 1)[:N].contiguous()


def _check(got, want, tag):
    """got: outputs of N rows; want: the oracle's of the base rows."""
    for g, w in zip(got, want):
        w = torch.from_numpy(np.ascontiguousarray(w)).cuda()
        whole = g.shape[0] // BASE * BASE
        assert bool((g[:whole].reshape(-1, *w.shape) == w).all()), tag
        assert bool((g[whole:] == w[: g.shape[0] - whole]).all()), tag


@pytest.mark.parametrize("M", [40, 64, 100, 128, 180, 250, 256, 300, 333, 440, 512, 700, 1000, 1024])
def test_fp32_rows(M):
    R = _gpu()
    base = workloads.normal(BASE, M, 8800 + M)
    base[::7] = np.round(base[::7] * 4) / 4  # tied rows
    k = max(1, M // 8) | 1
    exact, early = oracle.topk_exact(base, k), oracle.topk_earlystop(base, k, 8)
    eps, smallest, dense = oracle.alg1(base, k, eps_rel=1e-4), oracle.topk_exact_smallest(base, k), oracle.maxk_dense(base, k)
    for N in ROWS:
        if N * M > 50_000_000:
            break
        x, tag = _tiled(base, N), f"{N} x {M}"
        _check(R.rtopk_rowwise_exact(x, k), exact, tag + " exact")
        _check(R.rtopk_rowwise(x, k, 8), early, tag + " early")
        _check(R.rtopk_rowwise_eps(x, k, 1e-4, want_iters=True), eps, tag + " eps")
        _check(R.rtopk_rowwise_exact_smallest(x, k), smallest, tag + " smallest")
        _check([R.rtopk_maxk_dense(x, k)], [dense], tag + " dense")
        if M <= 256:
            v, i = R.rtopk_rowwise_u8(x, k, 8)
            _check((v, i.int()), early, tag + " byte columns")


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", [40, 128, 200, 256, 333, 512, 1000])
def test_16bit_rows(kind, M):
    R = _gpu()
    base = workloads.to_bits16(workloads.normal(BASE, M, 8900 + M), kind)
    k = max(1, M // 5)
    exact, early, dtype = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16, torch.float16) if kind == "f16" else (
        R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16, torch.bfloat16)
    want_exact, want_early = oracle.topk_exact_16(base, kind, k), oracle.topk_earlystop_16(base, kind, k, 6)
    for N in ROWS:
        if N * M > 50_000_000:
            break
        x, tag = _tiled(base.view(np.int16), N).view(dtype), f"{kind} {N} x {M}"
        for got, want in ((exact(x, k), want_exact), (early(x, k, 6), want_early)):
            _check((got[0].view(torch.int16), got[1]), (want[0].view(np.int16), want[1]), tag)


@pytest.mark.parametrize("M", [40, 100, 128, 180, 256, 300, 512, 514, 700])
def test_few_steps(M):
    """The lines of Algorithm 2 with few steps."""
    R = _gpu()
    base = workloads.normal(BASE, M, 9000 + M)
    half = workloads.to_bits16(base, "bf16")
    k = max(1, M // 6)
    for steps in (2, 5, 8):
        want, want16 = oracle.topk_earlystop(base, k, steps), oracle.topk_earlystop_16(half, "bf16", k, steps)
        for N in (2049, 4097, 6145, 12289, 16385, 24577, 73729, 110593, 147457):
            if N * M > 30_000_000:
                break
            tag = f"{N} x {M} steps {steps}"
            _check(R.rtopk_rowwise(_tiled(base, N), k, steps), want, tag)
            v, i = R.rtopk_rowwise_bf16(_tiled(half.view(np.int16), N).view(torch.bfloat16), k, steps)
            _check((v.view(torch.int16), i), (want16[0].view(np.int16), want16[1]), tag + " bf16")
