"""GPU parity of early stopping and of a precision where the steps are decided by the k-th and the next key: the next key in a lower
bin, in the same bin, equal to the k-th; neighbouring floats; far apart; as many steps as there are and more.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
from test_gpu_filtered_rows import _gpu, _rows, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gap_rows(M, k, seed):
    """Rows whose k-th and next key lie far apart, next to each other, or are equal."""
    g = np.random.default_rng(seed)
    base = g.standard_normal((8, M)).astype(np.float32)
    base = np.clip(base, -4, 4)
    place = np.argsort(g.random((8, M)), axis=1)
    x = base.copy()
    for r in range(8):
        top, rest = place[r, :k], place[r, k:]
        if r in (0, 1):  # a gap of thousands of bins under the k-th, or half the range
            x[r, top] += 9 if r == 0 else 4000
        elif r == 2:     # every winner in the first bin but one
            x[r, top] = 100 + g.random(k).astype(np.float32)
            x[r, top[-1]] = 50
        elif r in (3, 4):  # k-th and next: neighbouring floats, or equal
            v = np.float32(4.5)
            x[r, top] = v + 1 + g.random(k).astype(np.float32)
            x[r, top[0]] = np.nextafter(v, np.float32(9), dtype=np.float32) if r == 3 else v
            x[r, rest[0]] = v
        elif r == 5:     # k + 1 keys of one value above the others
            x[r, place[r, : k + 1]] = 5
        elif r == 6:     # the (k + 1)-th is the row's minimum
            x[r] = -7
            x[r, top] = g.random(k).astype(np.float32)
        else:            # around zero of both signs
            x[r] = -np.abs(x[r])
            x[r, top] = np.where(np.arange(k) % 2 == 0, np.float32(0.0), np.float32(-0.0))
            x[r, top[: k // 2]] = 1
    return x


def _check(R, x, k, steps, precisions, tag):
    xd = torch.from_numpy(x).cuda()
    for mi in steps:
        _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), f"{tag} early {mi}")
    _same(R.rtopk_rowwise_smallest(xd, k, steps[0]), oracle.topk_earlystop_smallest(x, k, steps[0]), f"{tag} smallest")
    for eps in precisions:
        ev, ei, et = oracle.alg1(x, k, eps_rel=eps)
        got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
        _same(got, (ev, ei), f"{tag} eps {eps}")
        assert np.array_equal(got[2].cpu().numpy(), et), f"{tag} eps {eps} iterations"


@pytest.mark.parametrize("M, k", [(32772, 1), (40000, 63), (65536, 300), (65537, 512), (150001, 20), (400000, 250), (262144, 700)])
def test_split_rows(M, k):
    x = np.concatenate([_rows(M, M + 1), _gap_rows(M, k, M + k)])
    _check(_gpu(), x, k, (11, 12, 13, 30, 400), (1e-3, 9e-4, 1e-5, 0.0), f"M={M} k={k}")


@pytest.mark.parametrize("M, k", [(8200, 257), (9312, 360), (12289, 400), (16384, 512), (16400, 513), (24577, 700), (30000, 1000),
                                  (32768, 1024)])
def test_longer_lists_of_a_workgroup(M, k):
    """The longer lists of the precision-bounded mode; rows that they do not hold; few rows at 1e-6, which take the search over the row."""
    x = np.concatenate([_rows(M, M + 1), _gap_rows(M, k, M + k)])
    x = np.concatenate([x] * (200 // len(x) + 1))
    _check(_gpu(), x, k, (12,), (0.05, 1e-3, 1e-5, 0.0), f"M={M} k={k}")
    _check(_gpu(), x[:40], k, (12,), (1e-2, 1e-6, 0.0), f"M={M} k={k} few")
