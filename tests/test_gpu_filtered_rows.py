"""GPU parity of the selection from lists of candidates (rows of more than 1024 columns): rows whose lists are whole,
overflow, or do not reach the last threshold; k around the lists' limits; values that crowd, tie or are sorted.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_00822_amd as R

    R.load_library()
    return R


def _rows(M, seed):
    """Rows of every kind: normal, heavy-tailed, sorted either way, nearly all equal, few values, all negative, subnormal."""
    g = np.random.Generator(np.random.Philox(seed))
    x = workloads.normal(10, M, seed)
    x[1] = g.standard_cauchy(M).astype(np.float32)
    x[2] = np.sort(x[2])
    x[3] = -np.sort(-x[3])
    x[4] = 1.0
    x[4, g.integers(0, M, 40)] = np.linspace(0.5, 2.0, 40, dtype=np.float32)
    x[5] = g.integers(-3, 4, M).astype(np.float32)
    x[6] = -np.abs(x[6]) - 100.0
    x[7] *= np.float32(1e-42)
    x[8, : M // 2] = -5.0  # the winners crowd one half
    x[9] = np.where(g.random(M) < 0.5, np.float32(0.0), np.float32(-0.0))
    x[9, g.integers(0, M, 700)] = 1e-3
    return x


def _same(got, want, tag):
    v, i = got[0].cpu().numpy(), got[1].cpu().numpy()
    bad = np.nonzero((i != want[1]).any(axis=1))[0]
    assert bad.size == 0, f"{tag}: columns differ in rows {bad}"
    assert np.array_equal(v.view(np.uint8), want[0].view(np.uint8)), f"{tag}: value bits differ"


# widths of one wavefront per row (24, 32, 48, 64, 96 and 128 values per lane) and of one workgroup per row
@pytest.mark.parametrize("M", [769, 1000, 1023, 1024, 1025, 1536, 2048, 3071, 3072, 4096, 6141, 8192,
                               8193, 12288, 16384, 16385, 24576, 32768, 32771, 49152, 65536])
def test_rows_the_lists_hold_and_rows_they_do_not(M):
    R = _gpu()
    x = _rows(M, 4000 + M)
    xd = torch.from_numpy(x).cuda()
    for k in (1, 2, 33, 64, 65, 140, 141, 210, 211, 280, 281, 420, 421) if M <= 8192 else (1, 2, 33, 255, 256, 257, 511, 512, 513):
        tag = f"M={M} k={k}"
        _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
        _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
        for mi in (4, 5, 8, 13, 40):
            _same(R.rtopk_rowwise(xd, k, mi), oracle.topk_earlystop(x, k, mi), tag + f" early {mi}")
        for eps in (1e-2, 1e-5):
            ev, ei, et = oracle.alg1(x, k, eps_rel=eps)
            got = R.rtopk_rowwise_eps(xd, k, eps, want_iters=True)
            _same(got, (ev, ei), tag + f" eps {eps}")
            assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"
        for mi in (-1, 8):
            y = R.rtopk_maxk_dense(xd, k, mi)
            assert np.array_equal(y.cpu().numpy().view(np.int32), oracle.maxk_dense(x, k, mi).view(np.int32)), tag + f" dense {mi}"


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", [513, 770, 1001, 1024, 1030, 2047, 4096, 8192, 8200, 16384, 32768, 40003, 65536])
def test_16bit_rows_tie_across_the_kth_place(kind, M):
    R = _gpu()
    x = _rows(M, 4100 + M)
    x[1] = np.clip(x[1], -1e4, 1e4)
    b = workloads.to_bits16(x, kind)
    xd = torch.from_numpy(b.view(np.int16)).cuda().view(torch.float16 if kind == "f16" else torch.bfloat16)
    exact, early = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16)
    for k in (1, 64, 256, 512):
        v, i = exact(xd, k)
        _same((v.view(torch.int16), i), oracle.topk_exact_16(b, kind, k), f"{kind} M={M} k={k} exact")
        v, i = early(xd, k, 8)
        _same((v.view(torch.int16), i), oracle.topk_earlystop_16(b, kind, k, 8), f"{kind} M={M} k={k} early")


def test_many_rows_share_the_resident_workgroups():
    # the widest shape walks several rows per workgroup, loading one while another is written; every tenth row falls
    # back to the full-width search, which reads its row again
    R = _gpu()
    x = np.tile(_rows(40000, 4200), (80, 1))
    x[:, 17] = np.arange(800, dtype=np.float32)
    xd = torch.from_numpy(x).cuda()
    _same(R.rtopk_rowwise_exact(xd, 100), oracle.topk_exact(x, 100), "exact")
    _same(R.rtopk_rowwise(xd, 100, 8), oracle.topk_earlystop(x, 100, 8), "early")
