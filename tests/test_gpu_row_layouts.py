"""GPU parity of the row layouts: widths around every edge of a layout (values per lane, groups of mixed width,
the lane whose group straddles the row's end), rows that start at any element, any k, against the oracle.

Selections are copies of inputs and their columns: tolerance 0.
"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one below, at and above the edges of the layouts, every remainder modulo 8, and each family's widest rows
WIDTHS = (1, 2, 3, 5, 63, 64, 65, 66, 127, 128, 129, 130, 191, 192, 193, 195, 255, 256, 257, 258, 319, 320, 321, 323,
          383, 384, 385, 386, 387, 447, 448, 449, 451, 510, 511, 512, 513, 514, 765, 767, 769, 1023, 1025, 1026, 1537,
          2047, 2049, 3071, 3073, 4093, 4097, 6143, 6145, 8190, 8191, 8193, 8197, 12287, 12291, 16383, 16385, 24575,
          24577, 32767, 32769, 49153, 65533, 65535)
STREAMED = (65537, 65538, 65539, 131075)


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_00822_amd as R

    R.load_library()
    return R


def _rows(M):
    return 37 if M <= 1024 else (9 if M <= 8192 else 3)


def _ks(M):
    return sorted({1, min(M, 7), max(1, M // 8 | 1) if M // 8 | 1 <= M else 1, max(1, min(M, 300) - 1)})


def _on_gpu(x, shift):
    """x on the GPU, starting `shift` elements into its buffer, with guard values around it."""
    t = torch.from_numpy(np.ascontiguousarray(x))
    buf = torch.full((x.size + 64,), 3e38 if t.dtype == torch.float32 else 0x7B7B, dtype=t.dtype, device="cuda")
    view = buf[shift:shift + x.size].view(x.shape)
    view.copy_(t)
    return view


def _same(got, want, tag):
    v, i = (t.cpu().numpy() for t in got[:2])
    assert np.array_equal(i.astype(np.int32), want[1]), f"{tag}: columns differ"
    assert np.array_equal(v.view(want[0].dtype).view(np.uint8), want[0].view(np.uint8)), f"{tag}: value bits differ"


@pytest.mark.parametrize("M", WIDTHS + STREAMED)
def test_fp32_rows_of_any_width_and_alignment(M):
    R = _gpu()
    N = _rows(M)
    for x, shift in ((workloads.normal(N, M, seed=3000 + M), M % 4), (workloads.small_ints(N, M, 3001 + M, span=6), 1)):
        xd = _on_gpu(x, shift)
        for k in _ks(M):
            tag = f"M={M} k={k} shift={shift}"
            _same(R.rtopk_rowwise_exact(xd, k), oracle.topk_exact(x, k), tag + " exact")
            _same(R.rtopk_rowwise(xd, k, 6), oracle.topk_earlystop(x, k, 6), tag + " early")
            _same(R.rtopk_rowwise_exact_smallest(xd, k), oracle.topk_exact_smallest(x, k), tag + " smallest")
            ev, ei, et = oracle.alg1(x, k, eps_rel=1e-3)
            got = R.rtopk_rowwise_eps(xd, k, 1e-3, want_iters=True)
            _same(got, (ev, ei), tag + " eps")
            assert np.array_equal(got[2].cpu().numpy(), et), tag + " iterations"
            if M <= 256:
                _same(R.rtopk_rowwise_exact_u8(xd, k), oracle.topk_exact(x, k), tag + " uint8")
            if M <= 65536:
                for mi in (-1, 5):
                    buf = torch.full((N * M + 8,), -7.0, device="cuda")
                    out = buf[3:3 + N * M].view(N, M)
                    R.rtopk_maxk_dense(xd, k, mi, out)
                    assert np.array_equal(out.cpu().numpy().view(np.int32), oracle.maxk_dense(x, k, mi).view(np.int32)), tag + f" dense {mi}"
                    assert bool((buf[:3] == -7.0).all()) and bool((buf[3 + N * M:] == -7.0).all()), tag + " dense guard"


@pytest.mark.parametrize("kind", ("f16", "bf16"))
@pytest.mark.parametrize("M", WIDTHS)
def test_16bit_rows_of_any_width_and_alignment(kind, M):
    R = _gpu()
    x = workloads.to_bits16(workloads.normal(_rows(M), M, seed=3100 + M), kind)
    dt = torch.float16 if kind == "f16" else torch.bfloat16
    xd = _on_gpu(x.view(np.int16), M % 8).view(dt)
    exact, early = (R.rtopk_rowwise_exact_f16, R.rtopk_rowwise_f16) if kind == "f16" else (R.rtopk_rowwise_exact_bf16, R.rtopk_rowwise_bf16)
    for k in _ks(M):
        v, i = exact(xd, k)
        _same((v.view(torch.int16), i), oracle.topk_exact_16(x, kind, k), f"{kind} M={M} k={k} exact")
        v, i = early(xd, k, 6)
        _same((v.view(torch.int16), i), oracle.topk_earlystop_16(x, kind, k, 6), f"{kind} M={M} k={k} early")


@pytest.mark.parametrize("k", (1, 2, 3, 5, 6, 31, 32, 33))
def test_pairs_leave_whole_whatever_k_is(k):
    # groups of four pairs shared by two wavefronts, the first and last rows of a launch, guard bands
    R = _gpu()
    for N, M in ((1, 64), (33, 64), (1001, 100), (32771, 70), (517, 256), (33000, 256), (129, 333), (65, 1000)):
        x = workloads.normal(N, M, seed=3200 + N + k)
        xd = torch.from_numpy(x).cuda()
        vb = torch.full((N * k + 32,), 9.0, device="cuda")
        ib = torch.full((N * k + 32,), -9, dtype=torch.int32, device="cuda")
        v, i = vb[16:16 + N * k].view(N, k), ib[16:16 + N * k].view(N, k)
        _same(R.rtopk_rowwise_exact(xd, k, v, i), oracle.topk_exact(x, k), f"N={N} M={M} k={k}")
        for b, g in ((vb, 9.0), (ib, -9)):
            assert bool((b[:16] == g).all()) and bool((b[16 + N * k:] == g).all()), f"N={N} M={M} k={k}: guard band"
