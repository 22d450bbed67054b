"""GPU parity of the backward edge of the MaxK non-linearity (scatter and gather forms) against the CPU
oracle, element by element; the values are bit copies, so the tolerance is 0."""
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


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.int32)


def check(R, N, M, k, seed, u8=False, idx=None, tag=""):
    x = workloads.normal(N, M, seed)
    if idx is None:
        _, idx = oracle.topk_exact(x, k)
    g = workloads.normal(N, k, seed + 1)
    w = workloads.normal(N, M, seed + 2)
    idx_d = torch.from_numpy(idx.astype(np.uint8) if u8 else idx).cuda()
    dense = R.rtopk_maxk_backward(torch.from_numpy(g).cuda(), idx_d, M)
    gath = R.rtopk_maxk_backward_gather(torch.from_numpy(w).cuda(), idx_d)
    torch.cuda.synchronize()
    assert np.array_equal(bits(dense.cpu().numpy()), bits(oracle.maxk_backward(g, idx, M))), f"{tag} scatter"
    assert np.array_equal(bits(gath.cpu().numpy()), bits(oracle.maxk_backward_gather(w, idx))), f"{tag} gather"


SHAPES = [(1, 1, (1,)), (5, 2, (1, 2)), (9, 7, (1, 3, 7)), (33, 63, (1, 8, 63)), (64, 64, (1, 5, 16, 64)),
          (100, 100, (10, 12)), (257, 128, (1, 16, 20, 128)), (31, 130, (13,)), (77, 200, (25, 32)),
          (4099, 256, (1, 16, 31, 32, 33, 64, 65, 128, 255, 256)), (50, 260, (33, 64)), (515, 512, (64, 100)),
          (129, 768, (96,)), (40, 1000, (125, 128)), (259, 1024, (128, 1000)), (33, 1500, (200,)), (67, 2048, (256, 2048)),
          (35, 3000, (64,)), (70, 4096, (64, 1024)), (9, 4095, (7, 512)), (20, 8192, (64, 4097)), (7, 10001, (33, 9000)),
          (5, 32768, (256,)), (3, 65536, (512, 65536))]


@pytest.mark.parametrize("N,M,ks", SHAPES)
def test_backward_small_shapes(N, M, ks):
    R = _gpu()
    for k in ks:
        check(R, N, M, k, seed=N * 13 + M + k, tag=f"N={N} M={M} k={k}")
        if M <= 256:
            check(R, N, M, k, seed=N * 17 + M + k, u8=True, tag=f"u8 N={N} M={M} k={k}")


def test_backward_columns_in_any_order_and_out_of_range_columns():
    R = _gpu()
    N, M, k = 3000, 256, 32
    rng = np.random.Generator(np.random.Philox(5))
    idx = np.stack([rng.permutation(M)[:k] for _ in range(N)]).astype(np.int32)  # distinct, unsorted
    check(R, N, M, k, seed=41, idx=idx, tag="unsorted")
    bad = idx.copy()
    bad[::3, 5] = -1
    bad[::5, 7] = M
    bad[::7, 0] = 2 ** 31 - 1
    bad[::11, 31] = -(2 ** 31)
    check(R, N, M, k, seed=43, idx=bad, tag="out-of-range columns")
    # wide rows (workgroup per row) too
    idx = np.stack([rng.permutation(9000)[:100] for _ in range(40)]).astype(np.int32)
    idx[::2, 3] = 9000
    idx[::3, 4] = -5
    check(R, 40, 9000, 100, seed=45, idx=idx, tag="wide, out-of-range columns")


def test_backward_unaligned_pointers_and_guard_bands():
    R = _gpu()
    N, M, k = 777, 256, 32
    x = workloads.normal(N, M, seed=51)
    _, idx = oracle.topk_exact(x, k)
    g = workloads.normal(N, k, seed=52)
    pad = 1024
    buf = torch.full((N * M + 2 * pad + 1,), 7.5, dtype=torch.float32, device="cuda")
    out = buf[pad + 1:pad + 1 + N * M].view(N, M)  # 4-byte aligned only: chunks cut rows, and the first and the last chunk are partial
    R.rtopk_maxk_backward(torch.from_numpy(g).cuda(), torch.from_numpy(idx).cuda(), M, out)
    torch.cuda.synchronize()
    assert np.array_equal(bits(out.cpu().numpy()), bits(oracle.maxk_backward(g, idx, M)))
    assert (buf[:pad + 1] == 7.5).all() and (buf[pad + 1 + N * M:] == 7.5).all()
    w = workloads.normal(N, M, seed=53)
    wb = torch.empty(N * M + 1, dtype=torch.float32, device="cuda")
    wd = wb[1:].view(N, M)
    wd.copy_(torch.from_numpy(w))
    gbuf = torch.full((N * k + 2 * pad,), 7.5, dtype=torch.float32, device="cuda")
    gv = gbuf[pad:pad + N * k].view(N, k)
    R.rtopk_maxk_backward_gather(wd, torch.from_numpy(idx).cuda(), gv)
    torch.cuda.synchronize()
    assert np.array_equal(bits(gv.cpu().numpy()), bits(oracle.maxk_backward_gather(w, idx)))
    assert (gbuf[:pad] == 7.5).all() and (gbuf[pad + N * k:] == 7.5).all()


def test_backward_round_trip_with_the_forward_pass_full_size():
    # the headline shape, with the columns the forward kernel itself saved (int32 and uint8)
    R = _gpu()
    x = workloads.make("c1_maxk")
    N, M, k = x.shape[0], x.shape[1], 32
    xd = torch.from_numpy(x).cuda()
    for u8 in (False, True):
        vals, idx = (R.rtopk_rowwise_exact_u8 if u8 else R.rtopk_rowwise_exact)(xd, k)
        g = workloads.normal(N, k, seed=61)
        dense = R.rtopk_maxk_backward(torch.from_numpy(g).cuda(), idx, M)
        torch.cuda.synchronize()
        idx_h = idx.cpu().numpy().astype(np.int32)
        assert np.array_equal(bits(dense.cpu().numpy()), bits(oracle.maxk_backward(g, idx_h, M))), f"scatter u8={u8}"
        del dense
        # gathering the forward input at the saved columns returns the forward values
        back = R.rtopk_maxk_backward_gather(xd, idx)
        torch.cuda.synchronize()
        assert torch.equal(back.view(torch.int32), vals.view(torch.int32)), f"gather u8={u8}"
        w = workloads.normal(N, M, seed=62)
        gath = R.rtopk_maxk_backward_gather(torch.from_numpy(w).cuda(), idx)
        torch.cuda.synchronize()
        assert np.array_equal(bits(gath.cpu().numpy()), bits(oracle.maxk_backward_gather(w, idx_h))), f"gather u8={u8}"


def test_backward_empty_batch_and_errors():
    R = _gpu()
    g = torch.empty((0, 32), dtype=torch.float32, device="cuda")
    i = torch.empty((0, 32), dtype=torch.int32, device="cuda")
    assert R.rtopk_maxk_backward(g, i, 256).shape == (0, 256)
    g = torch.zeros((4, 8), dtype=torch.float32, device="cuda")
    i = torch.zeros((4, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(R.RTopKError):
        R.rtopk_maxk_backward(g, i, 4)  # k > M
    with pytest.raises(ValueError):
        R.rtopk_maxk_backward(g, torch.zeros((4, 8), dtype=torch.uint8, device="cuda"), 300)


@pytest.mark.parametrize("M,k", [(1, 1), (2, 1), (31, 31), (33, 3), (100, 65), (129, 1), (251, 100), (256, 129), (257, 5), (683, 300), (1023, 77),
                                 (1025, 1025), (2047, 1), (2047, 2047), (2049, 40), (8193, 600)])
def test_backward_at_any_alignment(M, k):
    """Dense and pair arrays that start anywhere in a 128-byte line; whole and cut chunks, the first and last of the matrix."""
    import ctypes

    R = _gpu()
    lib = R.load_library()
    rng = np.random.default_rng(M * 7 + k)
    for N in (1, 7, 4100) if M <= 683 else (1, 67):
        idx = np.argsort(rng.random((N, M)), axis=1)[:, :k].astype(np.int32)  # any order
        g, w = workloads.normal(N, k, M + N), workloads.normal(N, M, M + N + 1)
        want, want_gather = oracle.maxk_backward(g, idx, M), oracle.maxk_backward_gather(w, idx)
        for u8 in (False, True) if M <= 256 else (False,):
            for shift in (0, 1, 2, 7, 31):
                dense = torch.full((N * M + 96,), 7.5, device="cuda")
                pairs = torch.full((N * k + 96,), 7.5, device="cuda")
                cols = torch.zeros(N * k + 96, device="cuda", dtype=torch.uint8 if u8 else torch.int32)
                cols[shift:shift + N * k] = torch.from_numpy(idx.ravel()).cuda()
                pairs[shift:shift + N * k] = torch.from_numpy(g.ravel()).cuda()
                suffix, ptr = "_u8" if u8 else "", lambda t, s: ctypes.c_void_p(t[s:].data_ptr())
                stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
                args = (ctypes.c_int64(N), ctypes.c_int32(M), ctypes.c_int32(k))
                rc = getattr(lib, "rtopk_maxk_backward" + suffix)(ptr(pairs, shift), ptr(cols, shift), *args, ptr(dense, 2 * shift), stream)
                assert rc == 0
                got = dense.cpu().numpy()
                assert np.array_equal(bits(got[2 * shift:2 * shift + N * M]), bits(want.ravel())), (N, shift, u8)
                assert (got[:2 * shift] == 7.5).all() and (got[2 * shift + N * M:] == 7.5).all(), "wrote outside the matrix"
                dense[shift:shift + N * M] = torch.from_numpy(w.ravel()).cuda()
                pairs.fill_(7.5)
                rc = getattr(lib, "rtopk_maxk_backward_gather" + suffix)(ptr(dense, shift), ptr(cols, shift), *args, ptr(pairs, shift), stream)
                assert rc == 0
                got = pairs.cpu().numpy()
                assert np.array_equal(bits(got[shift:shift + N * k]), bits(want_gather.ravel())), (N, shift, u8)
                assert (got[:shift] == 7.5).all() and (got[shift + N * k:] == 7.5).all(), "wrote outside the pairs"


@pytest.mark.parametrize("N,M,k", [(20011, 251, 31), (60001, 100, 12), (8200, 777, 40), (40003, 250, 100), (140001, 33, 4), (70001, 88, 4),
                                   (16385, 256, 32), (131077, 256, 5), (65541, 512, 7), (16387, 2048, 3), (18000, 1028, 9), (2100, 2047, 33),
                                   (32769, 1100, 2), (32771, 1101, 2), (12281, 440, 209), (3001, 384, 121), (30001, 644, 16), (30001, 640, 16),
                                   (9001, 1184, 304), (3001, 1496, 400), (20001, 96, 5), (5001, 1496, 300), (601, 224, 20), (40001, 1760, 220)])
def test_backward_of_many_rows(N, M, k):
    """Chunks of 2048 floats that cut rows, gathers of several rows to a wavefront at every kind of width, several loads of pairs."""
    import ctypes

    R = _gpu()
    lib = R.load_library()
    rng = np.random.default_rng(N + M)
    first = rng.integers(0, M, (N, 1))
    step = np.array([s for s in range(1, M + 1) if np.gcd(s, M) == 1])[rng.integers(0, 8 if M > 33 else 3, N)][:, None]
    idx = ((first + step * np.arange(k)) % M).astype(np.int32)  # distinct, any order
    g, w = workloads.normal(N, k, M + N), workloads.normal(N, M, M + N + 1)
    want, want_gather = oracle.maxk_backward(g, idx, M), oracle.maxk_backward_gather(w, idx)
    gd = torch.from_numpy(g).cuda()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    args = (ctypes.c_int64(N), ctypes.c_int32(M), ctypes.c_int32(k))
    for u8 in (False, True) if M <= 256 else (False,):
        cols = torch.from_numpy(idx.astype(np.uint8) if u8 else idx).cuda()
        suffix, ptr = "_u8" if u8 else "", lambda t, s: ctypes.c_void_p(t.flatten()[s:].data_ptr())
        for shift in (0, 3):
            dense = torch.full((N * M + 96,), 7.5, device="cuda")
            assert getattr(lib, "rtopk_maxk_backward" + suffix)(ptr(gd, 0), ptr(cols, 0), *args, ptr(dense, 32 + shift), stream) == 0
            got = dense.cpu().numpy()
            assert np.array_equal(bits(got[32 + shift:32 + shift + N * M]), bits(want.ravel())), (shift, u8)
            assert (got[:32 + shift] == 7.5).all() and (got[32 + shift + N * M:] == 7.5).all(), "wrote outside the matrix"
            dense[shift:shift + N * M] = torch.from_numpy(w.ravel()).cuda()
            pairs = torch.full((N * k + 96,), 7.5, device="cuda")
            assert getattr(lib, "rtopk_maxk_backward_gather" + suffix)(ptr(dense, shift), ptr(cols, 0), *args, ptr(pairs, 32 + shift), stream) == 0
            got = pairs.cpu().numpy()
            assert np.array_equal(bits(got[32 + shift:32 + shift + N * k]), bits(want_gather.ravel())), (shift, u8)
            assert (got[:32 + shift] == 7.5).all() and (got[32 + shift + N * k:] == 7.5).all(), "wrote outside the pairs"


def test_backward_of_most_wavefronts():
    """65537 wavefronts of whole 8 KiB and one of a single row: two quads per lane at a time, without a look at the end but in the last."""
    R = _gpu()
    N, M, k = 524289, 256, 32
    w = torch.randn(N, M, device="cuda")
    cols = ((torch.randint(0, M, (N, 1), device="cuda") + 5 * torch.arange(k, device="cuda")) % M).int()
    want = torch.gather(w, 1, cols.long())
    for c in (cols, cols.to(torch.uint8)):
        assert torch.equal(R.rtopk_maxk_backward_gather(w, c), want)
