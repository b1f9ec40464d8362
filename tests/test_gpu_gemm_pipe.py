"""The tiles that a prefill product can take (128 x 256, 128 x 192 with one or two workgroups to a unit, 64 x 128, the k loop
split over the waves): rows of one to five k steps, where the loads run ahead over one or more tile borders, with several tiles
to a workgroup; last tiles of one row, of one column and of all but one; half last steps; both layouts and every set of outputs,
in rows that start on whole, half and broken lines.  Bit for bit against an exact integer product."""
import pytest

from test_gpu_gemm_routes import _product

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


SHAPES = [(3969, 8961, k) for k in (64, 128, 192, 320, 640)] + [          # 128 x 256, three tiles and more to a unit
          (2048, 13824, 64), (2049, 13823, 448), (2047, 13825, 2496),     # 128 x 192, two workgroups
          (2048, 2560, 2560), (2047, 2497, 1984), (1921, 2689, 2112),     # 128 x 192, one
          (3000, 1600, 640), (1537, 897, 64), (1600, 1153, 192), (1599, 1151, 4032), (300, 14000, 448),   # 64 x 128
          (1, 1, 64), (65, 33, 128), (64, 32, 6912), (2528, 320, 1877), (63, 4097, 576), (3931, 256, 300)]  # split k loop


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_tiles(bl, layout, M, N, K):
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, layout, M, N, K)
    for _ in range(2):
        _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)
        assert torch.equal(y, y_want)
    acc, _ = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_y=False, K=K)
    assert torch.equal(acc, want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, None, N, K=K)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
    if K % 64 == 0:
        residual = torch.randn((M, N), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
        _, y = bl.bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, N, residual)
        assert torch.equal(y, residual + y_want)


@pytest.mark.parametrize("M,N,K", [(2100, 13700, 192), (1000, 3840, 320), (2048, 2560, 640)])
def test_nothing_beside_the_outputs(bl, M, N, K):
    """Rows past M and what lies behind the last column of the last row stay as they were, in memory around the outputs."""
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, 1, M, N, K)
    pad = 300 * N
    y, acc = torch.full((M * N + 2 * pad,), 7.0, device=DEV), torch.full((M * N + 2 * pad,), 7, dtype=torch.int32, device=DEV)
    for a, b in ((None, y), (acc, None), (acc, y)):
        bl._check(bl.load().bl_gemm_w158a8(packed.data_ptr(), beta.data_ptr(), 1, q.data_ptr(), scale.data_ptr(), rowsum.data_ptr(), M, N, K,
                                           None if a is None else a[pad:].data_ptr(), None if b is None else b[pad:].data_ptr(), None,
                                           torch.cuda.current_stream().cuda_stream), "bl_gemm_w158a8")
        torch.cuda.synchronize()
    for t, w in ((y, y_want), (acc, want)):
        assert torch.equal(t[pad:pad + M * N].view(M, N), w)
        assert (t[:pad] == 7).all() and (t[pad + M * N:] == 7).all()


@pytest.mark.parametrize("M,N,K", [(3969, 4100, 128), (2049, 13824, 384), (1000, 2560, 640), (129, 644, 128), (64, 384, 1280), (65, 13824, 256), (300, 1664, 512)])
def test_fused_epilogues(bl, M, N, K):
    """Residual, and the gate where N allows it: the fp32 value, its bf16 narrowing, the row maxima and the int32 output, in memory
    with something behind it."""
    import ctypes
    packed, beta, q, scale, rowsum, want, y_want = _product(bl, 1, M, N, K)
    residual = torch.randn((M, N), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV)
    for kind in (bl.BL_EPI_RESIDUAL, bl.BL_EPI_RELU2_GATE):
        if kind == bl.BL_EPI_RELU2_GATE and N % 128:
            continue
        gate, NO = kind == bl.BL_EPI_RELU2_GATE, N // 2 if kind == bl.BL_EPI_RELU2_GATE else N
        r = torch.relu(y_want[:, :NO])
        t = (r * r) * y_want[:, NO:] if gate else residual + y_want
        for with_y, with_acc in ((True, False), (False, True)):
            y, xb = torch.full((M * NO + 500,), 7.0, device=DEV), torch.full((M * NO + 500,), 7.0, dtype=torch.bfloat16, device=DEV)
            acc, top = torch.full((M * N + 500,), 7, dtype=torch.int32, device=DEV), torch.zeros(M + 8, device=DEV)
            ep = bl.GemmEpilogue()
            ep.kind, ep.residual, ep.x_bf16, ep.absmax = kind, None if gate else residual.data_ptr(), xb.data_ptr(), top.data_ptr()
            ep.y = y.data_ptr() if with_y else None
            bl._check(bl.load().bl_gemm_w158a8_fused(packed.data_ptr(), beta.data_ptr(), 1, q.data_ptr(), scale.data_ptr(), rowsum.data_ptr(), M, N, K,
                                                     ctypes.byref(ep), acc.data_ptr() if with_acc else None, torch.cuda.current_stream().cuda_stream),
                      "bl_gemm_w158a8_fused")
            torch.cuda.synchronize()
            b = t.to(torch.bfloat16)
            assert torch.equal(xb[:M * NO].view(M, NO), b) and torch.equal(top[:M], b.abs().amax(1).float())
            assert (xb[M * NO:] == 7).all() and (top[M:] == 0).all()
            assert not with_y or torch.equal(y[:M * NO].view(M, NO), t)
            assert not with_acc or torch.equal(acc[:M * N].view(M, N), want)
            assert (y[M * NO if with_y else 0:] == 7).all() and (acc[M * N if with_acc else 0:] == 7).all()
