"""The tiles that a prefill product can take (128 x 256, 128 x 192 with one or two workgroups to a unit, 128 x 128, 64 x 128, the k loop
split over the waves): rows of one to five k steps, where the loads run ahead over one or more tile borders, with several tiles
to a workgroup; last tiles of one row, of one column and of all but one; half last steps; both layouts and every set of outputs,
in rows that start on whole, half and broken lines.  Bit for bit against an exact integer product.  The lists are by the kernel that
fp32 output alone goes to (its place in the choice's list; test_gemm_choice.py asks the choice)."""
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


TILES = {
    0: [(3071, 8191, 320), (3072, 8192, 448), (1793, 8449, 448), (1921, 7937, 640), (1407, 8959, 1984)],        # 128 x 256
    1: [(2815, 4415, 448), (2817, 5761, 640), (2816, 4416, 1088), (2689, 4415, 1984)],                          # 128 x 192, two workgroups
    2: [(2048, 2560, 2560), (2047, 2497, 1984), (1921, 2689, 2112), (513, 7297, 1984)],                         # 128 x 192, one
    3: [(2049, 8833, 448), (2177, 8321, 640), (3073, 7681, 1088), (2047, 13825, 2496)],                         # 128 x 128
    4: [(3969, 8961, 64), (3969, 8961, 128), (3969, 8961, 192), (2048, 13824, 64), (3000, 1600, 640), (1537, 897, 64),
        (1600, 1153, 192), (1599, 1151, 4032), (300, 14000, 448), (3931, 256, 300)],                            # 64 x 128
    5: [(1, 1, 64), (65, 33, 128), (64, 32, 6912), (2528, 320, 1877), (63, 4097, 576)]}                         # split k loop
BETWEEN = [(3969, 8961, 320), (3969, 8961, 640), (2049, 13823, 448)]              # where two kernels are estimated the same
SHAPES = [s for shapes in TILES.values() for s in shapes] + BETWEEN
GUARDED = {0: [(1793, 8449, 448)], 1: [(2817, 5761, 640)], 2: [(2047, 2497, 1984)], 3: [(2177, 8321, 640)],
           4: [(2100, 13700, 192), (1000, 3840, 320), (2048, 2560, 640)], 5: [(395, 1601, 640)]}
# fused epilogues by their tiles: residual 128 x 256, 128 x 128, 64 x 128; gate 128 x 128, 64 x 64 (of outputs)
RESIDUAL = {0: [(2047, 4060, 256), (3073, 2536, 384), (1153, 12060, 1280)], 1: [(895, 9340, 1280), (3201, 2424, 1280)],
            2: [(129, 644, 128), (64, 384, 1280), (65, 13824, 256), (300, 1664, 512), (1000, 2560, 640)]}
GATE = {0: [(2049, 13824, 384), (1919, 12032, 1280), (3201, 12544, 128)],
        1: [(64, 384, 1280), (65, 13824, 256), (300, 1664, 512), (1000, 2560, 640)]}
FUSED = sorted({s for shapes in (*RESIDUAL.values(), *GATE.values()) for s in shapes} | {(3969, 4100, 128)})


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


@pytest.mark.parametrize("M,N,K", [s for shapes in GUARDED.values() for s in shapes])
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


@pytest.mark.parametrize("M,N,K", FUSED)
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
