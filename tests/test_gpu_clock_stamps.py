"""The clock counts of a prefill launch (bl_debug_clock_stamps): every kernel that a product can take leaves
them, the split k loop for few tiles as well as the tile kernels."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(70, 300, 128), (64, 1, 64), (512, 2560, 2560), (1024, 3840, 256), (2600, 3300, 320), (2048, 7000, 1024)])
def test_every_launch_leaves_its_counts(layout, M, N, K):
    from paper_2504_12285_amd import binding as bl
    lib = bl.load()
    W = torch.zeros((N, K), dtype=torch.int8, device=DEV)
    packed, beta = bl.bl_pack_ternary(W, layout, beta=0.5)
    q = torch.ones((M, K), dtype=torch.int8, device=DEV)
    scale, rowsum = torch.ones(M, device=DEV), torch.full((M,), K, dtype=torch.int32, device=DEV)
    for want_acc in (False, True):
        stamps = torch.full((2,), -1, dtype=torch.int64, device=DEV)
        assert lib.bl_debug_clock_stamps(stamps.data_ptr()) == 0
        try:
            _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=want_acc)
            torch.cuda.synchronize()
        finally:
            assert lib.bl_debug_clock_stamps(None) == 0
        clocks, ticks = stamps.tolist()
        assert clocks > 0 and ticks > 0 and not y.any()
