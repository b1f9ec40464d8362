"""The two tile orders of a prefill launch: a rectangle of tiles per XCD, or (where that loads the busiest compute
unit more) one banded sequence of which each XCD takes an eighth.  Shapes of the second kind whose last band is part
filled, for every tile of a plain product and of both fused epilogues (test_gemm_choice.py asks the choice whether these are the tiles that
they go to); every output against an exact integer product."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


def _order(tiles_m, tiles_n, bm, K):
    """(rectangles per column of XCDs or 0, row tiles of a band): the launcher's rule."""
    gm = 1
    while gm < 8 and -(-tiles_m // gm) * bm * K > 3 << 19:
        gm *= 2
    band = -(-tiles_m // gm)
    rect, share = band * -(-tiles_n // (8 // gm)), (tiles_m * tiles_n + 7) // 8
    if (rect + 31) // 32 <= (share + 31) // 32:
        return gm, band
    bands = -(-tiles_m // max(1, (3 << 19) // (bm * K)))
    return 0, -(-tiles_m // bands)


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _inputs(bl, layout, M, N, K):
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    q = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
    scale = torch.rand(M, generator=g, device=DEV) * 0.01 + 1e-3
    packed, beta = bl.bl_pack_ternary(W, layout, beta=0.03125)
    want = (q.float() @ W.float().t()).to(torch.int32)             # (exact: |sum| <= 127 K < 2^24)
    assert 127 * K < 1 << 24
    return packed, beta, q, scale, q.to(torch.int32).sum(1, dtype=torch.int32), want, want.float() * (beta * scale)[:, None], g


# M, N, K of fp32 output alone, place of the kernel, its tile
PLAIN = [(2100, 1664, 1024, 4, 64, 128), (2140, 3712, 1024, 3, 128, 128), (2140, 3712, 1088, 3, 128, 128), (2140, 4992, 2048, 1, 128, 192),
         (2700, 4224, 3328, 1, 128, 192), (3458, 1728, 1024, 2, 128, 192), (2634, 5184, 1024, 0, 128, 256)]
# M, N, K, place of the tile, the tile (of outputs)
RESIDUAL = [(2140, 3712, 1024, 0, 128, 256), (2573, 2432, 1024, 0, 128, 256), (2140, 4992, 2048, 1, 128, 128), (2700, 4224, 3328, 1, 128, 128),
            (2073, 640, 1024, 2, 64, 128)]
GATE = [(2140, 3712, 1024, 0, 128, 128), (2573, 2432, 1024, 0, 128, 128), (2073, 640, 1024, 1, 64, 64)]


def even_share_with_a_part_filled_last_band(M, outputs, K, bm, bn):
    gm, band = _order(-(-M // bm), -(-outputs // bn), bm, K)
    return gm == 0 and band < -(-M // bm) and -(-M // bm) % band != 0


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K,place,bm,bn", PLAIN)
def test_even_shares_with_a_part_filled_last_band(bl, layout, M, N, K, place, bm, bn):
    assert even_share_with_a_part_filled_last_band(M, N, K, bm, bn)
    packed, beta, q, scale, rowsum, want, y_want, g = _inputs(bl, layout, M, N, K)
    _, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N, want_acc=False)
    assert torch.equal(y, y_want)
    acc, y = bl.bl_gemm_w158a8(packed, beta, layout, q, scale, rowsum, N)
    assert torch.equal(acc, want) and torch.equal(y, y_want)
    res = torch.randn((M, N), generator=g, device=DEV)
    _, y = bl.bl_gemm_w158a8_res(packed, beta, layout, q, scale, rowsum, N, res)
    assert torch.equal(y, res + y_want)


@pytest.mark.parametrize("kind,M,N,K,place,bm,bn", [("residual",) + s for s in RESIDUAL] + [("gate",) + s for s in GATE])
def test_fused_epilogues_in_even_shares(bl, kind, M, N, K, place, bm, bn):
    assert even_share_with_a_part_filled_last_band(M, N // 2 if kind == "gate" else N, K, bm, bn)
    packed, beta, q, scale, rowsum, want, y_want, g = _inputs(bl, 1, M, N, K)
    if kind == "residual":
        res = torch.randn((M, N), generator=g, device=DEV)
        t = res + y_want
    else:
        res, r = None, torch.relu(y_want[:, :N // 2])
        t = (r * r) * y_want[:, N // 2:]
    xb, y = torch.empty(t.shape, dtype=torch.bfloat16, device=DEV), torch.empty_like(t)
    absmax = torch.zeros(M, device=DEV)
    bl.bl_gemm_w158a8_fused(packed, beta, 1, q, scale, rowsum, N, bl.BL_EPI_RESIDUAL if res is not None else bl.BL_EPI_RELU2_GATE,
                            xb, absmax, residual=res, y=y)
    assert torch.equal(y, t) and torch.equal(xb, t.to(torch.bfloat16))
    assert torch.equal(absmax, xb.float().abs().amax(1))
