"""Tables of more than 32 tokens on the prefill tile kernel, on both sides of the rules that take them there (33 to 48 tokens: 128
tiles of 256 rows, and a table that is not small against its longest row), with many tiles to a workgroup, products of different row lengths next to each other (the loads run ahead
into products of other sizes), one-step rows, last tiles of one row, and outputs of every kind.  Bit for bit."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _table(bl, M, shapes):
    g = torch.Generator(device=DEV).manual_seed(M)
    items, wants = [], []
    for i, (N, K) in enumerate(shapes):
        W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
        q = torch.zeros((M, bl.bl_padded_k(K)), dtype=torch.int8, device=DEV)
        q[:, :K] = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
        scale = torch.rand(M, generator=g, device=DEV) * 0.01 + 1e-3
        packed, beta = bl.bl_pack_ternary(W, 1, beta=0.03125)
        acc = (q[:, :K].double() @ W.double().t()).to(torch.int32)
        y = acc.float() * (beta * scale)[:, None]
        it = dict(packed=packed, beta=beta, N=N, K=K, q=q, scale=scale, rowsum=q.to(torch.int32).sum(1, dtype=torch.int32))
        if i % 3 == 1:
            it["residual"] = torch.randn((M, N), generator=g, device=DEV)
            y = it["residual"] + y
        if i % 5 != 2:
            it["y"] = torch.full((M, N), 7.0, device=DEV)
        if i % 4 == 2 or "y" not in it:
            it["acc"] = torch.full((M, N), 7, dtype=torch.int32, device=DEV)
        items.append(it)
        wants.append((acc, y))
    return items, wants


@pytest.mark.parametrize("M", [32, 33, 47, 48, 49, 64])
@pytest.mark.parametrize("shapes", [[(700, 2560), (256, 128), (257, 6912), (255, 384), (1, 256)],
                                    [(512, 128)] * 63 + [(256, 250)],                                # 127 tiles
                                    [(512, 128)] * 63 + [(257, 250)],                                # 128
                                    [(2561, 1280), (640, 128), (5120, 256), (1281, 3840)] * 25])     # seven to a workgroup
def test_tables_of_tiles(bl, M, shapes):
    items, wants = _table(bl, M, shapes)
    st = bl.Stack(items, 1, M, DEV)
    tiles = sum(-(-N // 256) for N, _ in shapes)
    assert (st.plan.norm == 3) == (M > 48 or (M > 32 and tiles >= 128))
    for _ in range(2):
        st.run()
    torch.cuda.synchronize()
    for it, (acc, y) in zip(items, wants):
        assert "y" not in it or torch.equal(it["y"], y)
        assert "acc" not in it or torch.equal(it["acc"], acc)


LAYER = [(3840, 2560), (2560, 2560), (13824, 2560), (2560, 6912)]


@pytest.mark.parametrize("M", [33, 48, 49])
@pytest.mark.parametrize("layers,in_tiles", [(3, False), (4, True)])
def test_few_layers_of_long_rows(bl, M, layers, in_tiles):
    """Up to 48 tokens three layers stay with the tokens in LDS, four go to the tiles."""
    items, wants = _table(bl, M, LAYER * layers)
    st = bl.Stack(items, 1, M, DEV)
    assert (st.plan.norm == 3) == (in_tiles or M > 48)
    for _ in range(2):
        st.run()
    torch.cuda.synchronize()
    for it, (acc, y) in zip(items, wants):
        assert "y" not in it or torch.equal(it["y"], y)
        assert "acc" not in it or torch.equal(it["acc"], acc)
