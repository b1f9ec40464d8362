"""What NaN and infinities spoil stays bounded: in the quantisers a NaN is passed over by the row maximum and
becomes -127 (every other value of its row as without it), an infinity makes the row's scale infinite; in
packing a quotient that is NaN becomes weight -1 and the padding keeps code 1.  Every kernel that quantises,
against the definition in numpy."""
import numpy as np
import pytest

import oracle
from helpers import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _quantised(x):
    """(q, scale, rowsum) of fp32 rows that hold bf16 values."""
    g = np.maximum(np.where(np.isnan(x), np.float32(0), np.abs(x)).max(1), np.float32(1e-5)).astype(np.float32)
    with np.errstate(invalid="ignore"):
        v = x * (np.float32(127.0) / g)[:, None]
        q = np.where(np.isnan(v), -127, np.clip(np.rint(v), -127, 127)).astype(np.int8)
    return q, g / np.float32(127.0), q.astype(np.int32).sum(1)


def _rows(M, K, seed):
    """Rows of bf16 values; every third has NaN (either sign), every fifth an infinity, one is NaN throughout."""
    rng = np.random.default_rng(seed)
    u = oracle.f32_to_bf16(rng.standard_normal((M, K)).astype(np.float32) * 3)
    for m in range(M):
        if m % 3 == 0:
            u[m, rng.integers(0, K, 2)] = [0x7FC0, 0xFFFF]
            u[m, K - 1] = 0x7FC1
        if m % 5 == 4:
            u[m, rng.integers(0, K, 2)] = [0x7F80, 0xFF80]
    if M > 6:
        u[6, :] = 0x7FC0
    return u, (u.astype(np.uint32) << 16).view(np.float32)


def _check(q, scale, want):
    assert np.array_equal(q.cpu().numpy()[:, :want[0].shape[1]], want[0])
    assert np.array_equal(scale.cpu().numpy().view(np.uint32), want[1].view(np.uint32))


@pytest.mark.parametrize("M,K", [(1, 64), (7, 100), (16, 2560), (11, 2999), (9, 8192), (5, 9024), (8, 9001), (4100, 320), (4099, 70), (4100, 4160)])
def test_quantisers(bl, M, K):
    u, x = _rows(M, K, K + M)
    want = _quantised(x)
    q, s, r = bl.bl_quant_act_int8(to_dev(u))
    _check(q, s, want)
    assert np.array_equal(r.cpu().numpy(), want[2])
    if K % 64 == 0:
        q, s, r = bl.bl_quant_act_ex(bl.make_producer(bl.BL_PROD_F32, to_dev(x)), M, K, torch.device(DEV))
        _check(q, s, want)
        q, s, r = bl.bl_quant_from_absmax(to_dev(u), to_dev(np.where(np.isnan(x), np.float32(0), np.abs(x)).max(1)))
        _check(q, s, want)


@pytest.mark.parametrize("M,K", [(1, 64), (1, 2560), (1, 8192), (2, 2560), (4, 2560), (16, 320), (9, 4096)])
def test_fused_decode(bl, M, K):
    N = 40
    for seed in range(3 if M > 1 else 8):
        u, x = _rows(max(M, 8), K, 7 * K + seed)
        u, x = (u[:M], x[:M]) if M > 1 else (u[seed:seed + 1], x[seed:seed + 1])
        want = _quantised(x)
        W = np.random.default_rng(seed).integers(-1, 2, size=(N, K)).astype(np.int8)
        packed, beta = bl.bl_pack_ternary(to_dev(W), 1, beta=0.5)
        acc, _, q, s = bl.bl_bitlinear_decode(packed, beta, 1, to_dev(u), N, want_acc=True, want_q=True)
        _check(q, s, want)
        assert np.array_equal(acc.cpu().numpy(), want[0].astype(np.int32) @ W.T.astype(np.int32))


@pytest.mark.parametrize("layout", [1, 2, 3])
def test_streamed_decode(bl, layout):
    K, N, rows = 2560, 48, 8
    u, x = _rows(rows, K, 5)
    W = np.random.default_rng(1).integers(-1, 2, size=(N, K)).astype(np.int8)
    packed, beta = bl.bl_pack_ternary(to_dev(W), layout, beta=0.5)
    items = [dict(packed=packed, beta=beta, N=N, K=K, X=to_dev(u[i:i + 1]), acc=torch.empty((1, N), dtype=torch.int32, device=DEV),
                  scale_out=torch.empty(1, device=DEV)) for i in range(rows)]
    bl.Stack(items, layout, 1, torch.device(DEV)).run()
    want = _quantised(x)
    for i, it in enumerate(items):
        assert np.array_equal(it["acc"].cpu().numpy()[0], W.astype(np.int32) @ want[0][i].astype(np.int32))
        assert np.array_equal(it["scale_out"].cpu().numpy().view(np.uint32), want[1][i:i + 1].view(np.uint32))


@pytest.mark.parametrize("kind", [1, 2])
def test_maximum_of_the_fused_epilogues(bl, kind):
    """The row maximum that a product's epilogue folds: a NaN in the residual, or in a row's scale, is passed over."""
    M, N, K = 130, 256, 128
    g = torch.Generator(device=DEV).manual_seed(3)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    packed, beta = bl.bl_pack_ternary(W, 1, beta=0.25)
    q = torch.randint(-127, 128, (M, K), generator=g, device=DEV).to(torch.int8)
    scale = torch.rand(M, generator=g, device=DEV) * 0.01
    res = torch.randn((M, N), generator=g, device=DEV)
    scale[5], res[9, 100], res[77, 255], res[78, 3] = float("nan"), float("nan"), float("inf"), -float("inf")
    n_out = N if kind == 1 else N // 2
    xb = torch.empty((M, n_out), dtype=torch.bfloat16, device=DEV)
    absmax = torch.zeros(M, device=DEV)
    bl.bl_gemm_w158a8_fused(packed, beta, 1, q, scale, q.to(torch.int32).sum(1, dtype=torch.int32), N, kind, xb, absmax,
                            residual=res if kind == 1 else None)
    v = xb.float().abs()
    assert torch.equal(absmax, torch.where(v.isnan(), torch.zeros_like(v), v).amax(1))


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("N,K", [(64, 320), (5, 70), (3, 333), (130, 81)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_packing(bl, layout, N, K, bad):
    W = np.random.default_rng(2).standard_normal((N, K)).astype(np.float32)
    W[N - 1, K // 2] = bad
    Wt = np.full((N, K), -1, np.int8) if np.isnan(bad) else np.where(np.isinf(W), -1, 0).astype(np.int8)
    packed, beta = bl.bl_pack_ternary(to_dev(W), layout)
    b = beta.item()
    assert np.isnan(b) if np.isnan(bad) else b == np.inf
    want = oracle.pack_kmajor(Wt) if layout == 3 else oracle.pack_trit5(Wt) if layout == 2 else oracle.pack_padded(Wt, layout)
    assert np.array_equal(packed.cpu().numpy(), want)


@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("M", [1, 2, 3, 4, 8, 16])
def test_produced_rows(bl, M, norm):
    """Rows that a producer makes in front of the product, for K with and without a second pass: a normalised row with
    a NaN is NaN throughout, one with an infinity is zeros and a NaN; the other rows do not change."""
    for K in (2560, 5952):
        N = 24
        u, x = _rows(max(M, 6), K, 11 + K)
        u, x = u[:M], x[:M].copy()
        if M == 1 and norm:
            x[0, 7] = np.inf
        t = x
        if norm:
            with np.errstate(invalid="ignore", divide="ignore", over="ignore"):
                r = (1.0 / np.sqrt((x.astype(np.float64) ** 2).sum(1) / K + float(np.float32(1e-5)))).astype(np.float32)
                t = x * r[:, None]
            t = (oracle.f32_to_bf16(np.where(np.isnan(t), np.float32(0), t)).astype(np.uint32) << 16).view(np.float32) + np.where(np.isnan(t), np.float32("nan"), np.float32(0))
        want = _quantised(t)
        W = np.random.default_rng(K).integers(-1, 2, size=(N, K)).astype(np.int8)
        packed, beta = bl.bl_pack_ternary(to_dev(W), 1, beta=0.5)
        prod = lambda: bl.make_producer(bl.BL_PROD_F32, xd, norm=norm, eps=1e-5)
        xd = to_dev(x)
        q, s = torch.empty((M, K), dtype=torch.int8, device=DEV), torch.empty(M, device=DEV)
        acc = torch.empty((M, N), dtype=torch.int32, device=DEV)
        acc_want = want[0].astype(np.int32) @ W.T.astype(np.int32)
        if M * (K + 16) <= 96 * 1024:
            item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, q_out=q, scale_out=s, prod=prod())
            bl.bl_bitlinear_decode_group(bl.make_decode_descs([item]), 1, M)
            _check(q, s, want)
            assert np.array_equal(acc.cpu().numpy(), acc_want)
        q, s, _ = bl.bl_quant_act_ex(prod(), M, K, torch.device(DEV))
        _check(q, s, want)
        if M == 1:
            item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc.fill_(7), q_out=torch.empty((1, K), dtype=torch.int8, device=DEV),
                        scale_out=torch.empty(1, device=DEV), prod=prod())
            bl.Stack([item], 1, 1, torch.device(DEV)).run()
            _check(item["q_out"], item["scale_out"], want)
            assert np.array_equal(acc.cpu().numpy(), acc_want)
