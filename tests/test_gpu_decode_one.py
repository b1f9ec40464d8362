"""The one-token, one-product decode kernel against the general dot4 kernel (test hook path 1), bit for
bit over every producer, normalisation with and without gains, both layouts, int8 inputs, residuals
and the edges of its size classes; and against the CPU oracle on rows whose maximum it cannot settle
from the sum of squares."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _both(bl, make, outs):
    """Runs the descriptor `make()` through the default kernel and the dot4 kernel; compares every output's bits."""
    got = []
    for path in (0, 1):
        bl._check(bl.load().bl_debug_force_path(path), "bl_debug_force_path")
        try:
            for t in outs:
                t.fill_(-1)
            item, layout = make()
            bl.bl_bitlinear_decode_group(bl.make_decode_descs([item]), layout, 1)
            torch.cuda.synchronize()
            got.append([t.cpu().numpy().view(np.uint8).copy() for t in outs])
        finally:
            bl.load().bl_debug_force_path(0)
    for a, b in zip(*got):
        assert np.array_equal(a, b)


SIZES = [(1, 64), (7, 128), (9, 960), (2048, 64), (2049, 3072), (4096, 3136), (4097, 4096), (300, 4160), (4100, 7168),
         (600, 7232), (4200, 8192), (16385, 256), (16390, 4096), (8200, 5120),
         # the edges of the ranges that go to this kernel
         (4097, 2368), (4352, 2304), (4352, 2368), (8192, 3072), (8192, 3136), (8448, 2112), (8448, 3136), (8449, 4160), (16384, 4096),
         (16385, 3072), (24576, 1024), (24577, 3136)]


@pytest.mark.parametrize("N,K", SIZES)
@pytest.mark.parametrize("kind", ["bf16", "f32", "attn", "residual", "gate", "int8"])
def test_against_the_dot4_kernel(bl, kind, N, K):
    g = torch.Generator(device=DEV).manual_seed(N + 7 * K)
    W = torch.randint(-1, 2, (N, K), generator=g, device=DEV, dtype=torch.int8)
    x = torch.randn(1, 2 * K, generator=g, device=DEV) * 3
    x2 = torch.randn(1, K, generator=g, device=DEV)
    gain = 1.0 + 0.2 * torch.randn(K, generator=g, device=DEV)
    res = torch.randn(1, N, generator=g, device=DEV)
    acc = torch.empty((1, N), dtype=torch.int32, device=DEV)
    y = torch.empty((1, N), device=DEV)
    q = torch.empty((1, K), dtype=torch.int8, device=DEV)
    sc, aux = torch.empty(1, device=DEV), torch.empty((1, K), device=DEV)
    for layout in (0, 1):
        packed, beta = bl.bl_pack_ternary(W, layout, beta=0.03)
        for norm, with_gain in ((False, False), (True, False), (True, True)):
            if kind == "int8" and norm:
                continue
            kw = dict(norm=norm, gain=gain if with_gain else None, eps=1e-5)
            hd = 64 if K % 64 == 0 else 16
            heads = K // hd
            kv = heads // 2 if heads % 2 == 0 else heads
            qkv = torch.cat([x, x2, x], 1)[:, :(heads + 2 * kv) * hd].contiguous()
            prod = {"bf16": lambda: bl.make_producer(bl.BL_PROD_BF16, xb, **kw),
                    "f32": lambda: bl.make_producer(bl.BL_PROD_F32, x, **kw),
                    "attn": lambda: bl.make_producer(bl.BL_PROD_ATTN_V, qkv, n_q=heads, n_kv=kv, head_dim=hd, **kw),
                    "residual": lambda: bl.make_producer(bl.BL_PROD_RESIDUAL, x, x2, aux, **kw),
                    "gate": lambda: bl.make_producer(bl.BL_PROD_RELU2_GATE, x, **kw)}
            xb = x[:, :K].to(torch.bfloat16).contiguous()
            item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, y=y, residual=res if with_gain or layout else None)
            outs = [acc, y]
            if kind == "int8":
                item["q"], item["scale"], item["rowsum"] = bl.bl_quant_act_int8(xb)
            else:
                item.update(prod=prod[kind](), q_out=q, scale_out=sc, fixed_scale=0.0 if layout else 0.5)
                outs += [q, sc] + ([aux] if kind == "residual" else [])
            _both(bl, lambda: (item, layout), outs)


@pytest.mark.parametrize("case", ["midpoint", "tiny", "huge gain", "zero", "large"])
def test_rows_whose_maximum_is_taken_directly(bl, case):
    """Rows outside the bound's range (tiny, huge gain, zero), and ordinary ones with large values; the rows on a bf16
    rounding boundary are those of test_maxima_on_both_sides_of_a_rounding_boundary."""
    K, N = 2560, 40
    rng = np.random.default_rng(5)
    t = rng.standard_normal(K).astype(np.float32)
    gain = np.ones(K, np.float32)
    if case == "midpoint":                       # many rows, their largest values 2^-12 apart
        rows = [t * np.float32(1) for _ in range(64)]
        for i, r_ in enumerate(rows):
            r_[17] = np.float32(8.0) + np.float32(i) * np.float32(2.0 ** -9)
    elif case == "tiny":
        rows = [(t * np.float32(1e-30)), (t * np.float32(1e-38))]
    elif case == "huge gain":
        gain[3] = np.float32(2.0 ** 90)
        rows = [t]
    elif case == "zero":
        rows = [t * np.float32(0)]
    else:
        rows = [t * np.float32(1e18)]
    W = rng.integers(-1, 2, size=(N, K)).astype(np.int8)
    packed, beta = bl.bl_pack_ternary(torch.from_numpy(W).to(DEV), 1, beta=0.5)
    q = torch.empty((1, K), dtype=torch.int8, device=DEV)
    acc, sc = torch.empty((1, N), dtype=torch.int32, device=DEV), torch.empty(1, device=DEV)
    for row in rows:
        xd, gd = torch.from_numpy(row.reshape(1, K)).to(DEV), torch.from_numpy(gain).to(DEV)
        item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, q_out=q, scale_out=sc,
                    prod=bl.make_producer(bl.BL_PROD_F32, xd, norm=True, gain=gd, eps=1e-5))
        _both(bl, lambda: (item, 1), [acc, q, sc])
        X = oracle.rmsnorm_rows(row.reshape(1, K), gain, 1e-5)
        q_o, s_o, _ = oracle.quant_act(X)
        assert np.array_equal(q.cpu().numpy(), q_o)
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), s_o.view(np.uint32))


def _settled(c):
    """Whether the kernel settles the row maximum from c = fl(r * max|t*gain|): both ends of the interval narrow to the same bf16."""
    f = np.float32
    ends = np.array([f(c * f(1.0 - 2.0 ** -20)), f(c * f(1.0 + 2.0 ** -20))], np.float32)
    lo, hi = oracle.f32_to_bf16(ends)
    return lo == hi and 2.0 ** -60 <= c <= 2.0 ** 120


def _rows_around_a_boundary(K, g):
    """Rows whose largest value is walked, one fp32 at a time, over the place where its normalised value lies in the
    middle of two bf16.  g: its gain.  Yields (row, settled)."""
    f = np.float32
    t = np.random.default_rng(5).standard_normal(K).astype(np.float32)
    t[17] = 0.0
    S = float((t.astype(np.float64) ** 2).sum())
    for mid in (4.015625, 4.046875, 7.984375, 8.03125 + 2.0 ** -5):     # odd multiples of half a bf16 step
        p = mid * np.sqrt((S / K + 1e-5) / (float(g) ** 2 - mid * mid / K))
        for step in range(-24, 25):
            row = t.copy()
            row[17] = (np.array([p], np.float32).view(np.int32) + step).view(np.float32)[0]
            r = f(1.0 / np.sqrt((row.astype(np.float64) ** 2).sum() / K + float(f(1e-5))))
            yield row, _settled(f(r * abs(f(row[17] * g))))


@pytest.mark.parametrize("g", [1.0, 1.3749, -0.8])
def test_maxima_on_both_sides_of_a_rounding_boundary(bl, g):
    K, N = 2560, 40
    gain = np.full(K, 0.125, np.float32)
    gain[17] = g
    W = np.random.default_rng(6).integers(-1, 2, size=(N, K)).astype(np.int8)
    packed, beta = bl.bl_pack_ternary(torch.from_numpy(W).to(DEV), 1, beta=0.5)
    q = torch.empty((1, K), dtype=torch.int8, device=DEV)
    acc, sc = torch.empty((1, N), dtype=torch.int32, device=DEV), torch.empty(1, device=DEV)
    gd = torch.from_numpy(gain).to(DEV)
    direct, largest = 0, set()
    for row, settled in _rows_around_a_boundary(K, np.float32(g)):
        direct += not settled
        xd = torch.from_numpy(row.reshape(1, K)).to(DEV)
        item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, q_out=q, scale_out=sc,
                    prod=bl.make_producer(bl.BL_PROD_F32, xd, norm=True, gain=gd, eps=1e-5))
        bl.bl_bitlinear_decode_group(bl.make_decode_descs([item]), 1, 1)
        q_o, s_o, _ = oracle.quant_act(oracle.rmsnorm_rows(row.reshape(1, K), gain, 1e-5))
        assert np.array_equal(q.cpu().numpy(), q_o)
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), s_o.view(np.uint32))
        largest.add(float(s_o[0]))
    assert 16 <= direct <= 4 * 49 - 16 and len(largest) >= 6           # (conditions of the rows: both ways are taken, both sides met)


def test_largest_values_beyond_the_range_of_the_shortcut(bl):
    """max|t*gain| > 2^120: the row maximum is taken itself."""
    K, N = 2560, 40
    row = (np.random.default_rng(8).standard_normal((1, K)) * 3e36).astype(np.float32)
    assert np.abs(row).max() > 2.0 ** 120
    W = np.random.default_rng(6).integers(-1, 2, size=(N, K)).astype(np.int8)
    packed, beta = bl.bl_pack_ternary(torch.from_numpy(W).to(DEV), 1, beta=0.5)
    q, sc = torch.empty((1, K), dtype=torch.int8, device=DEV), torch.empty(1, device=DEV)
    acc = torch.empty((1, N), dtype=torch.int32, device=DEV)
    xd = torch.from_numpy(row).to(DEV)
    item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, q_out=q, scale_out=sc,
                prod=bl.make_producer(bl.BL_PROD_F32, xd, norm=True, eps=1e-5))
    bl.bl_bitlinear_decode_group(bl.make_decode_descs([item]), 1, 1)
    q_o, s_o, _ = oracle.quant_act(oracle.rmsnorm_rows(row, None, 1e-5))
    assert np.array_equal(q.cpu().numpy(), q_o) and np.array_equal(sc.cpu().numpy().view(np.uint32), s_o.view(np.uint32))
