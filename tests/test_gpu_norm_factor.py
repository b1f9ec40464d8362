"""The normalisation factor r = fp32(1 / sqrt(ss/K + eps)) of the one-token decode kernel, bit for bit: rows whose
factor lies within 2^-53 (relative) of an fp32 rounding midpoint, and rows whose sum is zero with
eps = 0 (r is infinite).  The rows have two non-zero values a and b (K = 64, eps = 0), so that their fp64 sum is
exact in every order and r is fixed by IEEE alone."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"

# bit patterns of (a, b); found by going through all a in [1, 2) for random b in [0.5, 1)
ROWS = [
    (0x3f8ef49a, 0x3f3dfee8), (0x3fcc9166, 0x3f1c4446), (0x3f84213b, 0x3f714b09), (0x3fbbbe4e, 0x3f1ca035), (0x3fef8852, 0x3f6a6900), (0x3fcce382, 0x3f1888a7),
    (0x3f8b87b7, 0x3f51bdd9), (0x3fab44d1, 0x3f68e76e), (0x3fdfd6e1, 0x3f68e76e), (0x3ff72a5e, 0x3f2ee353), (0x3fd71155, 0x3f3c572a), (0x3f87a07e, 0x3f5aae76),
    (0x3ff4c6ca, 0x3f6fb5ce), (0x3fe0d515, 0x3f607cf4), (0x3fecddbf, 0x3f390e6d), (0x3fe1b39d, 0x3f781d90), (0x3fe73891, 0x3f65e725), (0x3fc4cbdd, 0x3f0708b2),
    (0x3f9556bf, 0x3f77cddf), (0x3fe14c6e, 0x3f5629ab), (0x3fc771d4, 0x3f5b9dcf), (0x3fa89f17, 0x3f426182), (0x3fcb102d, 0x3f6a77b7), (0x3f9ed61b, 0x3f24846c),
    (0x3fde54dd, 0x3f40ffe8), (0x3feefc52, 0x3f1d8638), (0x3fb4d9bf, 0x3f501590), (0x3f909b20, 0x3f14226a), (0x3f813606, 0x3f3b7e23), (0x3fa4f4ac, 0x3f781cb6),
    (0x3ff72613, 0x3f68e3cf), (0x3fa66ff9, 0x3f25b115), (0x3fb3eba4, 0x3f26a36a), (0x3f87fce2, 0x3f271adb), (0x3fd11308, 0x3f0cdb5c), (0x3ff68056, 0x3f2c3538),
    (0x3fee08eb, 0x3f1102b8), (0x3fcd5fec, 0x3f1fa61d), (0x3fdbc6cc, 0x3f6eff47), (0x3fdeed3a, 0x3f28012e), (0x3f807acf, 0x3f4a8b25), (0x3f9c5048, 0x3f545285),
    (0x3ffb835a, 0x3f686e60), (0x3f886849, 0x3f4545b2), (0x3fd8e61c, 0x3f5354ab), (0x3f8c9073, 0x3f38fb7f), (0x3f8e41de, 0x3f4cfaba), (0x3f9b8704, 0x3f27129b),
    (0x3fe5c431, 0x3f146a88), (0x3fd7b0bf, 0x3f432ef6), (0x3ff89e1b, 0x3f178c7d), (0x3fa5eb95, 0x3f33ba97), (0x3ff6e579, 0x3f09b9bf), (0x3f8fba43, 0x3f0d533b),
    (0x3f89f643, 0x3f2d3192), (0x3fdd097b, 0x3f7efdad), (0x3ffe1059, 0x3f6494ae), (0x3fc08d07, 0x3f38da41), (0x3faa6bd1, 0x3f51836c), (0x3f8f0f61, 0x3f002028),
    (0x3f8cbe77, 0x3f587884), (0x3f9fd31a, 0x3f216fb2), (0x3fff13c7, 0x3f1352b0), (0x3f96e465, 0x3f618109),
]


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _bf16(x):
    return (oracle.f32_to_bf16(np.array([x], np.float32)).astype(np.uint32) << 16).view(np.float32)[0]


def _row(a, b):
    """(row, gain, r): the gain puts bf16((t*r)*gain) of the row's largest value on different sides of a bf16
    midpoint for r and for each of its neighbours, where such a gain exists."""
    f = np.float32
    r = f(1.0 / np.sqrt((float(a) * float(a) + float(b) * float(b)) / 64.0))
    out = []
    for other in (np.nextafter(r, f(0)), np.nextafter(r, f(9))):
        for at, t in enumerate((a, b)):
            p, p2 = f(t * r), f(t * other)
            if p == p2:
                continue
            g = f(f(1.00390625) / p)
            for step in range(-6, 7):
                gain = np.array([int(g.view(np.uint32)) + step], np.uint32).view(np.float32)[0]
                if _bf16(f(p * gain)) != _bf16(f(p2 * gain)):
                    out.append((at, gain))
                    break
    return r, out


def _run(bl, row, gain, path):
    K, N = 64, 4
    W = torch.ones((N, K), dtype=torch.int8, device=DEV)
    packed, beta = bl.bl_pack_ternary(W, 1, beta=0.5)
    q = torch.empty((1, K), dtype=torch.int8, device=DEV)
    acc, sc = torch.empty((1, N), dtype=torch.int32, device=DEV), torch.empty(1, device=DEV)
    x, g = torch.from_numpy(row.reshape(1, K)).to(DEV), torch.from_numpy(gain).to(DEV)
    item = dict(packed=packed, beta=beta, N=N, K=K, acc=acc, q_out=q, scale_out=sc,
                prod=bl.make_producer(bl.BL_PROD_F32, x, norm=True, gain=g, eps=0.0))
    bl._check(bl.load().bl_debug_force_path(path), "bl_debug_force_path")
    try:
        bl.bl_bitlinear_decode_group(bl.make_decode_descs([item]), 1, 1)
        torch.cuda.synchronize()
    finally:
        bl.load().bl_debug_force_path(0)
    return q.cpu().numpy(), sc.cpu().numpy().view(np.uint32), acc.cpu().numpy()


def test_factors_at_a_rounding_midpoint(bl):
    seen = wrong = 0
    for ab, bb in ROWS:
        a, b = np.array([ab, bb], np.uint32).view(np.float32)
        r, gains = _row(a, b)
        for at, g in gains:
            row, gain = np.zeros(64, np.float32), np.full(64, 0.25, np.float32)
            row[0], row[1] = a, b
            gain[at] = g
            gain[1 - at] = 2.0 ** -6
            X = oracle.f32_to_bf16((row * r) * gain).reshape(1, 64)
            q_o, s_o, _ = oracle.quant_act(X)
            q, s, _ = _run(bl, row, gain, 0)
            seen += 1
            wrong += not (np.array_equal(q, q_o) and np.array_equal(s, s_o.view(np.uint32)))
    assert seen >= 64                              # (a condition of the inputs, not of the kernel)
    assert wrong == 0, "%d of %d" % (wrong, seen)


def test_zero_row_without_eps(bl):
    """r is infinite and every product NaN: undefined as a result, but the same on every route."""
    row, gain = np.zeros(64, np.float32), np.ones(64, np.float32)
    got, want = _run(bl, row, gain, 0), _run(bl, row, gain, 1)
    assert all(np.array_equal(g, w) for g, w in zip(got, want))
