"""The two roundings that every quantised activation goes through, over whole ranges of inputs: fp32 -> bf16 (one
hardware instruction) for every finite fp32 pattern, and bf16 -> int8 (by adding 1.5 * 2^23) for every finite bf16
value against many row maxima."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def test_narrowing_of_every_fp32(bl):
    """A product of zeros with the pattern as its residual: the epilogue narrows t = pattern + 0."""
    M, N, K = 4096, 4096, 128
    packed, beta = bl.bl_pack_ternary(torch.zeros((N, K), dtype=torch.int8, device=DEV), 1, beta=0.5)
    q = torch.zeros((M, K), dtype=torch.int8, device=DEV)
    scale, rowsum = torch.ones(M, device=DEV), torch.zeros(M, dtype=torch.int32, device=DEV)
    xb, absmax = torch.empty((M, N), dtype=torch.bfloat16, device=DEV), torch.zeros(M, device=DEV)
    low = torch.arange(M * N, dtype=torch.int32, device=DEV).view(M, N)
    for high in range(256):
        bits = low + ((high << 24) - (1 << 32 if high >= 128 else 0))
        bl.bl_gemm_w158a8_fused(packed, beta, 1, q, scale, rowsum, N, bl.BL_EPI_RESIDUAL, xb, absmax, residual=bits.view(torch.float32))
        u = bits & 0xFFFFFFFF if high < 128 else bits
        u = torch.where(u == -(1 << 31), torch.zeros_like(u), u)                     # -0 + 0 = +0
        # round to nearest even on the bits; the sum stays inside int32 for every finite pattern
        want = (u + (0x7FFF + ((u >> 16) & 1))) >> 16
        finite = (bits & 0x7F800000) != 0x7F800000
        got = xb.view(torch.int16).to(torch.int32)
        assert not ((((got ^ want) & 0xFFFF) != 0) & finite).any(), "high byte %02x" % high


def test_rounding_of_every_bf16(bl):
    u = np.concatenate([np.arange(0x7F80, dtype=np.uint16), np.arange(0x8000, 0xFF80, dtype=np.uint16)])   # 65280 = 255 * 256
    rows = np.zeros((16, 4096), np.uint16)
    rows.reshape(-1)[:u.size] = u
    x = (rows.astype(np.uint32) << 16).view(np.float32)
    X = torch.from_numpy(rows.view(np.int16)).to(DEV).view(torch.bfloat16)
    rng = np.random.default_rng(3)
    maxima = np.concatenate([[0.0, 1e-5, 127.0, 63.5, 254.0, 1.0, 3.0e38], np.exp(rng.uniform(np.log(1e-6), np.log(1e6), 249))]).astype(np.float32)
    for g in maxima:
        q, s, _ = bl.bl_quant_from_absmax(X, torch.full((16,), float(g), device=DEV))
        gg = np.maximum(g, np.float32(1e-5))
        with np.errstate(over="ignore"):
            want = np.clip(np.rint(x * (np.float32(127.0) / gg)), -127, 127).astype(np.int8)
        assert np.array_equal(q.cpu().numpy(), want), float(g)
        assert (s.cpu().numpy() == gg / np.float32(127.0)).all()
