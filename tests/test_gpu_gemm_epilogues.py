"""The fused epilogues of the prefill product at the edges of their tiles (64 x 128, one product 128 x 256; every tile is in
test_gpu_gemm_pipe.py), whole and cut by the last row or column, with and without the int32 and the fp32 output, a residual that is also the
output.  Bit for bit against the oracle's separate steps."""
import numpy as np
import pytest

import oracle
import synth
from helpers import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _inputs(M, N, K):
    rng = np.random.default_rng(M + N + K)
    Wt, q = synth.uniform_i8(90, (N, K), -1, 1), synth.uniform_i8(91, (M, K), -127, 127)
    beta, scale = np.float32(0.0173), (rng.uniform(0.5, 2.0, size=M) / 127.0).astype(np.float32)
    rowsum = q.astype(np.int32).sum(axis=1).astype(np.int32)
    acc = oracle.matmul_i32(q, Wt)
    dev = (to_dev(oracle.pack(Wt, 1)), to_dev(np.array([beta], dtype=np.float32)), 1, to_dev(q), to_dev(scale), to_dev(rowsum))
    return rng, acc, oracle.rescale(acc, beta, scale), dev


def _check(xb, absmax, want):
    xb_o = oracle.f32_to_bf16(want)
    assert np.array_equal(xb.view(torch.int16).cpu().numpy().view(np.uint16), xb_o)
    assert np.array_equal(absmax.cpu().numpy(), np.abs(synth.bf16_bits_to_f32(xb_o)).max(axis=1))


@pytest.mark.parametrize("with_acc,with_y", [(False, True), (True, True), (False, False)])
@pytest.mark.parametrize("M,N", [(1, 4), (63, 128), (64, 128), (65, 132), (128, 256), (130, 252), (2432, 2432), (2433, 2436), (2431, 2428)])
def test_residual(bl, M, N, with_acc, with_y):
    rng, acc_o, prod, dev = _inputs(M, N, 128)
    res = (rng.standard_normal((M, N)) * 5).astype(np.float32)
    want = oracle.chain_residual(res, prod)
    acc = torch.full((M, N), -7, dtype=torch.int32, device=DEV) if with_acc else None
    y = to_dev(res) if with_y else None
    residual = y if with_y and not with_acc else to_dev(res)
    xb, absmax = torch.empty((M, N), dtype=torch.bfloat16, device=DEV), torch.zeros(M, device=DEV)
    bl.bl_gemm_w158a8_fused(*dev, N, bl.BL_EPI_RESIDUAL, xb, absmax, residual=residual, y=y, acc=acc)
    torch.cuda.synchronize()
    _check(xb, absmax, want)
    if with_y:
        assert np.array_equal(y.cpu().numpy().view(np.uint32), want.view(np.uint32))
    if with_acc:
        assert np.array_equal(acc.cpu().numpy(), acc_o)


@pytest.mark.parametrize("with_acc,with_y", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("M,F", [(1, 64), (64, 64), (65, 128), (2432, 1216), (2433, 1216), (2303, 1280)])
def test_gate(bl, M, F, with_acc, with_y):
    rng, acc_o, prod, dev = _inputs(M, 2 * F, 128)
    want = oracle.chain_relu2_gate(prod)
    want_f32 = (np.maximum(prod[:, :F], np.float32(0)) ** 2 * prod[:, F:]).astype(np.float32)
    acc = torch.full((M, 2 * F), -7, dtype=torch.int32, device=DEV) if with_acc else None
    y = torch.empty((M, F), device=DEV) if with_y else None
    xb, absmax = torch.empty((M, F), dtype=torch.bfloat16, device=DEV), torch.zeros(M, device=DEV)
    bl.bl_gemm_w158a8_fused(*dev, 2 * F, bl.BL_EPI_RELU2_GATE, xb, absmax, y=y, acc=acc)
    torch.cuda.synchronize()
    assert np.array_equal(xb.view(torch.int16).cpu().numpy().view(np.uint16), want)
    assert np.array_equal(absmax.cpu().numpy(), np.abs(synth.bf16_bits_to_f32(want)).max(axis=1))
    if with_y:
        assert np.array_equal(y.cpu().numpy(), want_f32)
    if with_acc:
        assert np.array_equal(acc.cpu().numpy(), acc_o)


@pytest.mark.parametrize("M,N", [(1, 128), (65, 384), (300, 2560), (2433, 2560)])
@pytest.mark.parametrize("kind", ["residual", "gate"])
def test_bf16_output_at_every_second_byte(bl, kind, M, N):
    """x_bf16 one value into an aligned buffer: the values are in place, and nothing beside them changes."""
    rng, _, prod, dev = _inputs(M, N, 128)
    res = (rng.standard_normal((M, N)) * 5).astype(np.float32) if kind == "residual" else None
    NO = N if kind == "residual" else N // 2
    want = oracle.f32_to_bf16(oracle.chain_residual(res, prod)) if kind == "residual" else oracle.chain_relu2_gate(prod)
    buf = torch.full((M * NO + 64,), 7.0, dtype=torch.bfloat16, device=DEV)
    xb, absmax = buf[33:33 + M * NO].view(M, NO), torch.zeros(M, device=DEV)
    assert xb.data_ptr() % 4 == 2
    bl.bl_gemm_w158a8_fused(*dev, N, bl.BL_EPI_RESIDUAL if kind == "residual" else bl.BL_EPI_RELU2_GATE, xb, absmax,
                            residual=None if res is None else to_dev(res))
    torch.cuda.synchronize()
    assert np.array_equal(xb.view(torch.int16).cpu().numpy().view(np.uint16), want)
    assert np.array_equal(absmax.cpu().numpy(), np.abs(synth.bf16_bits_to_f32(want)).max(axis=1))
    assert (buf[:33] == 7).all() and (buf[33 + M * NO:] == 7).all()
