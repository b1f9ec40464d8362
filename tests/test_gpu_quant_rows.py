"""The row quantisers where their work split changes: four waves or one wave per row (from 1024 rows),
the register sizes (K up to 2048, 4096 and 8192, two passes beyond), ragged and aligned rows, row
maxima that are given (and may be smaller than the row's own: values are clamped).  Bit for bit
against the CPU oracle."""
import numpy as np
import pytest

import oracle
import synth
from helpers import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("M,K", [(1023, 64), (1024, 64), (1025, 7), (1024, 2048), (1024, 2049), (1027, 4096), (1024, 4104),
                                 (1024, 8191), (1024, 8192), (7, 4096), (7, 4097), (7, 8192), (3, 8256), (1030, 8200),
                                 (2047, 2049), (2048, 2049), (2049, 4096), (2050, 4040), (2048, 4097)])
def test_quant_rows_at_the_edges_of_the_split(bl, M, K):
    X = synth.activations_bf16(31 + K, M, K)
    q_o, s_o, r_o = oracle.quant_act(X)
    q, s, r = bl.bl_quant_act_int8(to_dev(X))
    assert np.array_equal(q.cpu().numpy(), oracle.pad_q(q_o))
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_o.view(np.uint32))
    assert np.array_equal(r.cpu().numpy(), r_o)


@pytest.mark.parametrize("M,K", [(5, 2560), (1026, 2560), (1024, 6912), (3, 8256), (2050, 2112)])
def test_quant_with_given_row_maxima(bl, M, K):
    X = synth.activations_bf16(77 + K, M, K)
    Xd = to_dev(X)
    x = (X.astype(np.uint32) << 16).view(np.float32)
    gamma = np.abs(x).max(axis=1)
    gamma[1::2] *= np.float32(0.25)                       # a maximum smaller than the row's own: clamped
    absmax = to_dev(gamma)
    q, s, r = bl.bl_quant_from_absmax(Xd, absmax)
    g = np.maximum(gamma, np.float32(1e-5))
    inv = np.float32(127.0) / g
    want = np.clip(np.rint(x * inv[:, None]), -127, 127).astype(np.int8)
    assert np.array_equal(q.cpu().numpy(), want)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), (g / np.float32(127.0)).view(np.uint32))
    assert np.array_equal(r.cpu().numpy(), want.astype(np.int32).sum(axis=1))
    assert not absmax.cpu().numpy().any()
