"""Packing where it can go wrong: latent weights on both sides of the ternariser's threshold (the fp32
quotient rounds to 0.5 or just above it), rows that end inside a chunk of 256, a quad of four or a
word, the transposed tiles of the k-major form, matrices below one float4.  Bytes and beta bit for bit
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


def _want(Wt, layout):
    return oracle.pack_kmajor(Wt) if layout == 3 else oracle.pack_trit5(Wt) if layout == 2 else oracle.pack_padded(Wt, layout)


def _check(bl, W, layout):
    beta = oracle.absmean_beta(W)
    Wt = oracle.ternarize(W, beta)
    packed, b = bl.bl_pack_ternary(to_dev(W), layout)
    assert np.array_equal(b.cpu().numpy().view(np.uint32), np.array([beta], np.float32).view(np.uint32))
    assert np.array_equal(packed.cpu().numpy(), _want(Wt, layout))
    packed8, _ = bl.bl_pack_ternary(to_dev(Wt), layout, beta=float(beta))
    assert np.array_equal(packed8.cpu().numpy(), _want(Wt, layout))


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("scale", [0.02, 1.0, 3e-6, 1e4])
def test_weights_at_the_threshold(bl, layout, scale):
    rng = np.random.default_rng(11)
    W = (rng.standard_normal((64, 1024)) * scale).astype(np.float32)
    at = [(int(r), int(c)) for r, c in zip(rng.integers(0, 64, 48), rng.integers(0, 1024, 48))]
    for _ in range(6):                                    # the planted values move beta a little: settle
        d = np.float32(oracle.absmean_beta(W)) + np.float32(1e-5)
        for i, (r, c) in enumerate(at):
            v = np.float32(d * np.float32(0.5 if i % 3 else 1.5))
            for _ in range(abs(i % 7 - 3)):
                v = np.nextafter(v, np.float32(np.inf) if i % 7 > 3 else np.float32(0), dtype=np.float32)
            W[r, c] = v if i & 1 else -v
    _check(bl, W, layout)


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("N,K", [(1, 1), (1, 3), (1, 5), (2, 255), (5, 257), (4, 64), (1028, 192), (257, 1023), (513, 20), (70, 4100)])
def test_ragged_edges(bl, layout, N, K):
    _check(bl, synth.latent_weights(40 + N + K, N, K), layout)
