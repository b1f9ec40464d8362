"""Packing a large matrix in one read: the codes that a sample of the weights settles, and the words taken up again once
beta is known.  Weights that are all undecided, a sample that misses beta, NaN and infinities, the smallest matrix of the
form with a remainder in every loop, and one above the size from which W is read past the caches.  Bytes and beta bit for bit
against the CPU oracle."""
import numpy as np
import pytest

import oracle
from helpers import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _weights(kind, N, K):
    rng = np.random.default_rng(N + K)
    W = rng.standard_normal((N, K), dtype=np.float32) * np.float32(0.02)
    if kind == "undecided":                     # |W| of half the weights within 0.1 % of beta / 2: every word is taken up again
        W = (np.sign(W) * np.where(rng.random((N, K)) < 0.5, 0.01, 0.03) * (1 + 0.001 * rng.standard_normal((N, K)))).astype(np.float32)
    elif kind == "sparse":                      # undecided words in some waves only, some of them more than half
        W[: N // 7] = np.float32(0.5) * np.abs(W).mean()
    elif kind == "missed":                      # beta comes from one weight that the sample does not see
        W *= np.float32(1e-9)
        W[N // 3, 77] = np.float32(1e9)
    elif kind == "zero":
        W[:] = 0
    elif kind == "nan":
        W[N // 2, K // 3] = np.nan
    elif kind == "inf":
        W[N - 1, K - 1] = -np.inf
        W[0, 0] = np.inf
    return W


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("kind,N,K", [("normal", 3076, 4096), ("undecided", 3076, 4096), ("sparse", 3076, 4096), ("missed", 3076, 4096),
                                      ("zero", 3076, 4096), ("nan", 3076, 4096), ("inf", 3076, 4096), ("normal", 196612, 64),
                                      ("normal", 13108, 2560), ("sparse", 13108, 2560)])
def test_large_matrix(bl, layout, kind, N, K):
    W = _weights(kind, N, K)
    beta, mean64 = oracle.absmean_beta(W, return_mean64=True)
    if kind == "inf":                           # (the oracle's compensated sum turns it into NaN)
        beta = np.float32(np.inf)
    assert not np.isfinite(mean64) or mean64 == 0 or oracle.beta_guard_ok(mean64)
    Wt = oracle.ternarize(W, beta) if np.isfinite(beta) else np.where(np.isnan(beta) | np.isinf(W), -1, 0).astype(np.int8)
    want = oracle.pack_padded(Wt, layout)       # (where the quotient is NaN the code is that of -1)
    packed, b = bl.bl_pack_ternary(to_dev(W), layout)
    assert np.array_equal(b.cpu().numpy(), np.array([beta], np.float32), equal_nan=True)
    assert np.array_equal(packed.cpu().numpy(), want)
