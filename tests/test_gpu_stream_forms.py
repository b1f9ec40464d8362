"""The two forms of the one-token stream on the same products: alone in a table (few row groups: the vector unit, where rows are long
enough) and beside a product of many short rows, which makes the table one of the matrix cores.  Edges of parts, lanes, row groups
and lines, bf16 and int8 rows, residuals, the extreme int8 values, NaN and infinities: bit for bit against the oracle, and the forms
against each other."""
import numpy as np
import pytest

import oracle
from helpers import Case, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


def _filler(layout):
    """40960 rows of 64: the packed zeros of one row, repeated."""
    c = Case(7, 1, 4, 64)
    packed = np.tile(c.packed(layout).reshape(-1), 10240)
    q = to_dev(oracle.pad_q(c.q))
    return dict(packed=to_dev(packed), beta=to_dev(np.array([c.beta], dtype=np.float32)), N=40960, K=64, q=q, rowsum=to_dev(c.rowsum),
                acc=torch.full((1, 40960), -99, dtype=torch.int32, device=DEV)), np.tile(c.acc, (1, 10240))


def _run(bl, items, layout, matrix):
    """Runs the items in a table of one form; returns their int32 and fp32 outputs."""
    for it in items:
        it["acc"].fill_(-99)
        if "y" in it:
            it["y"].fill_(-99.0)
    extra, want = _filler(layout) if matrix else (None, None)
    st = bl.Stack(items + ([extra] if matrix else []), layout, 1, DEV)
    st.run()
    torch.cuda.synchronize()
    if matrix:
        assert np.array_equal(extra["acc"].cpu().numpy(), want)
    return st.plan.red_ints, [(it["acc"].cpu().numpy(), it["y"].cpu().numpy() if "y" in it else None) for it in items]


def _item(c, layout, bf16, residual=None, q=None):
    it = dict(packed=to_dev(c.packed(layout)), beta=to_dev(np.array([c.beta], dtype=np.float32)), N=c.N, K=c.K,
              acc=torch.empty((1, c.N), dtype=torch.int32, device=DEV), y=torch.empty((1, c.N), dtype=torch.float32, device=DEV))
    if bf16:
        it["X"] = to_dev(c.X)
    else:
        q = oracle.pad_q(c.q if q is None else q)
        it.update(q=to_dev(q), rowsum=to_dev(q.astype(np.int32).sum(axis=1, dtype=np.int32)), scale=to_dev(c.scale))
    if residual is not None:
        it["residual"] = to_dev(residual)
    return it


@pytest.mark.parametrize("K", [64, 1280, 2560, 2624, 3200, 4032, 5120, 6912, 8448, 13760, 19200, 19264, 20480])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("bf16", [True, False])
def test_both_forms(bl, K, layout, bf16):
    cases = [Case(8700 + K + n, 1, n, K) for n in (1, 7, 8, 18, 33, 66)]
    rng = np.random.default_rng(K)
    residuals = [rng.standard_normal((1, c.N)).astype(np.float32) if c.N % 2 else None for c in cases]
    items = [_item(c, layout, bf16, r) for c, r in zip(cases, residuals)]
    for matrix in (False, True):
        form, out = _run(bl, items, layout, matrix)
        vector = not matrix and (K > 2560 or layout == 2)
        assert (form == 0) == vector or (layout == 2 and K > 19200), form
        for (acc, y), c, r in zip(out, cases, residuals):
            assert np.array_equal(acc, c.acc), (matrix, c.N)
            assert np.array_equal(y, c.y if r is None else r + c.y), (matrix, c.N)


@pytest.mark.parametrize("value", [-128, -1, 127])
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_extreme_sums(bl, value, layout):
    # The longest rows of which the layout has both forms.
    K = 19200 if layout == 2 else 20352
    c = Case(8800, 1, 9, K, full=False)
    c.Wt = np.tile(np.array([1, -1, 0], dtype=np.int8), 3)[:, None] * np.ones((9, K), dtype=np.int8)
    q = np.full((1, K), value, dtype=np.int8)
    it = _item(c, layout, False, q=q)
    for matrix in (False, True):
        assert np.array_equal(_run(bl, [it], layout, matrix)[1][0][0], q.astype(np.int32) @ c.Wt.T.astype(np.int32)), matrix


@pytest.mark.parametrize("value", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("layout", [1, 2])
def test_not_finite(bl, value, layout):
    cases = [Case(8900 + K, 1, 21, K, full=False) for K in (3200, 6912)]
    items = [_item(c, layout, True) for c in cases]
    for it, at in zip(items, (3199, 100)):
        it["X"][0, at] = value
        it["q_out"], it["scale_out"] = torch.empty((1, it["K"]), dtype=torch.int8, device=DEV), torch.empty(1, device=DEV)
    got = []
    for matrix in (False, True):
        form, out = _run(bl, items, layout, matrix)
        assert (form != 0) == matrix
        got.append([a.tobytes() for pair in out for a in pair] + [it[k].cpu().numpy().tobytes() for it in items for k in ("q_out", "scale_out")])
    assert got[0] == got[1]
