"""One-token streams at the edges of how a row is read: parts of three, four and five loads with idle slots at the
end, rows that start in the middle of a 128-byte line, row groups of eight that end inside, rows of more than
512 words, and the extreme int8 values.  Every sum is an exact integer: compared bit for bit with the oracle."""
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


def _item(c, layout, bf16, q=None, acc=None):
    it = dict(packed=to_dev(c.packed(layout)), beta=to_dev(np.array([c.beta], dtype=np.float32)), N=c.N, K=c.K,
              acc=torch.full((1, c.N), -99, dtype=torch.int32, device=DEV))
    if bf16:
        it["X"] = to_dev(c.X)
    else:
        q = oracle.pad_q(c.q if q is None else q)
        it.update(q=to_dev(q), rowsum=to_dev(q.astype(np.int32).sum(axis=1, dtype=np.int32)))
    return it


# loads of a row group per K (2-bit / five per byte): 1/1, 1/1 (a shifted odd row), 3/3, 5/4 (shifted), 5/4, 6/5 (shifted), 14/11, 17/14
@pytest.mark.parametrize("K", [64, 256, 1536, 2304, 2560, 2816, 6912, 8448])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("bf16", [True, False])
def test_one_width(bl, K, layout, bf16):
    """A table of one width, so that its own part length is taken; one to four row groups and a few rows."""
    cases = [Case(9100 + K + n, 1, n, K) for n in (1, 7, 8, 9, 29)]
    items = [_item(c, layout, bf16) for c in cases]
    bl.Stack(items, layout, 1, DEV).run()
    torch.cuda.synchronize()
    for it, c in zip(items, cases):
        assert np.array_equal(it["acc"].cpu().numpy(), c.acc), c.N


@pytest.mark.parametrize("K", [2624, 2688, 2752, 3200, 4032, 6976, 20416])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("bf16", [True, False])
def test_rows_across_lines(bl, K, layout, bf16):
    """Rows longer than 2560 that are no multiple of 64 bytes: row groups of two classes of rows out of sixteen or thirty-two, with
    blocks that end inside a class, a residual, and products of the plain form in the same table."""
    cases = [Case(9500 + K + n, 1, n, K) for n in (1, 2, 3, 8, 15, 17, 31, 33, 65, 130)] + [Case(9600 + K, 1, 21, 2560), Case(9601 + K, 1, 9, 6912)]
    rng = np.random.default_rng(K)
    items, residuals = [_item(c, layout, bf16) for c in cases], [rng.standard_normal(c.N).astype(np.float32) for c in cases]
    for it, c, r in zip(items, cases, residuals):
        it.update(y=torch.empty((1, c.N), dtype=torch.float32, device=DEV), residual=to_dev(r))
        if not bf16:
            it["scale"] = to_dev(np.array([c.scale[0]], dtype=np.float32))
    bl.Stack(items, layout, 1, DEV).run()
    torch.cuda.synchronize()
    for it, c, r in zip(items, cases, residuals):
        assert np.array_equal(it["acc"].cpu().numpy(), c.acc), c.N
        assert np.array_equal(it["y"].cpu().numpy()[0], r + c.y[0]), c.N


@pytest.mark.parametrize("layout", [0, 1, 2])
def test_mixed_widths(bl, layout):
    """Widths that favour different part lengths in one table: each is read in parts that are not its best."""
    cases = [Case(9300 + i, 1, 13 + i, K) for i, K in enumerate((320, 2304, 768, 6912, 64, 1600))]
    items = [_item(c, layout, i % 2 == 0) for i, c in enumerate(cases)]
    bl.Stack(items, layout, 1, DEV).run()
    torch.cuda.synchronize()
    for it, c in zip(items, cases):
        assert np.array_equal(it["acc"].cpu().numpy(), c.acc), c.K


@pytest.mark.parametrize("value", [-128, -127, -16, -1, 15, 16, 127])
@pytest.mark.parametrize("layout", [1, 2])
def test_extreme_sums(bl, value, layout):
    """The largest sums of the longest row: every weight of a row the same, every activation the same value."""
    c = Case(9400, 1, 9, 20480, full=False)
    c.Wt = np.tile(np.array([1, -1, 0], dtype=np.int8), 3)[:, None] * np.ones((9, 20480), dtype=np.int8)
    q = np.full((1, 20480), value, dtype=np.int8)
    it = _item(c, layout, False, q=q)
    bl.Stack([it], layout, 1, DEV).run()
    torch.cuda.synchronize()
    assert np.array_equal(it["acc"].cpu().numpy(), q.astype(np.int32) @ c.Wt.T.astype(np.int32))
