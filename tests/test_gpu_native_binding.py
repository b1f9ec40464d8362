"""The native form of the binding's small calls against its Python form: the same bits, the same errors, the same
stream, and whatever is out of the ordinary handed back."""
import numpy as np
import pytest

from helpers import Case, to_dev

torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module")
def bl():
    from paper_2504_12285_amd import binding
    binding.load()
    return binding


class _Back:
    """Hands every call back to the Python form."""

    def __getattr__(self, name):
        return lambda *a: NotImplemented


def _calls(bl, M, N, K):
    c = Case(77 + M + N + K, M, N, K)
    packed, beta, X = to_dev(c.packed(1)), to_dev(np.array([c.beta], dtype=np.float32)), to_dev(c.X)
    q, scale, rowsum = bl.bl_quant_act_int8(X)
    y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    out = [q, scale, rowsum, bl.bl_quant_act_int8(X, want_rowsum=False)[2]]
    out += bl.bl_gemv_w158a8(packed, beta, 1, q, scale, rowsum, N, K=K)
    out += bl.bl_gemv_w158a8(packed, beta, 1, q, scale, None, N, want_acc=False, K=K)          # needs a workspace
    out += bl.bl_gemm_w158a8(packed, beta, 1, q, scale, rowsum, N, want_acc=False, y=y, K=K)
    out += bl.bl_bitlinear_decode(packed, beta, 1, X, N, want_acc=True, want_q=True) if K % 64 == 0 else ()
    st = bl.Stack([dict(packed=packed, beta=beta, X=X[:1], N=N, K=K, y=y[:1])], 1, 1, DEV) if K % 64 == 0 else None
    if st is not None:
        st.run()
        out.append(y[:1].clone())
    return out, y


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 5, 64), (3, 130, 2560), (16, 37, 100)])
def test_same_results(bl, monkeypatch, M, N, K):
    got, y = _calls(bl, M, N, K)
    assert any(t is y for t in got), "a given output is returned itself"
    monkeypatch.setattr(bl, "_native", _Back())
    want, _ = _calls(bl, M, N, K)
    assert len(got) == len(want)
    for a, b in zip(got, want):
        assert (a is None) == (b is None)
        if a is not None:
            assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b)


@pytest.mark.gpu
def test_same_errors_and_unusual_arguments(bl, monkeypatch):
    c = Case(5, 2, 8, 64)
    packed, beta, X = to_dev(c.packed(1)), to_dev(np.array([c.beta], dtype=np.float32)), to_dev(c.X)
    q, scale, rowsum = bl.bl_quant_act_int8(X)
    class Sub(torch.Tensor):
        pass
    calls = [lambda: bl.bl_gemv_w158a8(packed, beta, 7, q, scale, rowsum, 8),                  # bad layout
             lambda: bl.bl_gemv_w158a8(packed, None, 1, q, scale, rowsum, 8),                  # no beta
             lambda: bl.bl_quant_act_int8(X[:, ::2]),                                          # not contiguous
             lambda: bl.bl_quant_act_int8(X.float()),
             lambda: bl.bl_quant_act_int8(X.cpu()),
             lambda: bl.bl_gemm_w158a8(packed, beta, 1, q, scale, rowsum, 8, K=128),           # not this q's K
             lambda: bl.bl_bitlinear_decode(packed, beta, 1, X, -3),
             lambda: bl.bl_gemv_w158a8(packed, beta, 1, q.as_subclass(Sub), scale, rowsum, 8)[1],
             lambda: bl.bl_gemv_w158a8(packed, beta, 1, q, scale, rowsum, 8, K=np.int64(64))[1]]

    def outcome(f):
        try:
            return f().cpu().numpy().tobytes()
        except Exception as e:                             # noqa: BLE001  (the kinds are compared)
            return type(e), getattr(e, "status", None)

    native = [outcome(f) for f in calls]
    monkeypatch.setattr(bl, "_native", _Back())
    assert native == [outcome(f) for f in calls]
    assert isinstance(native[-1], bytes) and isinstance(native[-2], bytes)


@pytest.mark.gpu
def test_current_stream(bl):
    native = bl._native or bl._first_native()
    assert native.current_stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert native.current_stream() == side.cuda_stream == bl._stream()
    graph = torch.cuda.CUDAGraph()
    c = Case(6, 1, 64, 64)
    packed, beta, X = to_dev(c.packed(1)), to_dev(np.array([c.beta], dtype=np.float32)), to_dev(c.X)
    bl.bl_bitlinear_decode(packed, beta, 1, X, 64)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        y = bl.bl_bitlinear_decode(packed, beta, 1, X, 64)[1]
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, bl.bl_bitlinear_decode(packed, beta, 1, X, 64)[1])


def test_host_tensors_are_refused(bl):
    with pytest.raises(AssertionError):
        bl.bl_quant_act_int8(torch.zeros((1, 64), dtype=torch.bfloat16))
