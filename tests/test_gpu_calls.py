"""The native call module against the methods' Python code: the same results bit for bit
(with buffers given or not, on a given stream, from strided operands), and what the Python
code refuses stays refused with the same error."""
import numpy as np
import pytest

from tests._gpu import darb, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


class Plain(torch.Tensor):
    """A tensor subclass: the native module leaves it to the Python code."""


def plain(t):
    return t.as_subclass(Plain)


@pytest.fixture(scope="module")
def fmt(darb):  # noqa: F811
    rng = np.random.default_rng(7)
    M, N, B = 70, 301, 6
    plan = darb.Plan(M, N, 1.0 / rng.choice([4, 8, 16], size=M), 0.1, 0, 4, 32).upload()
    W = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()
    v, o = plan.encode(W)
    q, s = plan.quantize_i8(v)
    x = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).cuda()
    X = torch.from_numpy(rng.standard_normal((N, B + 3)).astype(np.float32)).cuda()
    return dict(plan=plan, W=W, v=v, o=o, p=plan.pack_offsets(o), q=q, s=s, x=x, X=X[:, :B],
                M=M, N=N, B=B)


CALLS = {
    "spmv": lambda f, w, **k: f["plan"].spmv(w(f["v"]), f["o"], f["x"], **k),
    "spmv_packed": lambda f, w, **k: f["plan"].spmv_packed(w(f["v"]), f["p"], f["x"], **k),
    "spmv_i8": lambda f, w, **k: f["plan"].spmv_i8(w(f["q"]), f["s"], f["x"], offsets=f["o"], **k),
    "spmv_i8 packed": lambda f, w, **k: f["plan"].spmv_i8(w(f["q"]), f["s"], f["x"],
                                                          packed=f["p"], **k),
    "spmm": lambda f, w, **k: f["plan"].spmm(w(f["v"]), f["o"], f["X"], **k),
    "spmm_packed": lambda f, w, **k: f["plan"].spmm_packed(w(f["v"]), f["p"], f["X"], **k),
    "spmm_i8": lambda f, w, **k: f["plan"].spmm_i8(w(f["q"]), f["s"], f["X"], offsets=f["o"], **k),
    "spmm_i8 packed": lambda f, w, **k: f["plan"].spmm_i8(w(f["q"]), f["s"], f["X"],
                                                          packed=f["p"], **k),
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_native_call_equals_python_path(darb, fmt, name):  # noqa: F811
    say(f"native call: {name}")
    call = CALLS[name]
    want = call(fmt, plain)
    assert torch.equal(call(fmt, lambda t: t), want.as_subclass(torch.Tensor))
    key = "y" if name.startswith("spmv") else "Y"
    out = torch.full((fmt["M"],) if key == "y" else (fmt["M"], fmt["B"] + 2), 7.0, device="cuda")
    view = out if key == "y" else out[:, :fmt["B"]]         # a leading dimension of its own
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    got = call(fmt, lambda t: t, **{key: view}, stream=st)
    st.synchronize()
    assert got is view and torch.equal(view, want.as_subclass(torch.Tensor))
    if key == "Y":
        assert bool((out[:, fmt["B"]:] == 7.0).all())
    with torch.cuda.stream(st):                             # the current stream
        assert torch.equal(call(fmt, lambda t: t), want.as_subclass(torch.Tensor))


def test_native_encode_equals_python_path(darb, fmt):  # noqa: F811
    v, o = torch.empty_like(fmt["v"]), torch.empty_like(fmt["o"])
    got = fmt["plan"].encode(fmt["W"], values=v, offsets=o)
    assert got[0] is v and got[1] is o
    v2, o2 = fmt["plan"].encode(plain(fmt["W"]))
    assert torch.equal(v, v2.as_subclass(torch.Tensor))
    assert torch.equal(o, o2.as_subclass(torch.Tensor))


@pytest.mark.parametrize("bad", [
    (lambda f: f["plan"].spmv(f["v"], f["o"], f["x"][:-1]), ValueError),
    (lambda f: f["plan"].spmv(f["v"], f["o"], f["x"].cpu()), ValueError),
    (lambda f: f["plan"].spmv(f["v"][:-1], f["o"], f["x"]), ValueError),
    (lambda f: f["plan"].spmv(f["v"].double(), f["o"], f["x"]), TypeError),
    (lambda f: f["plan"].spmv(f["v"], f["o"].int(), f["x"]), TypeError),
    (lambda f: f["plan"].spmv(f["v"], f["o"], f["x"].half()), "DarbError"),
    (lambda f: f["plan"].spmv(f["v"], f["o"], f["x"], y=f["x"][:3]), ValueError),
    (lambda f: f["plan"].spmm(f["v"], f["o"], f["X"].t()), ValueError),
    (lambda f: f["plan"].spmm(f["v"], f["o"], f["X"], Y=f["X"].half()), TypeError),
    (lambda f: f["plan"].spmm(f["v"], f["o"], f["X"][:, :0]), "DarbError"),
    (lambda f: f["plan"].spmv_i8(f["q"], f["s"], f["x"]), ValueError),
    (lambda f: f["plan"].spmv_i8(f["q"], f["s"], f["x"], offsets=f["o"], packed=f["p"]), ValueError),
    (lambda f: f["plan"].encode(f["W"], values=f["v"].half(), offsets=f["o"]), TypeError),
    (lambda f: f["plan"].encode(f["W"].t()), ValueError)])
def test_refused_calls_stay_refused(darb, fmt, bad):  # noqa: F811
    call, err = bad
    with pytest.raises(darb.DarbError if err == "DarbError" else err):
        call(fmt)
