"""GPU kernels at the edges of their tiles and dispatch rules, against the oracle."""
import numpy as np
import pytest

import oracle
from tests._gpu import darb, dev, host, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# --------------------------------------------------------------------------------
# encode: waves take (row, chunk) pairs (a chunk is 1024 fp32 or 2048 fp16 columns),
# rows start at any element address
# --------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("N", [1, 5, 1023, 1024, 1025, 2047, 2049, 8193])
@pytest.mark.parametrize("skip", [0, 1, 3])
def test_encode_chunk_edges_any_alignment(darb, dtype, N, skip):  # noqa: F811
    say(f"encode N={N} {np.dtype(dtype).name}, first element {skip} past an aligned one")
    rng = np.random.default_rng(N * 8 + skip)
    M, ldw = 7, N + skip
    flat = (rng.integers(-50, 51, size=M * ldw + skip) * 0.25).astype(dtype)   # ties
    W = flat[skip:].reshape(M, ldw)[:, :N]
    d = 1.0 / rng.choice([1, 2, 4, 8, 32, 128], size=M)
    plan = darb.Plan(M, N, d, 0.05, 0, 1, 128).upload()
    lay = oracle.plan(N, d, 0.05, 0, 1, 128)
    vr, orf = oracle.encode(np.ascontiguousarray(W), lay)
    Wd = dev(flat)[skip:].view(M, ldw)[:, :N]
    v, o = plan.encode(Wd)
    ut = np.uint32 if dtype == np.float32 else np.uint16
    assert np.array_equal(host(o), orf)
    assert np.array_equal(host(v).view(ut), vr.view(ut))


# --------------------------------------------------------------------------------
# the LSTM layer's time steps as one launch: batch groups of 1, 2, 4 and 8 columns (the
# last one partly filled), one to many units per workgroup, odd H, final states after any
# T; matrices with more weights than the workgroups' registers hold take the steps
# --------------------------------------------------------------------------------

def _lstm_mats(darb, H, I, dtype, b_min, b_max, keep, seed):
    rng = np.random.default_rng(seed)
    dense, dev_mats = [], []
    for n in (I, H):
        W = (0.1 * rng.standard_normal((4 * H, n))).astype(dtype)
        d = np.clip(keep * rng.lognormal(0.0, 0.5, size=4 * H), 0.0, 1.0)
        plan = darb.Plan(4 * H, n, d, keep, 0, b_min, b_max).upload()
        lay = oracle.plan(n, d, keep, 0, b_min, b_max)
        v, o = plan.encode(dev(W))
        vr, orf = oracle.encode(W, lay)
        assert np.array_equal(host(o), orf)
        dense.append(oracle.decode(vr, orf, lay).astype(np.float64))
        dev_mats.append((plan, v, o))
    return dense, dev_mats, rng


def _lstm_reference(wih, whh, x, h, c, T, B):
    """Sequence, final states, and the largest sum of magnitudes that a gate adds up."""
    u = wih @ x.astype(np.float64)
    ua = np.abs(wih) @ np.abs(x).astype(np.float64)
    most = 0.0
    H = h.shape[0]
    seq = np.empty((H, T * B))
    sig = lambda z: 1.0 / (1.0 + np.exp(-z))  # noqa: E731
    for t in range(T):
        z = whh @ h + u[:, t * B:(t + 1) * B]
        most = max(most, float((np.abs(whh) @ np.abs(h) + ua[:, t * B:(t + 1) * B]).max()))
        c = sig(z[H:2 * H]) * c + sig(z[:H]) * np.tanh(z[2 * H:3 * H])
        h = sig(z[3 * H:]) * np.tanh(c)
        seq[:, t * B:(t + 1) * B] = h
    return seq, h, c, most


# An fp32 sum whose magnitudes add up to S is off by a few S * 2^-24 (in a chain of a
# thousand terms some 2^-24 S * sqrt(1000) / 4 at the very most, since partial sums grow as
# they go), the activations and the cell by a few 2^-24 of values below 1 to T.  The gates'
# slopes are at most 1, so a step adds its own error to what it inherits: T times the one of
# a step bounds the last.
def _lstm_tol(T, most):
    return 4.0 * T * (most + 1.0) * 2.0 ** -24


@pytest.mark.parametrize("case", [
    # H, I, T, B, dtype, b_min, b_max, keep
    (16, 24, 16, 2, "f32", 4, 32, 0.1), (33, 16, 17, 2, "f16", 4, 32, 0.1),
    (128, 64, 18, 1, "f16", 4, 64, 0.06), (96, 40, 16, 9, "f32", 4, 64, 0.1),
    (200, 64, 19, 16, "f16", 8, 128, 0.06), (130, 32, 16, 17, "f32", 4, 64, 0.1),
    (512, 64, 17, 20, "f32", 1, 4, 0.9), (512, 32, 16, 32, "f16", 1, 2, 0.9),
    (1024, 64, 16, 64, "f16", 4, 64, 0.05), (256, 64, 20, 40, "f32", 4, 64, 0.1),
    (1500, 64, 16, 20, "f16", 4, 64, 0.06), (64, 32, 15, 8, "f32", 4, 32, 0.1)])
def test_lstm_sequence_launch(darb, case):  # noqa: F811
    H, I, T, B, dt, b_min, b_max, keep = case
    say(f"lstm sequence {case}")
    dtype = np.float32 if dt == "f32" else np.float16
    (wih, whh), (dih, dhh), rng = _lstm_mats(darb, H, I, dtype, b_min, b_max, keep, H + B)
    x = rng.standard_normal((I, T * B)).astype(np.float32)
    h0 = (0.5 * rng.standard_normal((H, B))).astype(np.float32)
    c0 = rng.standard_normal((H, B)).astype(np.float32)
    seq, h, c = darb.lstm_layer(dih, dhh, dev(x), H, T, B, h=dev(h0), c=dev(c0))
    rs, rh, rc, most = _lstm_reference(wih, whh, x, h0.astype(np.float64), c0.astype(np.float64), T, B)
    for got, want, name in ((seq, rs, "h_seq"), (h, rh, "h"), (c, rc, "c")):
        err = float(np.abs(host(got) - want).max())
        say(f"  {name}: max abs err {err:.2e}, allowed {_lstm_tol(T, most):.2e}")
        assert err <= _lstm_tol(T, most), name
    assert np.array_equal(host(h), host(seq)[:, (T - 1) * B:])
    # the same bits again, with the buffers as the first call left them
    again = darb.lstm_layer(dih, dhh, dev(x), H, T, B, h=dev(h0), c=dev(c0))
    for a, b in zip((seq, h, c), again):
        assert torch.equal(a, b)


@pytest.mark.parametrize("case", [(96, 16, 9, "f32", 4, 64, 0.1), (520, 17, 20, "f16", 4, 64, 0.1),
                                  (512, 18, 18, "f32", 2, 8, 0.3), (256, 40, 64, "f16", 4, 64, 0.1),
                                  (130, 50, 3, "f32", 4, 64, 0.1)])
def test_lstm_sequence_forms(darb, case):  # noqa: F811
    # the exchange of workgroups on one XCD and on different ones; and a workgroup allowed no
    # wait, which gives up at once, so that the last launch computes the sequence by itself:
    # the same bits
    import ctypes
    H, T, B, dt, b_min, b_max, keep = case
    say(f"lstm sequence forms {case}")
    dtype = np.float32 if dt == "f32" else np.float16
    _, (_, (plan, v, o)), rng = _lstm_mats(darb, H, H, dtype, b_min, b_max, keep, 5)
    U = dev(rng.standard_normal((4 * H, T * B)).astype(np.float32))
    outs = []
    for polls, far in ((1 << 16, 0), (1 << 16, 1), (0, 0)):
        h = dev((0.5 * np.random.default_rng(1).standard_normal((H, B))).astype(np.float32))
        c = dev(np.random.default_rng(2).standard_normal((H, B)).astype(np.float32))
        seq = torch.zeros(H, T * B, device="cuda")
        scratch = torch.zeros(4 * H * B, device="cuda")
        P = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
        I64 = ctypes.c_int64
        rc = darb.lib().darb_test_lstm_seq(
            plan.handle, ctypes.c_int(0 if dt == "f32" else 1), P(v), P(o), I64(H), I64(T), I64(B),
            P(U), P(scratch), P(seq), P(h), P(c), ctypes.c_uint32(polls), ctypes.c_int(far),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        torch.cuda.synchronize()
        failed = int(scratch.view(torch.int32)[_seq_flag(H, B)])
        assert failed == (1 if polls == 0 else 0)
        outs.append((seq, h, c))
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert torch.equal(a, b)


def _seq_flag(H, B):
    """The failure flag's place in the scratch: after three slots of h."""
    cpg = 1 if B <= 8 else 2 if B <= 16 else 4 if B <= 32 else 8
    return 3 * H * (-(-B // cpg) * cpg)


def test_lstm_sequences_on_several_streams(darb):  # noqa: F811
    say("lstm sequences on three streams")
    H, T, B = 256, 40, 16
    _, (dih, dhh), rng = _lstm_mats(darb, H, 64, np.float16, 4, 64, 0.06, 3)
    xs = [dev(rng.standard_normal((64, T * B)).astype(np.float32)) for _ in range(3)]
    want = [darb.lstm_layer(dih, dhh, x, H, T, B) for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    got = []
    for _ in range(4):
        got = []
        for s, x in zip(streams, xs):
            with torch.cuda.stream(s):
                got.append(darb.lstm_layer(dih, dhh, x, H, T, B))
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        for a, b in zip(g, w):
            assert torch.equal(a, b)


def test_lstm_layer_under_capture(darb):  # noqa: F811
    say("lstm layer captured into a graph, replayed")
    H, T, B = 128, 16, 8
    # captured, each step is a launch, with sums of another order than the eager call's
    (wih, whh), (dih, dhh), rng = _lstm_mats(darb, H, 64, np.float16, 4, 64, 0.06, 4)
    xh = rng.standard_normal((64, T * B)).astype(np.float32)
    x = dev(xh)
    zero = np.zeros((H, B))
    tol = _lstm_tol(T, _lstm_reference(wih, whh, xh, zero, zero, T, B)[3])
    want = [host(t) for t in darb.lstm_layer(dih, dhh, x, H, T, B)]
    h, c = torch.zeros(H, B, device="cuda"), torch.zeros(H, B, device="cuda")
    seq = torch.empty(H, T * B, device="cuda")
    ws = torch.empty(darb.lstm_workspace_floats(H, T, B), device="cuda")
    run = lambda: darb.lstm_layer(dih, dhh, x, H, T, B, h=h, c=c, h_seq=seq,  # noqa: E731
                                  workspace=ws)
    run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for _ in range(3):
        h.zero_()
        c.zero_()
        seq.zero_()
        g.replay()
        torch.cuda.synchronize()
        for t, w in zip((seq, h, c), want):
            assert np.abs(host(t) - w).max() <= 2 * tol
