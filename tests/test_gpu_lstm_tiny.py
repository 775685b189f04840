"""The LSTM layer's step kernel on matrices of a few weights: rows shorter than a lane's
vector of weights, formats of fewer than 16 weights, against numpy in 64 bits."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H", [1, 2, 3, 5, 17])
@pytest.mark.parametrize("B", [1, 3, 4, 9])
def test_lstm_step_few_weights(H, B):
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_1911_08020_amd as darb
    print(f"lstm step H={H} B={B}", flush=True, file=sys.stderr)
    rng = np.random.default_rng(H * 16 + B)
    T, I = 3, 6
    dense, mats = [], []
    for n in (I, H):
        W = rng.standard_normal((4 * H, n)).astype(np.float32)
        d = np.full(4 * H, 1.0 / 4)
        plan = darb.Plan(4 * H, n, d, 0.25, 0, 4, 4).upload()
        lay = oracle.plan(n, d, 0.25, 0, 4, 4)
        vr, orf = oracle.encode(W, lay)
        dense.append(oracle.decode(vr, orf, lay).astype(np.float64))
        mats.append((plan,) + plan.encode(torch.from_numpy(W).cuda()))
    x = rng.standard_normal((I, T * B)).astype(np.float32)
    seq, h, c = darb.lstm_layer(mats[0], mats[1], torch.from_numpy(x).cuda(), H, T, B)
    hr, cr = np.zeros((H, B)), np.zeros((H, B))
    sig = lambda z: 1.0 / (1.0 + np.exp(-z))  # noqa: E731
    for t in range(T):
        z = dense[1] @ hr + dense[0] @ x[:, t * B:(t + 1) * B].astype(np.float64)
        i, f, g, o = z[:H], z[H:2 * H], z[2 * H:3 * H], z[3 * H:]
        cr = sig(f) * cr + sig(i) * np.tanh(g)
        hr = sig(o) * np.tanh(cr)
        # at most 7 products a gate, values of order 1: a few roundings of 2^-24 each,
        # times three steps
        assert np.abs(seq[:, t * B:(t + 1) * B].cpu().numpy() - hr).max() < 1e-5
    assert np.abs(c.cpu().numpy() - cr).max() < 1e-5


@pytest.mark.parametrize("B", [1, 2, 4, 8, 12])
def test_lstm_step_short_last_rows(B):
    # vectors of up to 16 weights, rows of 2 and 4: the format's last rows load vectors that
    # start before them and move them down
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_1911_08020_amd as darb
    print(f"lstm step, short last rows, B={B}", flush=True, file=sys.stderr)
    H, T, I = 128, 8, 32
    rng = np.random.default_rng(B)
    dense, mats = [], []
    for n in (I, H):
        W = (0.3 * rng.standard_normal((4 * H, n))).astype(np.float16)
        d = 1.0 / rng.choice([4, 16, 32, 64], size=4 * H)
        plan = darb.Plan(4 * H, n, d, 0.05, 0, 4, 64).upload()
        lay = oracle.plan(n, d, 0.05, 0, 4, 64)
        vr, orf = oracle.encode(W, lay)
        dense.append(oracle.decode(vr, orf, lay).astype(np.float64))
        mats.append((plan,) + plan.encode(torch.from_numpy(W).cuda()))
    x = rng.standard_normal((I, T * B)).astype(np.float32)
    seq, h, c = darb.lstm_layer(mats[0], mats[1], torch.from_numpy(x).cuda(), H, T, B)
    hr, cr = np.zeros((H, B)), np.zeros((H, B))
    sig = lambda z: 1.0 / (1.0 + np.exp(-z))  # noqa: E731
    for t in range(T):
        z = dense[1] @ hr + dense[0] @ x[:, t * B:(t + 1) * B].astype(np.float64)
        i, f, g, o = z[:H], z[H:2 * H], z[2 * H:3 * H], z[3 * H:]
        cr = sig(f) * cr + sig(i) * np.tanh(g)
        hr = sig(o) * np.tanh(cr)
        # a gate sums at most 8 + 32 products of about 0.3: some tens of roundings of 2^-24
        # of values below 10, damped by the gates (slopes of at most 1) from step to step
        assert np.abs(seq[:, t * B:(t + 1) * B].cpu().numpy() - hr).max() < 1e-5
    assert np.abs(h.cpu().numpy() - hr).max() < 1e-5
