"""The SpMM at ragged sizes, against the oracle: batches that no vector divides, X from any
element, rows that end inside a vector of weights, formats shorter than one."""
import numpy as np
import pytest

import oracle
from tests._gpu import darb, dev, host, say, torch  # noqa: F401
from tests._parity import compare

pytestmark = pytest.mark.gpu


# lanes per row 1 .. 64, column remainders, rows of the last group that end inside a vector
# of weights, formats of fewer than 16 weights; byte and packed offsets give the same bits
@pytest.mark.parametrize("types", ["f32", "f16", "f16f32", "i8"])
@pytest.mark.parametrize("M,N,B", [
    (1, 3, 2), (3, 5, 7), (5, 9, 1), (40, 301, 1), (40, 301, 2), (67, 1500, 3), (67, 301, 5),
    (33, 1027, 20), (2100, 130, 21), (2100, 130, 33), (50, 260, 34), (20, 333, 70),
    (2100, 96, 67), (9, 130, 257)])
def test_spmm_ragged(darb, types, M, N, B):  # noqa: F811
    say(f"spmm {types} {M}x{N} B={B}")
    rng = np.random.default_rng(M * 7 + N + B)
    wdt = np.float16 if types.startswith("f16") else np.float32
    xdt = np.float16 if types == "f16" else np.float32
    d = 1.0 / rng.choice([4, 8, 16], size=M)
    plan = darb.Plan(M, N, d, 0.1, 0, 4, 16).upload()
    lay = oracle.plan(N, d, 0.1, 0, 4, 16)
    W = rng.standard_normal((M, N)).astype(wdt)
    v, o = plan.encode(dev(W))
    vr, orf = oracle.encode(W, lay)
    pk = plan.pack_offsets(o)
    X = rng.standard_normal((N, B)).astype(xdt)
    Xp = torch.zeros(N * (B + 1) + 1, dtype=torch.from_numpy(X).dtype, device="cuda")
    Xv = Xp[1:].view(N, B + 1)[:, :B]                    # odd leading dimension and start
    Xv.copy_(dev(X))
    if types == "i8":
        q, s = plan.quantize_i8(v)
        qr, sr = oracle.quantize_i8(vr, lay)
        ref, scale = oracle.spmm_i8(qr, sr, orf, lay, X), oracle.spmm_i8_absdot(qr, sr, orf, lay, X)
        outs = [plan.spmm_i8(q, s, x, **kw) for x in (dev(X), Xv)
                for kw in (dict(offsets=o), dict(packed=pk))]
    else:
        ref, scale = oracle.spmm(vr, orf, lay, X), oracle.spmm_absdot(vr, orf, lay, X)
        outs = [f(v, p, x) for x in (dev(X), Xv)
                for f, p in ((plan.spmm, o), (plan.spmm_packed, pk))]
    # fp32 sums of at most N / 4 products of exact inputs: relative to the sum of
    # magnitudes, below 376 roundings of 2^-24 = 2.3e-5 at worst and about 20 in practice
    compare(host(outs[0]), ref, scale, 1e-5, f"spmm {types} {M}x{N} B={B}")
    for other in outs[1:]:
        assert torch.equal(outs[0], other)
