"""Packed offsets read eight and sixteen at a time: every block size, every place of an octet
in its run of 32 (rows of an odd number of octets start at each), the same bits as the byte
form from the SpMV (one block and looping) and from the SpMM at one and two lanes per row."""
import numpy as np
import pytest

from tests._gpu import darb, dev, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", range(8))
@pytest.mark.parametrize("nblk", [8, 16, 24, 200])
@pytest.mark.parametrize("M", [37, 4500])
def test_octets_equal_bytes(darb, l, nblk, M):  # noqa: F811
    say(f"packed octets log2 b = {l}, {nblk} weights a row, {M} rows")
    rng = np.random.default_rng(l * 100 + nblk)
    N = nblk << l
    if N > 16384 or M * N > 1 << 26:
        M, nblk = 37, min(nblk, 24)
        N = nblk << l
    if l > 1:
        N -= 1 + 7 * (l > 3)                             # a partial last block
    plan = darb.Plan(M, N, np.full(M, 1.0 / (1 << l)), 1.0 / (1 << l), 0, 1 << l, 1 << l).upload()
    assert [(b["log2b"], b["nblk"]) for b in plan.bins] == [(l, nblk)]
    last = N - ((nblk - 1) << l)                         # columns of a row's last block
    o = rng.integers(0, 1 << l, size=(M, nblk))
    o[:, -1] %= last
    o = dev(o.reshape(-1).astype(np.uint8))
    pk = plan.pack_offsets(o)
    assert torch.equal(plan.unpack_offsets(pk), o)
    v32 = rng.standard_normal(plan.nnz).astype(np.float32)
    x = rng.standard_normal(N).astype(np.float32)
    for wdt, xdt in ((np.float32, np.float32), (np.float16, np.float32), (np.float16, np.float16)):
        v, xd = dev(v32.astype(wdt)), dev(x.astype(xdt))
        assert torch.equal(plan.spmv_packed(v, pk, xd), plan.spmv(v, o, xd))
        for B in (1, 2):
            X = dev(np.repeat(x[:, None], B, axis=1).astype(xdt))
            assert torch.equal(plan.spmm_packed(v, pk, X), plan.spmm(v, o, X))
    q, s = plan.quantize_i8(dev(v32))
    for xdt in (np.float32, np.float16):
        xd = dev(x.astype(xdt))
        assert torch.equal(plan.spmv_i8(q, s, xd, packed=pk), plan.spmv_i8(q, s, xd, offsets=o))
        X = dev(np.repeat(x[:, None], 2, axis=1).astype(xdt))
        assert torch.equal(plan.spmm_i8(q, s, X, packed=pk), plan.spmm_i8(q, s, X, offsets=o))
