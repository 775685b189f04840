"""SpMM from an X that spans more than 4 GiB (64-bit addresses), just below and just past
the limit of the 32-bit form: the same bits as from the same X stored densely."""
import numpy as np
import pytest

from tests._gpu import darb, dev, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# few rows (a column per lane) and many (16 bytes per lane; from 16 waves per CU), batches
# that no vector divides and that fill several slabs of 16 lanes
@pytest.mark.parametrize("xdt", [torch.float32, torch.float16])
@pytest.mark.parametrize("M,B", [(40, 1), (40, 20), (40, 65), (9000, 2), (9000, 8), (9000, 11),
                                 (9000, 20),
                                 (9000, 33), (9000, 64), (9000, 67), (4100, 300)])
def test_spmm_past_4_gib(darb, xdt, M, B):  # noqa: F811
    say(f"spmm past 4 GiB: {M} rows, batch {B}, {xdt}")
    rng = np.random.default_rng(M + B)
    N = 37
    plan = darb.Plan(M, N, 1.0 / rng.choice([1, 2, 4, 8], size=M), 0.3, 0, 1, 8).upload()
    W = rng.standard_normal((M, N)).astype(np.float32)
    formats = []
    for wdt in (np.float32, np.float16) if xdt == torch.float32 else (np.float16,):
        v, o = plan.encode(dev(W.astype(wdt)))
        formats.append((v, o))
    pk = plan.pack_offsets(o)
    q, s = plan.quantize_i8(v)
    dense = dev(rng.standard_normal((N, B)).astype(np.float32)).to(xdt)
    size = dense.element_size()
    most = 0xFFFFFFFF // size                            # (N - 1) * ldx + B up to it: 32 bits
    below = (most - B) // (N - 1)
    flat = torch.empty((N - 1) * (below + 8) + B, dtype=xdt, device="cuda")
    assert flat.numel() * size > 1 << 32

    def products(X):
        out = [f(v, p, X) for v, _ in formats
               for f, p in ((plan.spmm, o), (plan.spmm_packed, pk))]
        return out + [plan.spmm_i8(q, s, X, offsets=o), plan.spmm_i8(q, s, X, packed=pk)]
    want = products(dense)
    for ldx in (below, below + 1, below + 7):            # +7: fp16 rows an odd number apart
        assert ((N - 1) * ldx + B > most) == (ldx > below)
        X = torch.as_strided(flat, (N, B), (ldx, 1))
        X.copy_(dense)
        for got, w in zip(products(X), want):
            assert torch.equal(got, w), ldx
    del flat
    torch.cuda.empty_cache()
