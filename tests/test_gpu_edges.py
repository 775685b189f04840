"""GPU kernels at the edges of their tiles and dispatch rules, against the oracle."""
import sys

import numpy as np
import pytest

import oracle
from tests._parity import compare

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True, file=sys.stderr)


@pytest.fixture(scope="module")
def darb():
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_1911_08020_amd as d
    return d


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# --------------------------------------------------------------------------------
# encode: waves take (row, chunk) pairs (a chunk is 1024 fp32 or 2048 fp16 columns),
# rows start at any element address
# --------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("N", [1, 5, 1023, 1024, 1025, 2047, 2049, 8193])
@pytest.mark.parametrize("skip", [0, 1, 3])
def test_encode_chunk_edges_any_alignment(darb, dtype, N, skip):
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
