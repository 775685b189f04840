"""The device plan in one launch (few rows) and in three, against the host-built plan."""
import sys

import numpy as np
import pytest


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


@pytest.mark.parametrize("M", [16384, 16385, 1, 1024, 4097])
def test_device_plan_one_launch_edges(darb, M):
    # up to 16384 rows in one workgroup (4 or 16 rows per thread), three launches beyond
    say(f"device plan M={M}")
    N = 300
    rng = np.random.default_rng(M)
    counts = np.minimum(rng.integers(0, N + 1, size=M), rng.integers(0, N + 1, size=M))
    kept = int(counts.sum())
    for mode in (0, 1):
        dp = darb.Plan.from_device_counts(N, dev(counts), kept, mode, 1, 128)
        hp = darb.Plan.from_counts(N, counts, kept, mode, 1, 128)
        for a, b in zip(dp.export(), hp.export()):
            assert np.array_equal(a, b)
        assert (dp.nnz, dp.packed_words, dp.bins) == (hp.nnz, hp.packed_words, hp.bins)
