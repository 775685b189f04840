"""The device plan in one launch (few rows) and in three, against the host-built plan."""
import threading

import numpy as np
import pytest

from tests._gpu import darb, dev, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [8192, 8193, 16384, 16385, 1, 1024, 4096, 4097])
def test_device_plan_one_launch_edges(darb, M):  # noqa: F811
    # up to 8192 rows in one workgroup (4 or 8 rows per thread), three launches beyond
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


def test_device_plans_of_many_threads(darb):  # noqa: F811
    # more threads than the 16 slots through which the summaries reach the host: those that
    # find none copy theirs
    say("device plans of 24 threads")
    N = 300
    rng = np.random.default_rng(24)
    counts = [rng.integers(0, N + 1, size=700 + i) for i in range(24)]
    on_dev = [dev(c) for c in counts]
    want = [darb.Plan.from_counts(N, c, int(c.sum()), 0, 1, 128) for c in counts]
    torch.cuda.synchronize()
    start = threading.Barrier(24, timeout=30)
    bad, errors = [], []

    def work(i):
        try:
            st = torch.cuda.Stream()
            start.wait()
            for _ in range(20):
                p = darb.Plan.from_device_counts(N, on_dev[i], int(counts[i].sum()), 0, 1, 128,
                                                 stream=st)
                if (p.nnz, p.packed_words, p.bins) != (want[i].nnz, want[i].packed_words,
                                                       want[i].bins):
                    bad.append(i)
            if not all(np.array_equal(a, b) for a, b in zip(p.export(), want[i].export())):
                bad.append(i)
        except Exception as e:                            # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(24)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors and not bad
