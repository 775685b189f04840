"""The LSTM layer's time steps run as one launch only where every workgroup's weights fit its
registers: the plan knows the most 16-weight chunks that one of them would hold."""
import ctypes

import numpy as np
import pytest

from tests._gpu import darb, dev, host, say, torch  # noqa: F401


def _chunks(d, plan):
    f = d.lib().darb_test_lstm_chunks
    f.restype = ctypes.c_int64
    return f(plan.handle)


def _applies(d, plan, H, T, B):
    f = d.lib().darb_test_lstm_seq_applies
    return f(plan.handle, ctypes.c_int64(H), ctypes.c_int64(T), ctypes.c_int64(B),
             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))


def _brute(log2b, H):
    """ceil(H / 32) units of all four gates per workgroup, each row in whole chunks."""
    units = -(-H // 32)
    rows = -(-(-(-H // (1 << log2b.astype(np.int64)))) // 16)
    return max(int(sum(rows[g * H + u0:g * H + min(u0 + units, H)].sum() for g in range(4)))
               for u0 in range(0, H, units))


def _counts(H, keep, seed, order="any"):
    """Kept counts of the rows; "end": the last units are the densest in every gate."""
    rng = np.random.default_rng(seed)
    d = keep * rng.lognormal(0.0, 0.5, size=4 * H)
    if order == "end":
        d = np.sort(d.reshape(4, H), axis=1).reshape(-1)
    return np.minimum(np.rint(d * H), H).astype(np.int64)


SIZES = [(1, 0.3), (2, 0.3), (16, 0.3), (31, 0.2), (32, 0.2), (33, 0.2), (250, 0.1), (1024, 0.05),
         (1025, 0.05), (1500, 0.065), (2049, 0.05), (4095, 0.02), (4096, 0.02)]


@pytest.mark.parametrize("H,keep", SIZES)
def test_host_plan_counts_chunks(H, keep):
    import paper_1911_08020_amd as d
    for order in ("any", "end"):
        c = _counts(H, keep, H, order)
        plan = d.Plan.from_counts(H, c, int(c.sum()), 0, 1, 64)
        assert _chunks(d, plan) == _brute(plan.export()[0], H)
    # no recurrent matrix, or too wide a one
    for M, N in ((4 * H + 1, H), (4 * 4097, 4097)):
        c = np.ones(M, dtype=np.int64)
        assert _chunks(d, d.Plan.from_counts(N, c, M, 0, 1, 64)) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("H,keep", SIZES)
def test_device_plan_counts_chunks(darb, H, keep):  # noqa: F811
    say(f"lstm chunks H={H}")
    for order in ("any", "end"):
        for mode in (0, 1):
            c = _counts(H, keep, H, order)
            plan = darb.Plan.from_device_counts(H, dev(c), int(c.sum()), mode, 1, 64)
            assert _chunks(darb, plan) == _brute(plan.export()[0], H)
    for M, N in ((4 * H + 1, H), (4 * 4097, 4097)):
        plan = darb.Plan.from_device_counts(N, dev(np.ones(M, dtype=np.int64)), M, 0, 1, 64)
        assert _chunks(darb, plan) == 0
        assert plan.packed_words == darb.Plan.from_counts(N, np.ones(M, dtype=np.int64), M, 0, 1,
                                                          64).packed_words


@pytest.mark.gpu
@pytest.mark.parametrize("H,B,limit", [(512, 20, 1536), (512, 33, 1024), (1024, 64, 1024),
                                       (1500, 20, 1536), (2048, 32, 1536), (4095, 8, 1536)])
def test_one_launch_up_to_the_limit(darb, H, B, limit):  # noqa: F811
    # the first workgroup's rows grow denser, block size by block size, up to the last form
    # that fits and the first that does not; all others stay at b = 128
    say(f"lstm rule H={H} B={B}")
    units = -(-H // 32)
    chunks = lambda l: -(-(-(-H // (1 << l))) // 16)  # noqa: E731
    log2b = np.full(4 * H, 7)
    fits = None
    for r in [g * H + u for u in range(units) for g in range(4)]:
        for l in range(6, -1, -1):
            if -(-H // (1 << l)) > 512:                  # the rule's other condition
                break
            fits = log2b.copy()
            log2b[r] = l
            if sum(chunks(int(log2b[g * H + u])) for u in range(units) for g in range(4)) > limit:
                break
        else:
            continue
        if sum(chunks(int(log2b[g * H + u])) for u in range(units) for g in range(4)) > limit:
            break
    for lb, want in ((fits, True), (log2b, False)):
        counts = np.maximum(H >> lb, 1).astype(np.int64)
        plan = darb.Plan.from_counts(H, counts, int(counts.sum()), 0, 1, 128).upload()
        assert np.array_equal(plan.export()[0], lb)
        assert _chunks(darb, plan) == _brute(lb, H) and (_chunks(darb, plan) <= limit) == want
        assert bool(_applies(darb, plan, H, 16, B)) == want
        assert not _applies(darb, plan, H, 15, B)
