"""The pruning's sampled split at ragged sizes, against the oracle: rows of any length and
alignment, rows of very different density."""
import numpy as np
import pytest

import oracle
from tests._gpu import darb, dev, host, say, torch  # noqa: F401

pytestmark = pytest.mark.gpu


# 20 MiB is where the sampled split begins: just below, just above (fp32, fp16), rows shorter
# than a sampled piece, rows that start on any element, a leading dimension of its own
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("M,N,skip", [(2621, 2000, 0), (2622, 2000, 0), (5242, 2000, 0),
                                      (5243, 2000, 0), (5243, 1001, 0),
                                      (1048600, 5, 0), (80000, 67, 1), (60000, 129, 0), (41, 131073, 3)])
def test_prune_split_at_ragged_sizes(darb, dtype, M, N, skip):  # noqa: F811
    say(f"prune {M}x{N} {np.dtype(dtype).name} skip {skip}")
    rng = np.random.default_rng(M + N)
    W = rng.standard_normal((M, N), dtype=np.float32)
    W *= np.exp(1.0 * rng.standard_normal((M, 1), dtype=np.float32))   # densities of rows differ
    W = W.astype(dtype)
    flat = np.zeros(M * (N + skip) + skip, dtype=dtype)
    flat[skip:].reshape(M, N + skip)[:, :N] = W
    Wd = dev(flat)[skip:].view(M, N + skip)[:, :N]
    for k in (int(0.06 * M * N), M * N // 2, 1):
        got = host(darb.prune_counts(Wd, k))
        assert np.array_equal(got, oracle.prune_counts(W, k)), k
        assert got.sum() == k


def test_biased_pieces_fall_back_to_w(darb):  # noqa: F811
    # the sample's pieces are 16 vectors of 4 fp32 keys, 32 times that plus 37 vectors
    # apart: rows exactly one such stride long put every piece at the first 64 columns.
    # Values spread over 20 octaves only there propose a bracket near the top, while the
    # threshold lies in the rest of W: the later passes must go back to W
    rng = np.random.default_rng(5)
    M, N = 2500, 32 * 64 + 37 * 4
    W = rng.uniform(0.0, 0.5, size=(M, N)).astype(np.float32)
    W[:, :64] = np.exp2(rng.uniform(0.0, 20.0, size=(M, 64))).astype(np.float32)
    k = int(0.05 * M * N)
    say(f"biased sample: {M}x{N} fp32, k = {k}")
    assert np.array_equal(host(darb.prune_counts(dev(W), k)), oracle.prune_counts(W, k))
