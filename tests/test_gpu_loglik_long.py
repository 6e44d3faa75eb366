"""The log joint's long documents (counted by a block of waves): against the
oracle to 1e-10 relative and the same value on every run, as for the others.
Lengths lie on either side of where a document is set aside (1,024 tokens, or
a wave's share where that is more), beside short and empty ones, more of them
than a wave sets aside, and the longest allowed."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1704_03581_amd import pulda
else:  # collected on CPU-only hosts, never run there
    pulda = None


@pytest.mark.parametrize("lens", [[1023, 1024, 1025, 0, 4096, 4097, 30], [65535, 0, 1], [20] * 500 + [5000] + [20] * 500,
                                  [1100] * 700 + [10] * 20, [90] * 40000 + [9000, 2000] + [90] * 10])
@pytest.mark.parametrize("K,priors", [(1, "symmetric"), (300, "symmetric"), (300, "vector"), (4096, "vector"),
                                      (4096, "symmetric")])
def test_long_documents(lens, K, priors):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(len(lens) + K)
    V = 200
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(np.asarray(lens, np.int64), out=off[1:])
    words = rng.integers(0, V, size=int(off[-1])).astype(np.int32)
    # topics of a skewed law, so that counts pass the table of 256 logs
    z = np.minimum(rng.geometric(min(1.0, 8.0 / K), size=int(off[-1])) - 1, K - 1).astype(np.uint16)
    alpha = rng.uniform(0.01, 1.0, size=K) if priors == "vector" else 0.1
    say(f"long documents: K={K} {priors} D={len(lens)} N={off[-1]}")
    p = pulda.Plan(K, V, len(lens), int(off[-1]), alpha=alpha, beta=0.02, seed=1)
    p.upload(off, words)
    p.init(z)
    want = oracle.loglik(off, words, z, alpha, 0.02, K, V)
    got = [p.loglik() for _ in range(3)]
    assert got[0] == got[1] == got[2]
    assert abs(got[0] - want) <= 1e-10 * abs(want), (got, want)
