"""The scan of Phi's columns past 16 tiles of 4,096 words (each tile summed
before) and on either side of that, against the oracle; integers and phi exactly.
Long columns (more than 256 nonzeros) lie in the first, a middle and the last
tile."""
import numpy as np
import pytest

from tests.gpu_helpers import assert_phi_equal, oracle_phi, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1704_03581_amd import pulda
else:  # collected on CPU-only hosts, never run there
    pulda = None


@pytest.mark.parametrize("V,K", [(65535, 1), (65536, 2), (65537, 2), (69633, 300), (524289, 3), (1200000, 1)])
def test_scan_of_many_columns(V, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(V)
    N, D = 60000, 600
    words = rng.integers(0, V, size=N).astype(np.int32)
    for w in (0, V // 2, V - 1):
        words[rng.choice(N, size=4000, replace=False)] = w
    off = np.arange(D + 1, dtype=np.int64) * (N // D)
    say(f"columns: V={V} K={K}")
    beta = 0.01 if K < 100 else 1e-4
    p = pulda.Plan(K, V, D, N, alpha=0.1, beta=beta, seed=4)
    p.upload(off, words)
    p.init()
    z = p.get_z()
    p.phi_step(2)
    gam, S, phi, wt = oracle_phi(off, words, z, K, V, 0.1, beta, 100, 4, 2)
    if K > 256:
        assert (np.diff(wt.colptr) > 256).sum() == 3
    assert_phi_equal(p.get_phi(), gam, S, phi, wt, K, V)
    st = p.stats()
    assert st["nnz_phi"] == len(wt.topic) and st["empty_rows"] == int((S == 0).sum())
