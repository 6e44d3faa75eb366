"""Rows of draws past the 4 GiB that their three tables may span (one table
then): the same draws, z-steps and fold-in as with a smaller vocabulary, whose
tables lie within.  beta is so small that words without tokens draw nothing, so
both vocabularies give the same Phi."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_helpers import say

torch = pytest.importorskip("torch")
pulda = None
if torch.cuda.is_available():
    from paper_1704_03581_amd import pulda

K = 1000                        # padded to 1,024
V_THREE, V_ONE = 600000, 620000  # (4 K + 3 * 1024) V bytes: below and above 4 GiB


def _workspace(V):
    import os
    lib = C.CDLL(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1704_03581_amd",
                              "libpulda.so"))
    from tests.test_abi import Desc
    d, h, n = Desc(K, V, 0.01, 0.1, None, 100, 1), C.c_void_p(), C.c_int64()
    assert lib.pulda_plan_create(C.byref(d), C.c_int64(1), C.c_int64(1), C.byref(h)) == 0
    assert lib.pulda_plan_workspace_bytes(h, C.byref(n)) == 0
    lib.pulda_plan_destroy(h)
    return n.value


def test_one_table_holds_every_format():
    # the rows of a word: 4 bytes a padded topic, from 4 and 3 more in three
    # tables; everything else grows with V
    three, one = _workspace(V_THREE), _workspace(V_ONE)
    rest = three - V_THREE * (4 * K + 3 * 1024)
    assert abs(one - (rest / V_THREE + 4 * 1024) * V_ONE) <= 0.001 * one


@pytest.mark.gpu
@pytest.mark.parametrize("group", [64, 16, 1])
def test_one_table_draws_the_same(group):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(group)
    D, n = 4000, 100
    # two words hold most tokens, in few topics: rows of 32 and 16 bits
    words = rng.integers(0, V_THREE, size=D * n).astype(np.int32)
    z = rng.integers(0, K, size=D * n).astype(np.uint16)
    u = rng.random(D * n)
    words[u < 0.5], words[(u >= 0.5) & (u < 0.6)] = V_THREE - 1, 12345
    z[u < 0.5] = 999
    z[(u >= 0.5) & (u < 0.6)] = rng.integers(0, 20, size=int(((u >= 0.5) & (u < 0.6)).sum()))
    off = np.arange(D + 1, dtype=np.int64) * n
    docs = [words[a:a + 150] for a in (0, 1000, 5000)]
    out = []
    for V in (V_THREE, V_ONE):
        say(f"rows: group={group} V={V}")
        p = pulda.Plan(K, V, D, D * n, beta=1e-12, seed=4)
        p.upload(off, words)
        p.set_schedule([0], [group], [64])
        p.init(z)
        p.phi_step(1)
        g = p.get_phi()
        r = [p.get_z()]
        p.z_step(1)
        r.append(p.get_z())
        r += [pulda.FoldIn(p, sweeps=4, burn_in=1, max_slots=4, arena_tokens=600, max_len=200,
                           group=max(group, 16)).run_one(i, w)["theta"] for i, w in enumerate(docs)]
        # and from the values of that Phi
        p.set_phi(g["colptr"], g["topic"], g["phi"], g["alias_thr"], g["alias_topic"], g["sigma_a"])
        p.set_z(r[0])
        p.z_step(1)
        r.append(p.get_z())
        p.set_z(r[1])
        p.sweep(2, 2, want_ll=False)
        r.append(p.get_z())
        top = np.zeros(V, np.int64)
        np.maximum.at(top, np.repeat(np.arange(V), np.diff(g["colptr"].astype(np.int64))), g["gamma"])
        assert top[V_THREE - 1] >= 0xFFFF and 0xFF < top[12345] < 0xFFFF and 0 < np.median(top[top > 0]) <= 0xFF
        out.append((g, r))
        del p
        torch.cuda.empty_cache()
    for key in ("topic", "gamma", "phi", "alias_thr", "alias_topic", "S"):
        assert np.array_equal(out[0][0][key], out[1][0][key]), key
    assert np.array_equal(out[0][0]["colptr"], out[1][0]["colptr"][:V_THREE + 1])
    assert np.array_equal(out[0][0]["sigma_a"], out[1][0]["sigma_a"][:V_THREE])
    for a, b in zip(out[0][1], out[1][1]):
        assert np.array_equal(a, b)
    assert np.array_equal(out[0][1][1], out[0][1][-2])
