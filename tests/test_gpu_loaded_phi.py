"""Phi loaded as values of any size: a column's largest value is a bound in the
word's record, beside the row's format.  Scaling every value and sigma_a by a
power of two scales every sum exactly, so the draws are the same; single values
of 2 and more, of the largest floats and infinite ones are drawn as the oracle
draws them (its sparse z-step, where a topic without a count has no term)."""
import numpy as np
import pytest

import oracle
from paper_1704_03581_amd import synth
from tests.gpu_helpers import phi_from_gpu, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1704_03581_amd import pulda
else:  # collected on CPU-only hosts, never run there
    pulda = None


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _corpus(K, seed):
    rng = np.random.default_rng(seed)
    lens = np.concatenate([[0, 1, 2, 7, 8, 9, 63, 64, 65, 110], rng.integers(3, 100, size=120)])
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    V = 150
    words = rng.integers(0, V, size=int(off[-1])).astype(np.int32)
    return synth.Corpus("loaded", len(lens), V, K, 0.1, 0.01, off, words, None)


def _plan(c, group, seed=3):
    p = pulda.Plan(c.K, c.V, c.D, c.N, alpha=c.alpha, beta=c.beta, seed=seed)
    p.upload(c.doc_off, c.words)
    p.set_schedule([0], [group], [64])
    p.init()
    p.phi_step(1)
    return p


def _load(p, g, **changed):
    a = dict(g, **changed)
    p.set_phi(a["colptr"], a["topic"], a["phi"], a["alias_thr"], a["alias_topic"], a["sigma_a"])


@pytest.mark.parametrize("K", [24, 300])
@pytest.mark.parametrize("group", [64, 32, 16, 8, 1])
def test_scaled_phi_draws_the_same(group, K):
    c = _corpus(K, seed=K)
    say(f"scaled phi: group={group} K={K}")
    p, q = _plan(c, group), _plan(c, group)
    g = p.get_phi()
    z0 = p.get_z()
    f = 2.0 ** 16
    big = (g["phi"] * np.float32(f)).astype(np.float32)
    assert big.max() >= 1024.0
    _load(p, g)
    _load(q, g, phi=big, sigma_a=g["sigma_a"] * f)
    docs = [np.arange(n, dtype=np.int32) % c.V for n in (1, 60, 140)]
    out = []
    for x in (p, q):
        x.z_step(2)
        h = x.heldout_loglik(docs, particles=3, group=64 if group < 16 else group, want_Z=True)[2]
        r = [pulda.FoldIn(x, sweeps=6, burn_in=2, max_slots=4, arena_tokens=400, max_len=200,
                          group=64 if group < 16 else group, seed=5).run_one(0, w) for w in docs]
        out.append((x.get_z(), r, h))
    assert np.array_equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1], out[1][1]):
        assert (a["kept"], a["dropped"]) == (b["kept"], b["dropped"])
        assert np.array_equal(a["theta"], b["theta"])
    for a, b in zip(out[0][2], out[1][2]):
        assert np.array_equal(a * f, b)
    phi, wt = phi_from_gpu(q.get_phi(), c.K, c.V)
    r = oracle.replay(c.doc_off, c.words, z0, out[1][0], 3, 2, phi, wt, c.K, c.V)
    assert r["bad"] == 0 and r["agree"] >= 0.9999 * c.N, r


@pytest.mark.parametrize("value", [np.nextafter(np.float32(2.0), np.float32(0.0)), 2.0, 4.0, 3.0e38, np.inf])
@pytest.mark.parametrize("group", [64, 32, 16, 8, 1])
def test_single_large_values(group, value):
    c = _corpus(24, seed=9)
    say(f"large values: group={group} value={value}")
    p = _plan(c, group)
    g = p.get_phi()
    z0 = p.get_z()
    phi = g["phi"].copy()
    cols = np.repeat(np.arange(c.V), np.diff(g["colptr"].astype(np.int64)))
    # the whole first word (the row that a record without a draw reads), the
    # last word's first topic, and every 11th entry
    phi[cols == 0] = value
    phi[np.flatnonzero(cols == cols[-1])[0]] = value
    phi[::11] = value
    _load(p, g, phi=phi)
    p.z_step(2)
    dense, wt = phi_from_gpu(p.get_phi(), c.K, c.V)
    assert np.array_equal(wt.phi.view(np.uint32), phi.view(np.uint32))
    with np.errstate(all="ignore"):
        want = oracle.z_step(c.doc_off, c.words, z0, 3, 2, dense, wt, c.K, c.V, sparse=True)
    z1 = p.get_z()
    assert np.array_equal(z1, want[0])
    n_o, _, _ = oracle.counts(c.doc_off, c.words, z1, c.K, c.V, with_m=False)
    assert np.array_equal(p.counts_dense()[0], n_o)
    st = p.stats()
    assert (st["sum_J"], st["sum_A"], st["degenerate_tokens"]) == (want[2], want[3], want[1])
