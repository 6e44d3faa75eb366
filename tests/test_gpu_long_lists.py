"""Topic lists past the slots: documents on 64 lanes with more than 1,024 topics
sum their words' columns (short ones in registers, long ones in runs of 16
entries a lane), and fold-in and held-out documents that do not fit the lanes
asked for take more.  Compared with the oracle as in the other parity tests:
z by the teacher-forced replay, theta exactly, sums of logs to 1e-12 and the
held-out normalisers to 1e-10 relative."""
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


def _plan(lens, V, K, method, seed):
    rng = np.random.default_rng(seed)
    off = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    pr = 1.0 / (3.0 + np.arange(V))
    words = rng.choice(V, size=int(off[-1]), p=pr / pr.sum()).astype(np.int32)
    c = synth.Corpus("lists", len(lens), V, K, 0.1, 0.01, off, words, None)
    p = pulda.Plan(K, V, c.D, c.N, alpha=0.1, beta=0.01, seed=seed)
    p.upload(off, words)
    p.set_phi_method(method)
    p.init()
    return c, p


# columns of few entries (the urn) and of all topics (Gamma draws; 18, 32 and
# 64 entries a lane: runs of 16 with a rest of 2, whole, and the most)
@pytest.mark.parametrize("method", ["polya_urn", "dirichlet"])
@pytest.mark.parametrize("K", [1025, 1100, 2048, 4096])
def test_z_step_of_long_lists(K, method):
    c, p = _plan([30, 1200, 6000, 300, 20000], 400, K, method, seed=K)
    say(f"long lists: K={K} {method} N={c.N}")
    p.set_schedule([0], [64], [1])
    for t in (1, 2):
        z0 = p.get_z()
        p.phi_step(t)
        phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
        p.z_step(t)
        z1 = p.get_z()
        r = oracle.replay(c.doc_off, c.words, z0, z1, K, t, phi, wt, K, c.V)
        say(f"  sweep {t}: {r}")
        assert r["bad"] == 0 and r["agree"] >= 0.9999 * c.N, r
        n_o, _, _ = oracle.counts(c.doc_off, c.words, z1, K, c.V, with_m=False)
        assert np.array_equal(p.counts_dense()[0], n_o)
        _, deg, sumJ, sumA = oracle.z_step(c.doc_off, c.words, z0, K, t, phi, wt, K, c.V, sparse=True)
        st = p.stats()
        assert st["degenerate_tokens"] == deg
        if r["ties"] == 0:
            assert (st["sum_J"], st["sum_A"]) == (sumJ, sumA)


# requests and documents on either side of what the lanes' slots hold, alone
# and beside each other (a step's lanes follow its longest request)
@pytest.mark.parametrize("method", ["polya_urn", "dirichlet"])
@pytest.mark.parametrize("group,K,lens", [(16, 300, [0, 40, 239, 240, 241, 600]), (32, 600, [10, 479, 480, 481, 1300]),
                                          (16, 1500, [5, 400, 900, 3000]), (64, 1500, [100, 960, 961, 4000])])
def test_lanes_for_new_documents(group, K, lens, method):
    c, p = _plan([200] * 40, 500, K, method, seed=group + K)
    say(f"lanes: group={group} K={K} {method}")
    p.sweep(1, 2, want_ll=False)
    p.phi_step(3)
    phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
    rng = np.random.default_rng(K)
    docs = [rng.integers(0, c.V, size=n).astype(np.int32) for n in lens]
    f = pulda.FoldIn(p, sweeps=3, burn_in=1, max_slots=8, arena_tokens=sum(lens) + 8, max_len=max(lens), group=group,
                     seed=5)
    want = [oracle.foldin(phi, wt, 0.1, 5, i, w, S=3, burn_in=1) for i, w in enumerate(docs)]
    got = [f.run_one(i, w) for i, w in enumerate(docs)]
    # all at once, in steps that end inside sweeps
    for i, w in enumerate(docs):
        assert f.submit(i, w)
    more = {}
    for _ in range(3 * max(lens) // 333 + 4):
        f.step(333)
        for r in f.poll(8):
            more[r["request_id"]] = r
    for i, (theta, ll, kept, dropped, _) in enumerate(want):
        for r in (got[i], more[i]):
            assert (r["kept"], r["dropped"]) == (kept, dropped)
            assert np.array_equal(r["theta"], theta), (i, len(docs[i]))
            assert abs(r["loglik"] - ll) <= 1e-12 * max(1.0, abs(ll))


# topics that were not likely to pass the slots of 16 lanes (240 of 4,096 at up to
# 247 tokens) and do, beside a block's 16 a-parts
@pytest.mark.parametrize("method", ["polya_urn", "dirichlet"])
def test_lists_that_overflow_few_lanes(method):
    K, n, R = 4096, 247, 24
    c, p = _plan([200] * 40, 500, K, method, seed=7)
    say(f"overflow: {method}")
    p.sweep(1, 1, want_ll=False)
    p.phi_step(2)
    phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
    rng = np.random.default_rng(1)
    docs = [rng.integers(0, c.V, size=n).astype(np.int32) for _ in range(R)]
    first = [len({(int(oracle.philox([q, i, 0, 4], [5, 0])[0]) * K) >> 32 for q in range(n)}) for i in range(R)]
    assert max(first) >= 243
    f = pulda.FoldIn(p, sweeps=3, burn_in=1, max_slots=R, arena_tokens=R * n, max_len=n, group=16, seed=5)
    for i, w in enumerate(docs):
        assert f.submit(i, w)
    f.step(2 ** 31 - 1)
    got = {r["request_id"]: r for r in f.poll(R)}
    for i, w in enumerate(docs):
        theta, ll, kept, dropped, _ = oracle.foldin(phi, wt, 0.1, 5, i, w, S=3, burn_in=1)
        r = got[i]
        assert (r["kept"], r["dropped"]) == (kept, dropped)
        assert np.array_equal(r["theta"], theta), (i, first[i])
        assert abs(r["loglik"] - ll) <= 1e-12 * max(1.0, abs(ll))


# many documents (a document's blocks on one XCD) and few; some past 32 lanes
@pytest.mark.parametrize("group", [16, 32, 64])
@pytest.mark.parametrize("D", [3, 63, 64, 70])
def test_held_out_blocks(D, group):
    K = 600
    c, p = _plan([200] * 40, 500, K, "polya_urn", seed=3)
    say(f"held-out blocks: D={D} group={group}")
    p.sweep(1, 1, want_ll=False)
    p.phi_step(2)
    phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
    rng = np.random.default_rng(D)
    lens = rng.integers(0, 40, size=D)
    lens[D // 2] = 1100 if D == 70 else 45
    docs = [rng.integers(0, c.V, size=n).astype(np.int32) for n in lens]
    R = 3
    ll, kept, Z = p.heldout_loglik(docs, particles=R, group=group, seed=9, want_Z=True)
    for i, w in enumerate(docs):
        if len(w) > 1000:
            continue   # (long for the oracle; the documents beside it are checked)
        e, k, Zo = oracle.heldout_ltr(phi, wt, 0.1, 9, i, w, R, want_Z=True)
        assert kept[i] == k
        assert np.all(np.abs(Z[i] - Zo) <= 1e-10 * np.abs(Zo))
        assert abs(ll[i] - e) <= 1e-12 * max(1.0, abs(e))


@pytest.mark.parametrize("group,K,lens", [(16, 300, [30, 250]), (32, 520, [500]), (64, 1100, [20, 1200])])
def test_lanes_for_held_out_documents(group, K, lens):
    c, p = _plan([200] * 40, 500, K, "polya_urn", seed=group + K)
    say(f"held-out lanes: group={group} K={K}")
    p.sweep(1, 2, want_ll=False)
    p.phi_step(3)
    phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
    rng = np.random.default_rng(K)
    docs = [rng.integers(0, c.V, size=n).astype(np.int32) for n in lens]
    ll, kept, Z = p.heldout_loglik(docs, particles=2, group=group, seed=9, want_Z=True)
    for i, w in enumerate(docs):
        e, k, Zo = oracle.heldout_ltr(phi, wt, 0.1, 9, i, w, 2, want_Z=True)
        assert kept[i] == k
        assert np.all(np.abs(Z[i] - Zo) <= 1e-10 * np.abs(Zo))
        assert abs(ll[i] - e) <= 1e-12 * abs(e)


# phi's own rows: documents not likely to fit 32 lanes' slots on 64, beside the others;
# rows of draws: all on 64 where one could fill them
@pytest.mark.parametrize("method", ["polya_urn", "dirichlet"])
@pytest.mark.parametrize("group", [16, 32])
def test_held_out_lanes_by_the_document(group, method):
    K = 4096
    c, p = _plan([200] * 40, 500, K, method, seed=group)
    say(f"held-out lanes by the document: group={group} {method}")
    p.sweep(1, 1, want_ll=False)
    p.phi_step(2)
    phi, wt = phi_from_gpu(p.get_phi(), K, c.V)
    rng = np.random.default_rng(group)
    docs = [rng.integers(0, c.V, size=n).astype(np.int32) for n in (30, 520, 0, 300, 525, 40)]
    ll, kept, Z = p.heldout_loglik(docs, particles=2, group=group, seed=9, want_Z=True)
    for i, w in enumerate(docs):
        e, k, Zo = oracle.heldout_ltr(phi, wt, 0.1, 9, i, w, 2, want_Z=True)
        assert kept[i] == k
        assert np.all(np.abs(Z[i] - Zo) <= 1e-10 * np.abs(Zo))
        assert abs(ll[i] - e) <= 1e-12 * max(1.0, abs(e))
