"""Draws behind an undecided one.  On 64 lanes a round of draws is made at once;
where fp32 leaves one undecided, the round is taken back and the draws behind it
are made again, now with that token's count.  Here the third draw of a round
takes a slot in the first pass and the a-part in the second: its drawn slot must
not be left behind.

The document: every token has a word of its own, whose column, sigma_a and a-part
topic are chosen.  Tokens 0 to 2 start in topic 3, m_0 others in topic 0.
  token 0: y = u (sigma_a + T) - sigma_a within rounding of 0, exactly just
           below: undecided in fp32, the a-part (topic 1) in fp64;
  token 1: topics 0 and 1, topic 1 far heavier: topic 1 if token 0 counts there,
           else topic 0;
  token 2: topic 0 only, sigma_a between what m_0 and m_0 + 1 tokens give: the
           a-part (topic 4) unless token 1 went to topic 0."""
import numpy as np
import pytest

import oracle
from tests.gpu_helpers import say

torch = pytest.importorskip("torch")
pulda = None
if torch.cuda.is_available():
    from paper_1704_03581_amd import pulda

TAG_Z = 3
T_SWEEP = 1
# tokens in topic 0 and topics with one token each: one to four slots a lane,
# counts in bytes of one register and (past 255 tokens) in registers of their own
SHAPES = [(37, 0), (40, 80), (30, 150), (12, 235), (300, 0), (250, 100), (200, 180)]


def _u(seed, i):
    r = oracle.philox([i, 0, T_SWEEP, TAG_Z], [seed & 0xFFFFFFFF, seed >> 32])
    return float(int(r[0]) >> 8) * 2.0 ** -24


def _seed():
    for seed in range(1, 1000):
        if all(0.3 < _u(seed, i) < 0.7 for i in range(3)):
            return seed
    raise AssertionError("no seed")


def _document(m0, others, seed):
    """K, z, and the columns: per word a list of (topic, phi), sigma_a, the
    a-part's topic."""
    K = 5 + others
    z = np.array([3, 3, 3] + [0] * m0 + list(range(5, 5 + others)), np.uint16)
    u = [_u(seed, i) for i in range(3)]
    a = 2.0 ** -14
    cols = [([(0, 0.25)], u[0] * 0.25 * m0 / (1.0 - u[0]) * (1.0 + 2.0 ** -30), 1),
            ([(0, a), (1, 30.0 * m0 * a)], 1e-3 * a, 2),
            ([(0, 0.125)], u[2] * 0.125 * (m0 + 0.5) / (1.0 - u[2]), 4)]
    for i in range(3, len(z)):
        cols.append(([(int(z[i]), 0.5)], 1e-4, int(z[i])))
    return K, z, cols


def _tables(K, cols):
    V = len(cols)
    phi = np.zeros((K, V), np.float32)
    colptr, topic, val, thr, alias, sa = [0], [], [], [], [], []
    for v, (entries, s, ka) in enumerate(cols):
        for k, f in entries:
            phi[k, v] = f
            topic.append(k)
            val.append(f)
            thr.append(0)          # (never below it: always the alias)
            alias.append(ka)
        colptr.append(len(topic))
        sa.append(s)
    return phi, oracle.WordTables(np.array(colptr, np.int64), np.array(topic, np.uint16), np.array(val, np.float32),
                                  np.array(thr, np.uint32), np.array(alias, np.uint16), np.array(sa, np.float64))


def _first_round(m0, cols, seed, restore):
    """The first three draws as rounds make them, in a model on the CPU: topics
    drawn, and which draws the first pass left undecided.  restore: the draws
    behind the undecided one are a-parts again before they are made anew."""
    tol = 72.0 * 2.0 ** -24
    u = [_u(seed, i) for i in range(3)]
    out = [cols[i][2] for i in range(3)]       # the a-part's, until a slot is drawn
    counts = {0: m0}

    def draw(i, exact):
        entries, sa, ka = cols[i]
        terms = [(k, np.float32(f) * counts.get(k, 0)) for k, f in entries]
        T = sum(float(b) for _, b in terms)
        y = u[i] * (sa + T) - sa
        if not exact and abs(y) < tol * (sa + T):
            return None
        if y < 0:
            return -1
        c = 0.0
        for k, b in terms:
            c += float(b)
            if c > y:
                return k
        raise AssertionError("no crossing")

    open_draws = []
    for i in range(3):
        k = draw(i, False)
        if k is None:
            open_draws.append(i)
            continue
        k1 = cols[i][2] if k < 0 else k
        if k >= 0:
            out[i] = k
        counts[k1] = counts.get(k1, 0) + 1
    assert open_draws == [0]
    first = list(out)
    counts = {0: m0}
    if restore:
        out = [cols[i][2] for i in range(3)]
    for i in range(3):
        k = draw(i, i == 0)
        assert k is not None
        k1 = cols[i][2] if k < 0 else k
        if k >= 0:
            out[i] = k
        counts[k1] = counts.get(k1, 0) + 1
    return first, out


@pytest.mark.parametrize("m0,others", SHAPES)
def test_the_third_draw_turns_to_the_a_part(m0, others):
    seed = _seed()
    K, z, cols = _document(m0, others, seed)
    first, out = _first_round(m0, cols, seed, restore=True)
    assert first[1:] == [0, 0] and out == [1, 1, 4]
    # a slot left behind is another result
    assert _first_round(m0, cols, seed, restore=False)[1] == [1, 1, 0]
    phi, wt = _tables(K, cols)
    off = np.array([0, len(z)], np.int64)
    zo = oracle.z_step(off, np.arange(len(z)), z, seed, T_SWEEP, phi, wt, K, len(z), sparse=True)[0]
    assert list(zo[:3]) == out


@pytest.mark.gpu
@pytest.mark.parametrize("m0,others", SHAPES)
def test_no_slot_is_left_behind(m0, others):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    seed = _seed()
    K, z, cols = _document(m0, others, seed)
    phi, wt = _tables(K, cols)
    N = len(z)
    off, words = np.array([0, N], np.int64), np.arange(N, dtype=np.int32)
    want = oracle.z_step(off, words, z, seed, T_SWEEP, phi, wt, K, N, sparse=True)[0]
    for group in (64, 32):
        p = pulda.Plan(K, N, 1, N, alpha=0.1, beta=0.01, seed=seed)
        p.upload(off, words)
        p.set_schedule([0], [group], [64])
        p.init(z)
        p.set_phi(wt.colptr, wt.topic, wt.phi, wt.thr, wt.alias_topic, wt.sigma_a)
        p.z_step(T_SWEEP)
        got = p.get_z()
        st = p.stats()
        say(f"open draw: group={group} m0={m0} others={others}: {list(got[:3])}, {st['fallback_draws']} undecided")
        assert st["fallback_draws"] >= 1
        assert np.array_equal(got, want), (group, list(got[:3]), list(want[:3]))
