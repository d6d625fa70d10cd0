"""Finite embeddings whose squared norm is beyond float32: distances to such a
word are +inf, which must reach the sums of the documents that hold it and no
others, and must not be taken for a missing list entry."""
import numpy as np
import pytest

from oracle import emd_oracle as O
from synth.generators import CSR
import parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_02091_amd import lcemd

    lcemd.load_library()
    return lcemd


def _csr(rows):
    ptr = np.concatenate([[0], np.cumsum([len(c) for c, _ in rows])]).astype(np.int64)
    return CSR(ptr, np.concatenate([c for c, _ in rows]).astype(np.int32),
               np.concatenate([w for _, w in rows]).astype(np.float32))


def _rows(rng, lo, v, lengths):
    """Rows of the given lengths: distinct words of [lo, v), weights 1 - U[0,1)."""
    out = []
    for n in lengths:
        w = 1.0 - rng.random(n)
        out.append((np.sort(lo + rng.choice(v - lo, n, replace=False)), w / w.sum()))
    return out


# a group of eight non-zeros and its edges, two groups and theirs
LENGTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 33]


def _far_word(L, method, k, m, precision):
    """The lowest-numbered used word is infinitely far from everything: the
    documents without it have the oracle's distances whatever their length and
    the batch, those with it +inf."""
    rng = np.random.default_rng(51)
    v = 400
    V = rng.standard_normal((v, m)).astype(np.float32)
    V[0, 0] = 1e20
    rows = _rows(rng, 1, v, LENGTHS)
    db = _csr(rows + [(np.array([0, 9]), np.array([0.5, 0.5])), (np.array([0]), np.array([1.0]))])
    q = _csr(_rows(rng, 1, v, [int(x) for x in rng.integers(6, 60, 70)]))
    near = _csr(rows)
    want = O.Oracle(V, near.rowptr, near.col, near.val).matrix(q.rowptr, q.col, q.val, method, k, "d2q")
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    for B in (1, 8, 33, 64, 70):
        print(f"[gpu] far word {method} k={k} m={m} {precision} B={B}", flush=True)
        s = q.take(range(B))
        got = ctx.distances(s.rowptr, s.col, s.val, method=method, k=k, direction="d2q", precision=precision)
        P.assert_distances(got[:, :len(rows)], want[:B], f"B={B}")
        assert np.all(np.isposinf(got[:, len(rows):])), B
    ctx.close()


MEASURES = [("rwmd", 1), ("act", 2), ("act", 5), ("ict", 1)]


@pytest.mark.parametrize("method,k", MEASURES)
def test_a_far_word_is_in_its_own_documents_only(L, method, k):
    """Phase 2: batches per document, of 64 queries and (up to two entries a
    row) from LDS."""
    _far_word(L, method, k, 40, "fp32")


@pytest.mark.parametrize("B", [1, 64])
def test_a_far_entry_past_a_word_s_mass(L, B):
    """Walks that end before an infinite entry of their table row, at every
    entry of its second and third pair: lists of up to eight near words, then
    two far ones (each word is a document of its own too, so that its list goes
    on to them)."""
    rng = np.random.default_rng(52)
    v, m = 64, 4
    V = rng.standard_normal((v, m)).astype(np.float32)
    far, near = [10, 20], [1, 3, 5, 7, 11, 13, 15, 17]
    V[far, 0] = 1e20
    words = np.arange(40, 49)
    rows = [(words[:2], np.array([x, 1 - x])) for x in (0.95, 0.9, 0.8, 0.7, 0.6, 0.5)]
    rows += [(words, np.full(9, 1.0 / 9)), (words[:7], np.full(7, 1.0 / 7))]
    rows += [(np.array([w]), np.array([1.0])) for w in words]
    db = _csr(rows)
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    for used in range(3, 9):  # near words of weight 0.96 / used each, the far ones hold the rest
        c = np.array(sorted(near[:used] + far))
        q = _csr([(c, np.where(np.isin(c, far), 0.02, 0.96 / used))] * B)
        print(f"[gpu] far entry, {used} near words, B={B}", flush=True)
        got = ctx.distances(q.rowptr, q.col, q.val, method="act", k=c.size, direction="d2q")
        want = O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, "act", c.size, "d2q")
        for u, (_, x) in enumerate(rows):
            if x.max() > 0.96:  # some mass goes to the far words
                assert np.all(np.isposinf(got[:, u])), (used, u)
            else:
                P.assert_distances(got[:, u:u + 1], want[:, u:u + 1], f"{used} near words, document {u}")
    ctx.close()


@pytest.mark.parametrize("method,k", MEASURES)
def test_float32_tables_of_a_far_row(L, method, k):
    """At most 28 dims: positions past the query's words, which stand for word
    0, are no candidates."""
    _far_word(L, method, k, 3, "fp32")


@pytest.mark.parametrize("m", [3, 40])
def test_far_query_words_need_no_redo(L, monkeypatch, m):
    """A query word infinitely far from every row is a list entry like any
    other: no row has to be redone for it, so a redo list of one row is
    enough."""
    rng = np.random.default_rng(53)
    v = 300
    V = rng.standard_normal((v, m)).astype(np.float32)
    V[7, 0] = 1e20
    db = _csr(_rows(rng, 8, v, LENGTHS) + [(np.array([9]), np.array([1.0]))])
    q = _csr([(np.array([1, 4, 7]), np.array([0.5, 0.4, 0.1])), (np.array([7]), np.array([1.0])),
              (np.array([2, 7, 100]), np.array([0.2, 0.3, 0.5]))])
    monkeypatch.setenv("LCEMD_FIX_CAP", "1")
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    for method, k in (("rwmd", 1), ("act", 2), ("act", 3)):
        print(f"[gpu] far query word {method} k={k} m={m}", flush=True)
        got = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q")
        # (over several groups of eight the sum's compensation is inf - inf)
        assert not np.any(np.isfinite(got[1])), (method, k)
        if method == "rwmd":
            want = O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, method, k, "d2q")
            P.assert_distances(got[[0, 2]], want[[0, 2]])
    S, Z, _ = ctx.tables(q.rowptr, q.col, q.val, 3)
    assert np.all(S[1] == [0, -1, -1]) and np.all(np.isposinf(Z[1, :, 0]))
    for b, far in ((0, 2), (2, 1)):
        assert np.all(S[b, :, 2] == far) and np.all(np.isposinf(Z[b, :, 2])) and np.all(np.isfinite(Z[b, :, :2]))
    ctx.close()


@pytest.mark.parametrize("m", [3, 40])
def test_candidate_pairs_with_a_far_word(L, m):
    """A document of the far word alone, which the query holds too: nothing to
    move one way, an infinite way for the query's other word."""
    V = np.random.default_rng(54).standard_normal((50, m)).astype(np.float32)
    V[3, 0] = 1e20
    one = np.array([1.0])
    db = _csr([(np.array([3]), one)] + [(np.array([10 + i]), one) for i in range(30)])
    q = _csr([(np.array([2, 3]), np.array([0.5, 0.5]))])
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    print(f"[gpu] far pair m={m}", flush=True)
    idx, dist = ctx.topl(q.rowptr, q.col, q.val, db.n, method="rwmd", direction="sym")
    assert np.all(np.isposinf(dist)), (idx, dist)
    ctx.close()


@pytest.mark.parametrize("m", [3, 40])
@pytest.mark.parametrize("method,k", MEASURES)
def test_bf16_tables_of_a_far_row(L, method, k, m):
    """The exact re-sort keeps a listed word at an infinite distance."""
    _far_word(L, method, k, m, "bf16")


@pytest.mark.parametrize("m", [3, 40])
def test_bf16_tables_of_a_far_query_word(L, m):
    """Its listed entries are those of float32 keys."""
    rng = np.random.default_rng(55)
    v = 300
    V = rng.standard_normal((v, m)).astype(np.float32)
    V[7, 0] = 1e20
    db = _csr(_rows(rng, 8, v, LENGTHS))
    q = _csr([(np.array([1, 4, 7]), np.array([0.5, 0.4, 0.1])), (np.array([7]), np.array([1.0])),
              (np.array([20, 30]), np.array([0.5, 0.5]))])
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    print(f"[gpu] bf16, far query word m={m}", flush=True)
    for k in (1, 2, 3):
        a = ctx.tables(q.rowptr, q.col, q.val, k)
        b = ctx.tables(q.rowptr, q.col, q.val, k, precision="bf16")
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[2], b[2]) and np.allclose(a[1], b[1], rtol=1e-6), k
    want = O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, "rwmd", 1, "d2q")
    got = ctx.distances(q.rowptr, q.col, q.val, method="rwmd", direction="d2q", precision="bf16")
    P.assert_distances(got[[0, 2]], want[[0, 2]])
    assert not np.any(np.isfinite(got[1]))
    ctx.close()


def test_bf16_tables_of_a_row_of_zeros_and_a_far_query_word(L):
    """The row's error band has no number (0 times infinity), so nothing is
    listed: its table row is written all the same."""
    V = np.random.default_rng(56).standard_normal((60, 40)).astype(np.float32)
    V[7, 0] = 1e20
    V[9] = 0.0
    db = _csr([(np.array([9]), np.array([1.0])), (np.array([8, 9, 12]), np.array([0.5, 0.25, 0.25]))])
    q = _csr([(np.array([1, 7]), np.array([0.5, 0.5]))])
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    print("[gpu] bf16, row of zeros, far query word", flush=True)
    S, Z, W = ctx.tables(q.rowptr, q.col, q.val, 2, precision="bf16")
    assert np.all(S[0] == [0, 1]) and np.all(W[0] == 0.5) and np.all(np.isposinf(Z[0, :, 1]))
    assert np.allclose(Z[0, 1, 0], np.linalg.norm(V[1].astype(np.float64)), rtol=1e-6)  # (the used words: 8, 9, 12)
    got = ctx.distances(q.rowptr, q.col, q.val, method="rwmd", direction="d2q", precision="bf16")
    P.assert_distances(got, O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, "rwmd", 1, "d2q"))
    ctx.close()


@pytest.mark.parametrize("m", [3, 40])
@pytest.mark.parametrize("method,k", MEASURES)
def test_far_words_near_each_other(L, monkeypatch, method, k, m):
    """Far words that differ from each other by little: their keys are no
    numbers, so their order is that of the distances by direct differences."""
    rng = np.random.default_rng(57)
    v = 120
    V = rng.standard_normal((v, m)).astype(np.float32)
    far = rng.choice(v, 30, replace=False)
    V[far, 0] = 1e20
    group = [np.sort(far), np.setdiff1d(np.arange(v), far)]
    rows = []
    for i in range(40):  # documents and queries of far words only, or near ones only
        g = group[0] if i % 4 else group[1]
        n = int(rng.integers(1, 13))
        w = 1.0 - rng.random(n)
        rows.append((np.sort(rng.choice(g, n, replace=False)), w / w.sum()))
    db, q = _csr(rows[:30]), _csr([r for i, r in enumerate(rows) if i % 4])
    print(f"[gpu] far words near each other {method} k={k} m={m}", flush=True)
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    got = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q")
    want = O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, method, k, "d2q")
    docs = [u for u in range(30) if u % 4]  # (the others are infinitely far)
    P.assert_distances(got[:, docs], want[:, docs])
    assert not np.any(np.isfinite(got[:, [u for u in range(30) if u % 4 == 0]]))
    ctx.close()
    # without room for the redo the call still answers
    monkeypatch.setenv("LCEMD_FIX_CAP", "1")
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    got = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q")
    assert np.all(np.isfinite(got[:, docs]))
    ctx.close()
