"""Float32 phase-1 tables selected in registers: list sizes, tile and pass
edges, row-block edges, ties and negative keys, against float64 tables."""
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


# query lengths: one word, a 32-word tile and its edges, a pass of four tiles
# and its edges, even splits into two and three passes
HQ = [1, 2, 16, 31, 32, 33, 64, 65, 96, 97, 127, 128, 129, 160, 161, 257, 300]


def _queries(rng, v, lengths):
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(v, n, replace=False)) for n in lengths]).astype(np.int32)
    val = np.concatenate([w / w.sum() for w in (1.0 - rng.random(n) for n in lengths)]).astype(np.float32)
    return CSR(ptr, col, val)


@pytest.mark.parametrize("m", [3, 28, 29, 44, 100])
@pytest.mark.parametrize("k", [1, 2, 3, 8, 16, 17, 32])
def test_tables(L, m, k):
    """S/Z/W of every used word (row blocks of 128 and a part one) for list
    sizes 1-32; words scaled so that keys of both signs occur."""
    rng = np.random.default_rng(41)
    v = 400
    V = (rng.standard_normal((v, m)) * rng.choice([0.3, 1.0, 3.0], (v, 1))).astype(np.float32)
    words = np.arange(0, v, 1)[: 128 * 2 + 37].astype(np.int32)
    dbptr = np.array([0, words.size], dtype=np.int64)
    ctx = L.open_context(V, dbptr, words, np.full(words.size, 1.0 / words.size, np.float32))
    q = _queries(rng, v, HQ)
    print(f"[gpu] tables m={m} k={k}", flush=True)
    S, Z, W = ctx.tables(q.rowptr, q.col, q.val, k)
    for b in range(q.n):
        qc, qw = q.row(b)
        R = O.squared_distances(V[words], V[qc])
        So = np.argsort(R, axis=1, kind="stable")
        P.check_table_rows(S[b], Z[b], W[b], So[:, : min(k, qc.size)], R, qw, k, qc.size)
    ctx.close()


def test_ties_go_to_the_lower_position(L):
    """Grid coordinates: every distance ties with others, exactly."""
    rng = np.random.default_rng(42)
    side = 20
    V = np.stack(np.divmod(np.arange(side * side), side), 1).astype(np.float32)
    words = np.arange(side * side, dtype=np.int32)
    ctx = L.open_context(V, np.array([0, words.size], dtype=np.int64), words, np.full(words.size, 1 / words.size, np.float32))
    q = _queries(rng, side * side, [5, 40, 130, 200])
    for k in (2, 4, 16):
        S, _, _ = ctx.tables(q.rowptr, q.col, q.val, k)
        for b in range(q.n):
            qc, _ = q.row(b)
            So = np.argsort(O.squared_distances(V, V[qc]), axis=1, kind="stable")[:, : min(k, qc.size)]
            assert np.array_equal(S[b][:, : So.shape[1]], So), (k, b)
    ctx.close()


@pytest.mark.parametrize("method,k", [("rwmd", 1), ("omr", 1), ("act", 3), ("act", 20), ("ict", 1)])
@pytest.mark.parametrize("m", [2, 50])
def test_distances(L, method, k, m):
    rng = np.random.default_rng(43)
    v = 500
    V = rng.standard_normal((v, m)).astype(np.float32)
    db, q = _queries(rng, v, [1, 3, 40, 128, 200, 77] * 6), _queries(rng, v, HQ)
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    orc = O.Oracle(V, db.rowptr, db.col, db.val)
    print(f"[gpu] distances {method} k={k} m={m}", flush=True)
    for d in ("d2q", "q2d"):
        got = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction=d)
        P.assert_distances(got, orc.matrix(q.rowptr, q.col, q.val, method, k, d), f"{method} {d}")
    ctx.close()


@pytest.mark.parametrize("method,k", [("omr", 1), ("act", 2), ("act", 7), ("act", 30)])
@pytest.mark.parametrize("m", [2, 27, 60])
def test_candidate_pairs(L, method, k, m):
    """Q2D of candidate pairs: row blocks of 128 query words (partial sums of
    64 at up to 28 dims), segments around the tile and pass edges."""
    rng = np.random.default_rng(44)
    v = 600
    V = rng.standard_normal((v, m)).astype(np.float32)
    db = _queries(rng, v, [1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 300, 513, 40, 90])
    q = _queries(rng, v, [1, 31, 33, 63, 64, 65, 127, 128, 129, 192, 193, 300, 520])
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    orc = O.Oracle(V, db.rowptr, db.col, db.val)
    print(f"[gpu] pairs {method} k={k} m={m}", flush=True)
    idx, dist = ctx.topl(q.rowptr, q.col, q.val, 5, method=method, k=k, direction="sym")
    want = orc.matrix(q.rowptr, q.col, q.val, method, k, "sym")
    off = sum(P.check_topl(idx[b], dist[b], want[b], 5, f"{method} query {b}") for b in range(q.n))
    assert off <= 2
    ctx.close()


@pytest.mark.parametrize("k", [1, 2, 8, 16])
def test_queries_that_share_an_item(L, k):
    """Batches large enough that an item takes eight queries end to end give
    what each query alone gives (one query per item), bit for bit: queries
    that end inside, at and past a tile's edge, several within one tile, and
    more words than an item holds at a time."""
    rng = np.random.default_rng(46)
    v, nu, m, nq = 17000, 16500, 40, 150
    V = rng.standard_normal((v, m)).astype(np.float32)
    words = np.arange(nu, dtype=np.int32)
    ptr = np.arange(0, nu + 1, 500, dtype=np.int64)
    ctx = L.open_context(V, ptr, words, np.full(nu, 1.0 / 500, np.float32))
    lengths = rng.integers(1, 70, nq)
    lengths[:24] = [1, 1, 1, 29, 32, 64, 31, 33, 1024, 1024, 1, 1023, 1024, 2, 500, 700, 32, 32, 32, 32, 5, 6, 7, 8]
    q = _queries(rng, v, lengths.tolist())
    print(f"[gpu] shared items k={k}", flush=True)
    S, Z, W = ctx.tables(q.rowptr, q.col, q.val, k)
    for b in list(range(24)) + [70, 147, 148, 149]:
        qc, qw = q.row(b)
        s1, z1, w1 = ctx.tables(np.array([0, qc.size], dtype=np.int64), qc, qw, k)
        assert np.array_equal(S[b], s1[0]) and np.array_equal(Z[b], z1[0]) and np.array_equal(W[b], w1[0]), b
    for method in ("rwmd", "omr", "act"):
        g = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q")
        for b in (0, 8, 9, 15, 149):
            qc, qw = q.row(b)
            one = ctx.distances(np.array([0, qc.size], dtype=np.int64), qc, qw, method=method, k=k, direction="d2q")
            assert np.allclose(g[b], one[0], rtol=1e-6, atol=1e-7), (method, b)
    ctx.close()
