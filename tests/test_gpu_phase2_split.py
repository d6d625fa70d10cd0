"""Phase 2's splits over lanes and waves (chosen by the batch size and the
table size): every split gives the bits of every other, and the float64
oracle's distances."""
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


def _histograms(rng, v, lengths):
    """Rows of the given lengths: distinct words, weights 1 - U[0,1)."""
    ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(v, n, replace=False)) for n in lengths]).astype(np.int32)
    val = np.concatenate([w / w.sum() for w in (1.0 - rng.random(n) for n in lengths)]).astype(np.float32)
    return CSR(ptr, col, val)


# one group of eight non-zeros, its edges, a step of eight groups and its edges
LENGTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 71, 72, 73, 127, 128, 129, 3]


@pytest.mark.parametrize("method,k", [("act", 1), ("act", 2), ("act", 5), ("ict", 1)])
def test_batch_sizes_give_the_same_bits(L, method, k):
    """Lane widths 1-64: a query's distances do not depend on the batch."""
    rng = np.random.default_rng(31)
    v, m = 300, 12
    V = rng.standard_normal((v, m)).astype(np.float32)
    db = _histograms(rng, v, LENGTHS)
    q = _histograms(rng, v, [int(x) for x in rng.integers(1, 60, 70)])
    ctx = L.open_context(V, db.rowptr, db.col, db.val)
    full = ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q")
    P.assert_distances(full, O.Oracle(V, db.rowptr, db.col, db.val).matrix(q.rowptr, q.col, q.val, method, k, "d2q"))
    for B in (1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65):
        print(f"[gpu] {method} k={k} B={B}", flush=True)
        s = q.take(range(B))
        got = ctx.distances(s.rowptr, s.col, s.val, method=method, k=k, direction="d2q")
        assert np.array_equal(got.view(np.uint32), full[:B].view(np.uint32)), B
    ctx.close()


@pytest.mark.parametrize("method,k,words", [("rwmd", 1, 784), ("act", 2, 784), ("omr", 1, 809), ("act", 2, 810),
                                            ("act", 1, 2048), ("act", 5, 784)])
@pytest.mark.parametrize("n,B", [(127, 33), (129, 49), (300, 64), (4000, 31)])
def test_small_vocabulary_gives_the_per_document_bits(L, monkeypatch, method, k, words, n, B):
    """Tables in LDS (up to 809 words at two entries per row, 2,048 at one)
    against the per-document walk, over part windows, part query groups and
    document lengths around a step of 16; a few rows against the oracle."""
    rng = np.random.default_rng(32)
    V = rng.standard_normal((words, 3)).astype(np.float32)
    lengths = [int(x) for x in rng.choice([1, 7, 8, 9, 15, 16, 17, 24, 25, 33, 48], n)]
    db = _histograms(rng, words, [words // 2] + lengths[1:])
    q = _histograms(rng, words, [int(x) for x in rng.integers(1, 40, B)])
    rows = [db.row(i) for i in range(db.n)]
    # every word is used, so the table has `words` rows
    for a in range(0, words, 900):
        c = np.arange(a, min(words, a + 900), dtype=np.int32)
        rows.append((c, np.full(c.size, 1.0 / c.size, np.float32)))
    ptr = np.concatenate([[0], np.cumsum([len(c) for c, _ in rows])]).astype(np.int64)
    col, val = np.concatenate([c for c, _ in rows]), np.concatenate([w for _, w in rows])
    got = []
    for route in ("0", "2"):  # by size; per document
        monkeypatch.setenv("LCEMD_PHASE2", route)
        ctx = L.open_context(V, ptr, col, val)
        print(f"[gpu] {method} k={k} words={words} n={n} B={B} route={route}", flush=True)
        got.append(ctx.distances(q.rowptr, q.col, q.val, method=method, k=k, direction="d2q"))
        ctx.close()
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    few = q.take([0, B - 1])
    orc = O.Oracle(V, ptr[:41], col[:ptr[40]], val[:ptr[40]])
    P.assert_distances(got[0][[0, B - 1], :40], orc.matrix(few.rowptr, few.col, few.val, method, k, "d2q"))
