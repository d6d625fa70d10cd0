"""bfloat16 phase-1 tables selected in registers: both list sizes, tile, pass
and row-block edges, the stage widths of the recompute, against float64."""
import numpy as np
import pytest

from oracle import emd_oracle as O
from synth.generators import CSR
import parity as P

pytestmark = pytest.mark.gpu

# query lengths: one word, a 32-word tile and a 64-word pass with their edges,
# the last length of the wide stage and the first of the narrow one, and the
# longest that the kernel takes with the one that goes elsewhere
HQ = [1, 8, 31, 32, 33, 63, 64, 65, 127, 128, 129, 192, 255, 256, 257, 300, 511, 512, 513]


@pytest.fixture(scope="module")
def L():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1812_02091_amd import lcemd

    lcemd.load_library()
    return lcemd


@pytest.mark.parametrize("m", [3, 58, 59, 122, 300])
@pytest.mark.parametrize("k", [1, 8, 9, 24])
def test_tables(L, m, k):
    """S/Z/W of every used word: a block of 256 rows, a part one, odd and even
    numbers of 64-dim slices; the longest query of a batch decides the layout,
    so the queries run one by one and together."""
    rng = np.random.default_rng(45)
    v = 700
    V = (rng.standard_normal((v, m)) * rng.choice([0.3, 1.0, 3.0], (v, 1))).astype(np.float32)
    words = np.arange(256 + 37, dtype=np.int32)
    ctx = L.open_context(V, np.array([0, words.size], dtype=np.int64), words,
                         np.full(words.size, 1.0 / words.size, np.float32))
    ptr = np.concatenate([[0], np.cumsum(HQ)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.choice(v, n, replace=False)) for n in HQ]).astype(np.int32)
    val = np.concatenate([w / w.sum() for w in (1.0 - rng.random(n) for n in HQ)]).astype(np.float32)
    q = CSR(ptr, col, val)
    print(f"[gpu] bf16 tables m={m} k={k}", flush=True)
    S, Z, W = ctx.tables(q.rowptr, q.col, q.val, k, precision="bf16")
    for b in range(q.n):
        qc, qw = q.row(b)
        R = O.squared_distances(V[words], V[qc])
        So = np.argsort(R, axis=1, kind="stable")[:, : min(k, qc.size)]
        P.check_table_rows(S[b], Z[b], W[b], So, R, qw, k, qc.size)
        one = ctx.tables(np.array([0, qc.size], dtype=np.int64), qc, qw, k, precision="bf16")
        P.check_table_rows(one[0][0], one[1][0], one[2][0], So, R, qw, k, qc.size)
    ctx.close()
