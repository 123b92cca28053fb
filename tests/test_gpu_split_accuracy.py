"""Row sums split by entries: a row of 65 to 256 entries among short ones is
summed no less accurately than a wavefront would."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2312_14832_amd import gen
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,unit", [("fp64", 2.0 ** -53), ("mixed", 2.0 ** -24)])
@pytest.mark.parametrize("n,length", [(2000, 65), (2000, 130), (2000, 255), (24000, 255)])   # the last: full-sized blocks
def test_long_row_among_short_ones(lpmod, precision, unit, n, length):
    """One large product and many small ones whose chunk sums are each below
    half a unit of the total: adding the chunks one by one loses them all."""
    say(f"case split accuracy {precision} {n} {length}")
    rng = np.random.default_rng(length)
    m = n
    counts = np.where(np.arange(m) % 10 == 3, length, 3)
    rows = np.repeat(np.arange(m), counts)
    cols = np.concatenate([np.sort((rng.integers(n) + 7 * np.arange(k)) % n) for k in counts])
    K = sp.csr_matrix((rng.choice([-1.0, 1.0], rows.size) * rng.uniform(0.5, 2.0, rows.size), (rows, cols)), (m, n))
    data = gen.LPData(m, n, m // 2, K.indptr.astype(np.int32), K.indices.astype(np.int32), K.data,
                      np.ones(n), np.ones(m), np.zeros(n), np.full(n, 10.0))
    p = lpmod.Problem(data, precision=precision, split_sums=1, persistent=0)
    assert p.layout() == (1, 1) and p.layout_split(0) == 1
    Dr, Dc = p.scaling()
    Ks = sp.csr_matrix(K.multiply(1 / Dr[:, None]).multiply(1 / Dc[None, :]))
    for r in range(3, m, m // 5):
        a, b = K.indptr[r], K.indptr[r + 1]
        # the products of row r: the last 1 / unit, the others 0.11 (0.88 a chunk of 8)
        want = np.full(length, 0.11)
        want[-1] = 1 / unit
        x = np.zeros(n)
        x[K.indices[a:b]] = want / Ks.data[Ks.indptr[r]:Ks.indptr[r + 1]]
        if precision == "mixed":
            x = x.astype(np.float32).astype(np.float64)
        got = p.spmv(x)[r]
        # roundings: of K~ and of each product, 7 in the walk of the large
        # product's own chunk and one of the result, all of the size of the
        # total; the scaled value is within 4 units of FP64 of the library's
        exact = float(np.dot(Ks.data[Ks.indptr[r]:Ks.indptr[r + 1]].astype(np.longdouble), x[K.indices[a:b]]))
        terms = 1 + 1 + 7 + 1 + (4 if precision == "fp64" else 0)
        assert abs(got - exact) <= terms * unit * np.abs(want).sum(), (r, got - exact)
