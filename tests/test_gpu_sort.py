"""The library's radix sort (index build, extension chunks) at the edges of its
tiles (4,096 elements): templates whose cell counts fill one tile, several, and
one element more or less, with few and many distinct digits, in random,
ascending and descending order.  Every index array is bit-exact against numpy's
stable sorts; extension chunks in any order give the same bits (integers and copies:
no tolerance)."""
import numpy as np
import pytest

from gpu_util import note
from test_gpu_extend_gram import _run, _set_rank

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    yield t
    t.close()


@pytest.mark.parametrize("nnz", [1, 2, 63, 64, 65, 4095, 4096, 4097, 8192, 12289, 300_001])
@pytest.mark.parametrize("shape,order", [((3, 200_003), "random"), ((70_000, 300), "random"), ((900, 1100), "down"),
                                         ((900, 1100), "up")])
def test_index_is_bit_exact(T, nnz, shape, order):
    m, n = shape
    g = np.random.default_rng(nnz)
    cells = g.choice(m * n, min(nnz, m * n // 2), replace=False)
    cells = {"random": cells, "up": np.sort(cells), "down": np.sort(cells)[::-1]}[order]
    u, i = (cells // n).astype(np.int32), (cells % n).astype(np.int32)
    r = g.standard_normal(cells.size).astype(np.float32)
    note(f"sort build nnz={cells.size} {shape} {order}")
    T.build_template(m, n, u, i, r, np.arange(m), np.arange(n), 8)
    csr, csc = np.lexsort((i, u)), np.lexsort((u, i))
    for name, want in (("csr_col", i[csr]), ("csr_val", r[csr]), ("csc_row", u[csc]), ("csc_val", r[csc]),
                       ("row_ptr", np.concatenate([[0], np.cumsum(np.bincount(u, minlength=m))])),
                       ("col_ptr", np.concatenate([[0], np.cumsum(np.bincount(i, minlength=n))]))):
        np.testing.assert_array_equal(T.export_index(name), want, err_msg=name)


@pytest.mark.parametrize("nnz", [1, 2, 4096, 4097, 50_000])
@pytest.mark.parametrize("n_fixed,n_free", [(300, 200), (70_000, 5), (40, 300_000)])
def test_chunk_order_does_not_matter(T, nnz, n_fixed, n_free):
    """The same cells in line order, reversed and shuffled, chunk after chunk
    (the order flag of one chunk must not reach the next), and a repeated cell
    far apart is still found."""
    import paper_2608_00977_amd as tsid
    g = np.random.default_rng(nnz + n_free)
    cells = np.sort(g.choice(n_fixed * n_free, min(nnz, n_fixed * n_free // 3), replace=False))
    free, fixed = (cells // n_fixed).astype(np.int32), (cells % n_fixed).astype(np.int32)
    r = g.standard_normal(cells.size).astype(np.float32)
    F = (g.standard_normal((n_fixed, 8)) * 0.35).astype(np.float32)
    _set_rank(T, 8)
    opts = tsid.make_opts(epochs=3, lam=0.01, lr=0.05, step="degree")
    note(f"sort chunk nnz={cells.size} fixed={n_fixed} free={n_free}")
    want = None
    for perm in (g.permutation(cells.size), np.arange(cells.size), np.arange(cells.size)[::-1], g.permutation(cells.size),
                 np.arange(cells.size)):
        X = _run(T, F, fixed[perm], free[perm], r[perm], n_free, opts)
        want = X if want is None else want
        np.testing.assert_array_equal(X, want)
    if cells.size > 2:
        a, b = np.append(fixed, fixed[0]), np.append(free, free[0])
        with pytest.raises(tsid.TsidError) as e:
            _run(T, F, a, b, np.append(r, r[0]), n_free, opts)
        assert e.value.status == 3
