"""The exact extension solve at the edges of its kernel: rows of lengths
around the rounds in which the Gram matrix is accumulated (16 cells at
k = 64, 32 below), row counts that leave a workgroup of four rows partly empty,
and rows whose Gram matrix is singular up to lambda, against the oracle's
fp64 normal equations (1e-6 relative per row, a few fp32 ulps: both solve in
fp64 and round once)."""
import numpy as np
import pytest

import oracle
from gpu_util import note
from test_gpu_extend_gram import _chunk, _row_err, _run, _set_rank

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    yield t
    t.close()


@pytest.mark.parametrize("k", [8, 16, 32, 64])
@pytest.mark.parametrize("extra", [0, 1, 2, 3])
def test_round_edges_match_oracle(T, k, extra):
    lengths = [0, 1, 2, 3, 4, 5, k - 1, k, k + 1] + [c + d for c in (16, 32, 64, 96, 128) for d in (-1, 0, 1)]
    lengths += [700, 0] + [7] * ((extra - len(lengths) - 2) % 4)
    assert len(lengths) % 4 == extra
    F, fixed, free, r = _chunk(50 + k, k, 900, lengths)
    _set_rank(T, k)
    note(f"ridge edges k={k} rows={len(lengths)}")
    for lam in (0.3, 1e-3):
        X = _run(T, F, fixed, free, r, len(lengths), lam)
        Xo = oracle.ridge(fixed, free, r, len(lengths), F, float(np.float32(lam)))
        Xo = Xo[1] if isinstance(Xo, tuple) else Xo
        err = _row_err(X, Xo)
        assert err.max() <= 1e-6, (lam, err.max(), lengths[int(err.argmax())])
        assert np.all(X[np.asarray(lengths) == 0] == 0.0)


@pytest.mark.parametrize("k", [8, 32, 64])
def test_singular_row_among_regular_ones_is_reported(T, k):
    """lambda = 0: a row with half as many cells as coordinates has no minimiser."""
    import paper_2608_00977_amd as tsid
    lengths = [3 * k, 4 * k, k // 2, 5 * k, 3 * k + 1]
    F, fixed, free, r = _chunk(9, k, 6 * k, lengths)
    _set_rank(T, k)
    note(f"ridge singular k={k}")
    with pytest.raises(tsid.TsidError) as e:
        _run(T, F, fixed, free, r, len(lengths), 0.0)
    assert e.value.status == 7
    sel = free != 2
    X = _run(T, F, fixed[sel], free[sel], r[sel], len(lengths), 1e-3)
    assert np.all(np.isfinite(X)) and np.all(X[2] == 0.0)
