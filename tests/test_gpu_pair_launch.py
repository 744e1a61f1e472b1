"""Mini-batch steps and simultaneous epochs send both sides' passes, and both
sides' fixups, in one launch each: bitwise the results of the launches one by
one, on every rank and precision, with buckets split over several waves on both
sides, on one side and on none.

A timed single-batch fit makes its launches one by one (the timer counts them).
It stands for the others: with lambda = 0 its step is the full-gradient epoch (a
line without a cell keeps its row either way), and a mini-batch epoch is one such
step after another, each on the template of that batch's cells alone."""
import numpy as np
import pytest

import oracle
import tsid_synth as synth
from gpu_util import gpu_fit, note, oracle_template, rel_fro

pytestmark = pytest.mark.gpu

SEED = 3
# cells of a bucket beyond one wave: the wave's lane groups (64 / (k / V)) take up to 128 each
WAVE = {"fp32": {8: 4096, 16: 2048, 32: 1024, 64: 512, 128: 512},
        "bf16": {8: 8192, 16: 4096, 32: 2048, 64: 1024, 128: 1024}}


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    t.set_pass_kernel("item")
    t.set_dense_tiles(0)
    yield t
    t.close()


def _case(k, hot_rows, hot_cols, size):
    p = synth.random_case(size, size, 3 * size, size, size, k, seed=k, hot_rows=hot_rows, hot_cols=hot_cols)
    p.lam = 0.0
    return p


def _build(T, p, sel=slice(None)):
    T.build_template(p.m, p.n, p.u[sel], p.i[sel], p.r[sel], p.I, p.J, p.k)


def _one_by_one(T, p, prec, epochs, P0=None, Q0=None):
    """Single-batch epochs, every launch by itself; fixups launched per epoch."""
    T.set_minibatch(1, SEED)
    T.set_timing(1)
    try:
        got = gpu_fit(T, p, epochs=epochs, lr=0.05, step="degree", prec=prec, P0=P0, Q0=Q0)
        tm = T.timing()
    finally:
        T.set_timing(0)
        T.set_minibatch(0, 0)
    assert got[0] == 0 and tm["pass_launches"] == [epochs, epochs]
    return got[1], got[2], tm["fixup_launches"] / epochs


def _same(a, b):
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


CASES = [(8, 2, 2), (16, 0, 2), (32, 3, 0), (64, 0, 0), (64, 1, 1), (128, 1, 1)]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("k,hot_rows,hot_cols", CASES)
def test_pairs_match_single_launches(T, k, hot_rows, hot_cols, prec):
    p = _case(k, hot_rows, hot_cols, WAVE[prec][k] + 300)
    note(f"pair launches k={k} hot {hot_rows} {hot_cols} {prec}")
    _build(T, p)
    P, Q, fixups = _one_by_one(T, p, prec, 4)
    assert fixups == (hot_rows > 0) + (hot_cols > 0)
    T.set_minibatch(1, SEED)
    try:
        st, *got = gpu_fit(T, p, epochs=4, lr=0.05, step="degree", prec=prec)
    finally:
        T.set_minibatch(0, 0)
    assert st == 0
    _same(got, (P, Q))
    st, *full = gpu_fit(T, p, epochs=4, lr=0.05, step="degree", prec=prec)  # full-gradient epochs
    assert st == 0
    _same(full, (P, Q))
    np.testing.assert_array_equal(full[2], got[2])
    if prec == "fp32":
        _, _, a, b, v = oracle_template(p)
        _, Po, Qo, ho, _ = oracle.fit(a, b, v, p.P0, p.Q0, 4, p.lam, 0.05, "degree", False, p.xi)
        assert rel_fro(P, Po) <= 1e-4 and rel_fro(Q, Qo) <= 1e-4
        np.testing.assert_allclose(got[2], ho, rtol=1e-3)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("k,hot_rows,hot_cols", CASES)
def test_batches_match_single_launches(T, k, hot_rows, hot_cols, prec):
    """Two epochs of three batches against six single-batch steps, each on the
    template that holds that batch's cells alone: lines without a cell in a batch,
    and hot lines that span waves within a batch."""
    p = _case(k, hot_rows, hot_cols, 3 * WAVE[prec][k] + 900)
    note(f"pair launches of 3 batches k={k} hot {hot_rows} {hot_cols} {prec}")
    _build(T, p)
    T.set_minibatch(3, SEED)
    try:
        st, *got = gpu_fit(T, p, epochs=2, lr=0.05, step="degree", prec=prec)
    finally:
        T.set_minibatch(0, 0)
    assert st == 0
    place = []  # template positions of the cells' rows and columns
    for ids, x, size in ((p.I, p.u, p.m), (p.J, p.i, p.n)):
        at = np.full(size, -1, np.int64)
        at[ids] = np.arange(ids.size)
        place.append(at[x])
    batch = oracle.batch_of_many(place[0].astype(np.int32), place[1].astype(np.int32), SEED, 3)
    P, Q = p.P0, p.Q0
    for step in range(6):
        _build(T, p, batch == step % 3)
        P, Q, fixups = _one_by_one(T, p, prec, 1, P, Q)
        assert fixups == (hot_rows > 0) + (hot_cols > 0)
    _same(got, (P, Q))
