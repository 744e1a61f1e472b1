"""Mini-batch steps and simultaneous epochs send both sides' passes, and both
sides' fixups, in one launch each: bitwise the results of the launches one by
one (which a timed first batch still makes), on every rank and precision, with
split buckets on both sides, on one side and on none, and with batches that
hold no cell of a line."""
import numpy as np
import pytest

import oracle
import tsid_synth as synth
from gpu_util import gpu_fit, note, oracle_template, rel_fro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    yield t
    t.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("k,hot_rows,hot_cols", [(8, 2, 2), (16, 0, 2), (32, 3, 0), (64, 0, 0), (128, 1, 1)])
def test_pairs_match_single_launches(T, k, hot_rows, hot_cols, prec):
    p = synth.random_case(500, 400, 6000, 220, 180, k, seed=k, hot_rows=hot_rows, hot_cols=hot_cols)
    note(f"pair launches k={k} hot {hot_rows} {hot_cols} {prec}")
    T.build_template(p.m, p.n, p.u, p.i, p.r, p.I, p.J, p.k)
    got = []
    try:
        for timing in (0, 1):
            T.set_minibatch(1, 3)  # one batch: every step's launches are timed, or none
            T.set_timing(timing)
            got.append(gpu_fit(T, p, epochs=4, lr=0.05, step="degree", prec=prec))
    finally:
        T.set_timing(0)
        T.set_minibatch(0, 0)
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    if prec == "fp32":  # the full-gradient epochs, paired passes and fixups
        T.set_pass_kernel("item")
        try:
            st, P, Q, hist = gpu_fit(T, p, epochs=4, lr=0.05, step="degree", prec=prec)
        finally:
            T.set_pass_kernel("auto")
        _, _, a, b, v = oracle_template(p)
        _, Po, Qo, ho, _ = oracle.fit(a, b, v, p.P0, p.Q0, 4, p.lam, 0.05, "degree", False, p.xi)
        assert st == 0 and rel_fro(P, Po) <= 1e-4 and rel_fro(Q, Qo) <= 1e-4
        np.testing.assert_allclose(hist, ho, rtol=1e-3)
