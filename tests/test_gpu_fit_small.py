"""Fits that run as one workgroup (k_fit_small): small fp32 templates under the
automatic modes.  Against the oracle with the bars of the other fp32 fits
(factors 1e-4, loss trajectory 1e-3, final loss 1e-6), on ranks 8 to 64, with empty
rows and columns, more owner rows than the workgroup takes at a time, the step
options and clips; against the item pass of the same template (1e-5: fp32 sums
in another order, 20 contractive epochs); repeatability, 5 + 5 epochs = 10, the
history without and with a non-finite stop; the same bits with timing on and
for any number of epochs."""
import numpy as np
import pytest

import oracle
import tsid_synth as synth
from gpu_util import gpu_fit, note, oracle_template, rel_fro

pytestmark = pytest.mark.gpu

# (m, n, nnz, m_t, n_t, k): factors and streams within 150 KB, short buckets
CASES = [(300, 260, 3500, 200, 160, 8), (3000, 2400, 4000, 1000, 900, 8), (260, 240, 2000, 240, 200, 16),
         (150, 140, 900, 130, 120, 32), (120, 100, 500, 90, 80, 64), (90, 80, 250, 60, 50, 64),
         (64, 64, 300, 1, 40, 16), (64, 64, 300, 40, 1, 32), (50, 40, 12, 30, 20, 64)]


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    yield t
    t.close()


def _case(c):
    m, n, nnz, m_t, n_t, k = c
    return synth.random_case(m, n, nnz, m_t, n_t, k, seed=m + k)


def _build(T, p):
    T.build_template(p.m, p.n, p.u, p.i, p.r, p.I, p.J, p.k)


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("step,clip", [("degree", False), ("degree", True), ("col_degree", "printed"), ("sum", False)])
def test_small_fit_matches_oracle(T, case, step, clip):
    p = _case(case)
    p.xi = 0.05
    lr = 0.02 if step == "degree" else 0.002  # contractive for rows of a single cell
    note(f"small fit {case} {step} clip={clip}")
    _build(T, p)
    st, P, Q, hist = gpu_fit(T, p, epochs=20, lr=lr, step=step, clip=clip, prec="fp32")
    assert st == 0 and T.epochs_done() == 20 and T.pass_kernels() == ("small", "small")
    _, _, a, b, v = oracle_template(p)
    so, Po, Qo, ho, _ = oracle.fit(a, b, v, p.P0, p.Q0, 20, p.lam, lr, step, clip, p.xi)
    assert so == 0
    assert rel_fro(P, Po) <= 1e-4 and rel_fro(Q, Qo) <= 1e-4
    np.testing.assert_allclose(hist, ho, rtol=1e-3)
    want = oracle.loss(a, b, v, P.shape[0], Q.shape[0], P, Q, p.lam)
    assert abs(hist[-1] - want) <= 1e-6 * abs(want)
    T.set_pass_kernel("item")
    try:
        _, Pi, Qi, hi = gpu_fit(T, p, epochs=20, lr=lr, step=step, clip=clip, prec="fp32")
        assert "small" not in T.pass_kernels()
    finally:
        T.set_pass_kernel("auto")
    assert rel_fro(P, Pi) <= 1e-5 and rel_fro(Q, Qi) <= 1e-5
    np.testing.assert_allclose(hist, hi, rtol=1e-5)


def test_repeats_and_resumes_bitwise(T):
    p = _case(CASES[0])
    _build(T, p)
    _, P, Q, h = gpu_fit(T, p, epochs=10, lr=0.1, step="degree", prec="fp32")
    _, P2, Q2, h2 = gpu_fit(T, p, epochs=10, lr=0.1, step="degree", prec="fp32")
    np.testing.assert_array_equal(P, P2)
    np.testing.assert_array_equal(Q, Q2)
    np.testing.assert_array_equal(h, h2)
    _, P5, Q5, h5 = gpu_fit(T, p, epochs=5, lr=0.1, step="degree", prec="fp32")
    _, P6, Q6, h6 = gpu_fit(T, p, epochs=5, lr=0.1, step="degree", prec="fp32", P0=P5, Q0=Q5)
    np.testing.assert_array_equal(P, P6)
    np.testing.assert_array_equal(Q, Q6)
    np.testing.assert_array_equal(h, np.concatenate([h5[:5], h6]))
    assert T.pass_kernels() == ("small", "small")


def test_nonfinite_stop_returns_the_last_finite_iterate(T):
    p = _case(CASES[2])
    _build(T, p)
    note("small fit non-finite stop")
    st, P, Q, hist = gpu_fit(T, p, epochs=60, lr=1e6, step="sum", clip=False, prec="fp32")
    done = T.epochs_done()
    assert st == 7 and 0 < done < 60 and T.pass_kernels() == ("small", "small")
    assert np.all(np.isfinite(P)) and np.all(np.isfinite(Q)) and np.all(np.isnan(hist[done + 1:]))
    T.set_pass_kernel("item")
    try:
        st, Pi, Qi, _ = gpu_fit(T, p, epochs=60, lr=1e6, step="sum", clip=False, prec="fp32")
        assert st == 7 and T.epochs_done() == done
    finally:
        T.set_pass_kernel("auto")
    st, P2, Q2, h2 = gpu_fit(T, p, epochs=done, lr=1e6, step="sum", clip=False, prec="fp32")
    assert st == 0
    np.testing.assert_array_equal(P, P2)
    np.testing.assert_array_equal(hist[:done + 1], h2)


def test_timing_and_epoch_count_leave_the_bits_alone(T):
    """Timing a fit, no epochs at all and more epochs than one launch takes give
    the same bits; the timer sees the launches and every epoch."""
    p = _case(CASES[0])
    _build(T, p)
    note("small fit timing")
    want = gpu_fit(T, p, epochs=12, lr=0.1, step="degree", prec="fp32")
    T.set_timing(5)
    try:
        got = gpu_fit(T, p, epochs=12, lr=0.1, step="degree", prec="fp32")
        tm = T.timing()
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
        assert T.pass_kernels() == ("small", "small")
        assert tm["pass_launches"] == [1, 0] and tm["epochs"] == 12
        assert tm["epoch_ms"] == tm["pass_ms"][0] > 0 and tm["fixup_launches"] == tm["reduce_launches"] == 0
    finally:
        T.set_timing(0)
    st, P, Q, hist = gpu_fit(T, p, epochs=0, lr=0.1, step="degree", prec="fp32")
    assert st == 0 and hist[0] == want[3][0]
    np.testing.assert_array_equal(P, p.P0)
    np.testing.assert_array_equal(Q, p.Q0)
    note("small fit in more than one launch")
    n = 66_000
    P0, Q0 = p.P0, p.Q0
    st, P, Q, hist = gpu_fit(T, p, epochs=n, lr=0.01, step="degree", prec="fp32")
    assert st == 0 and T.epochs_done() == n and T.pass_kernels() == ("small", "small")
    parts = []
    for _ in range(2):
        st, P0, Q0, h = gpu_fit(T, p, epochs=n // 2, lr=0.01, step="degree", prec="fp32", P0=P0, Q0=Q0)
        parts.append(h)
    np.testing.assert_array_equal(P, P0)
    np.testing.assert_array_equal(Q, Q0)
    np.testing.assert_array_equal(hist, np.concatenate([parts[0][:-1], parts[1]]))


def test_small_is_reported_and_not_a_mode(T):
    from paper_2608_00977_amd.binding import E_INVAL, tsid_set_pass_kernel
    assert tsid_set_pass_kernel(T.ctx, 3) == E_INVAL
    with pytest.raises(KeyError):
        T.set_pass_kernel("small")
