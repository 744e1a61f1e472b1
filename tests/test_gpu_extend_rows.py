"""The per-cell extension steps (Section 5.2; k_extend_steps and
k_extend_group) at the edges of what one wave and each workgroup form hold:
rows of no cells, one cell, and one below, at and one above every capacity,
against the oracle's one-sided steps of the same cells (1e-4 relative per row,
the fp32 bar of the extension: 20 steps of sums of a few thousand terms, a
few 1e-7 each).  The Gram form is off, so every row takes the per-cell form.
A second run in chunks gives the same bits: a row's form depends on its own
length alone.  Forms that no row can take are not launched.  With few steps longer
rows are streamed, by one wave each where they are many, with the same bits."""
import numpy as np
import pytest

import oracle
from gpu_util import note
from test_gpu_extend_gram import _chunk, _gram_env, _row_err, _run, _set_rank

pytestmark = pytest.mark.gpu

# cells that one wave holds, and workgroups of 2, 4 and 8 waves: lane groups of
# k / 4 (k < 64) or k / 8 lanes, 16 cells each in the one-wave form, 24 in the others
GROUPS = {8: 32, 16: 16, 32: 8, 64: 8, 128: 4}
CAPS = {k: [16 * g, 48 * g, 96 * g, 192 * g] for k, g in GROUPS.items()}


@pytest.fixture(scope="module")
def T():
    import paper_2608_00977_amd as tsid
    t = tsid.Tsid(0)
    yield t
    t.close()


@pytest.mark.parametrize("k", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("step,clip", [("degree", "printed"), ("sum", True)])
def test_rows_at_capacity_edges_match_oracle(T, k, step, clip):
    from paper_2608_00977_amd import make_opts
    caps = CAPS[k]
    lengths = [0, 1, 2, GROUPS[k] - 1, GROUPS[k] + 1]
    lengths += [c + d for c in caps for d in (-1, 0, 1)] + [0, caps[3] + 77, 2 * caps[1] + 3]
    n_fixed = caps[3] + 500
    F, fixed, free, r = _chunk(7 + k, k, n_fixed, lengths)
    _set_rank(T, k)
    lr = 0.05 if step == "degree" else 0.2 / max(lengths)
    opts = make_opts(epochs=20, lam=0.05, lr=lr, step=step, clip=clip, xi=0.05)
    note(f"extend rows k={k} {step} clip={clip} capacities={caps}")
    with _gram_env(-1):
        X = _run(T, F, fixed, free, r, len(lengths), opts)
        st, Xo = oracle.extend(fixed, free, r, len(lengths), F, 20, 0.05, lr, step, clip, 0.05)
        assert st == 0
        err = _row_err(X, Xo)
        assert err.max() <= 1e-4, (err.max(), lengths[int(err.argmax())])
        assert np.all(X[np.asarray(lengths) == 0] == 0.0)
        half = len(lengths) // 2
        parts = []
        for lo, hi in ((0, half), (half, len(lengths))):
            sel = (free >= lo) & (free < hi)
            parts.append(_run(T, F, fixed[sel], free[sel] - lo, r[sel], hi - lo, opts))
        np.testing.assert_array_equal(X, np.concatenate(parts))


@pytest.mark.parametrize("k", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("steps", [0, 1, 2, 3, 5, 7, 8])
def test_few_steps_match_oracle(T, k, steps):
    """With few steps rows beyond one wave are streamed, up to a step count that
    depends on the rank, the form and whether the table (the same rows, or more
    that no cell names) lies within 4 MiB."""
    from paper_2608_00977_amd import make_opts
    caps = CAPS[k]
    lengths = [0, 1, caps[0], caps[0] + 1, caps[0] + 40, caps[1], caps[1] + 1, caps[2] + 1, caps[3], caps[3] + 130]
    F, fixed, free, r = _chunk(9 + k, k, caps[3] + 500, lengths)
    _set_rank(T, k)
    opts = make_opts(epochs=steps, lam=0.05, lr=0.05, step="degree", clip=True, xi=0.05)
    st, Xo = oracle.extend(fixed, free, r, len(lengths), F, steps, 0.05, 0.05, "degree", True, 0.05)
    assert st == 0
    beyond = np.concatenate([F, np.zeros(((4 << 20) // (4 * k) + 1, k), np.float32)])
    for table in (F, beyond):
        note(f"extend rows, few steps k={k} steps={steps} table rows={table.shape[0]}")
        with _gram_env(-1):
            X = _run(T, table, fixed, free, r, len(lengths), opts)
        err = _row_err(X, Xo)
        assert err.max() <= 1e-4, (err.max(), lengths[int(err.argmax())])


@pytest.mark.parametrize("k", [8, 32, 64, 128])
@pytest.mark.parametrize("rows,in_l2", [(1700, False), (6300, True)])
def test_many_streamed_rows_have_the_bits_of_few(T, k, rows, in_l2):
    """Beyond a row count (1,024, or 6,144 with the table within 4 MiB) each streamed
    row goes to one wave, except those of more than a 1,024th of the chunk: the same
    bits as chunks of few rows, where a workgroup takes every one of them."""
    from paper_2608_00977_amd import make_opts
    g = np.random.default_rng(k)
    lengths = CAPS[k][0] + 1 + g.integers(0, 70, rows)
    lengths[[3, 900]] = CAPS[k][0] * 8 * (rows // 1000)
    n_fixed = lengths.max() + 100
    F = (g.standard_normal((n_fixed, k)) * k ** -0.5).astype(np.float32)
    fixed = np.concatenate([np.sort(g.choice(n_fixed, n, replace=False)) for n in lengths]).astype(np.int32)
    free = np.repeat(np.arange(lengths.size), lengths).astype(np.int32)
    r = g.standard_normal(fixed.size).astype(np.float32)
    assert lengths.max() > fixed.size // 1024 > np.sort(lengths)[-3]
    assert F.nbytes <= 4 << 20
    table = F if in_l2 else np.concatenate([F, np.zeros(((4 << 20) // (4 * k) + 1, k), np.float32)])
    _set_rank(T, k)
    opts = make_opts(epochs=1, lam=0.05, lr=0.05, step="degree")
    note(f"many streamed rows k={k} rows={rows} cells={fixed.size}")
    with _gram_env(-1):
        X = _run(T, table, fixed, free, r, lengths.size, opts)
        at = np.concatenate([[0], np.cumsum(lengths)])
        for lo in range(0, lengths.size, 900):
            hi = min(lengths.size, lo + 900)
            s = slice(at[lo], at[hi])
            part = _run(T, table, fixed[s], free[s] - lo, r[s], hi - lo, opts)
            np.testing.assert_array_equal(X[lo:hi], part)
    st, Xo = oracle.extend(fixed, free, r, lengths.size, F, 1, 0.05, 0.05, "degree", False, 0.05)
    assert st == 0 and _row_err(X, Xo).max() <= 1e-4


def test_nonfinite_step_is_reported_from_every_form(T):
    """A step size that overflows: E_NONFINITE at sync whichever form the row takes."""
    import paper_2608_00977_amd as tsid
    k = 32
    _set_rank(T, k)
    for n in [3] + [c for c in CAPS[k]] + [CAPS[k][3] + 1]:
        F, fixed, free, r = _chunk(n, k, n + 10, [n])
        note(f"extend rows non-finite n={n}")
        with _gram_env(-1), pytest.raises(tsid.TsidError) as e:
            _run(T, F, fixed, free, r, 1, tsid.make_opts(epochs=30, lam=0.0, lr=1e30, step="sum"))
        assert e.value.status == 7


def _kernels(run):
    """Names of the kernels that run() launches, from the runtime's trace."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        run()
        torch.cuda.synchronize()
    return [e.name for e in p.events()]


@pytest.mark.parametrize("k", [8, 32, 64])
def test_forms_without_a_row_are_not_launched(T, k):
    """Rows at or above the Gram threshold leave the per-cell forms: the list
    kernel and a workgroup form are launched only where the threshold (or the
    chunk) leaves room for a row beyond the form before it, and the results do not
    depend on that."""
    from paper_2608_00977_amd import make_opts
    caps = CAPS[k]
    lengths = [caps[3] + 200, 30, caps[2], caps[3] + 3]
    F, fixed, free, r = _chunk(5 + k, k, caps[3] + 500, lengths)
    _set_rank(T, k)
    opts = make_opts(epochs=20, lam=0.05, lr=0.05, step="degree")
    st, Xo = oracle.extend(fixed, free, r, len(lengths), F, 20, 0.05, 0.05, "degree", False, 0.05)
    assert st == 0
    for threshold, forms in ((16, 0), (caps[0], 0), (caps[0] + 1, 0), (caps[0] + 2, 1), (caps[1] + 1, 1),
                             (caps[1] + 2, 2), (caps[2] + 2, 3), (caps[3] + 1, 3), (caps[3] + 2, 4), (-1, 4)):
        note(f"extend launches k={k} threshold {threshold}")
        with _gram_env(threshold):
            out = []
            names = _kernels(lambda: out.append(_run(T, F, fixed, free, r, len(lengths), opts)))
        if not any("k_extend_steps" in n for n in names):
            pytest.skip("no kernel trace on this machine")
        assert sum("k_extend_lists" in n for n in names) == (forms > 0)
        assert sum("k_extend_group" in n for n in names) == forms
        assert _row_err(out[0], Xo).max() <= 1e-4


def test_rank_changes_do_not_grow_the_buffers():
    """A context that goes back and forth between ranks keeps buffers of the
    largest chunk's size: 60 changes fit a cap of 64 MiB."""
    import paper_2608_00977_amd as tsid
    T = tsid.Tsid(0, max_device_bytes=64 << 20)
    try:
        note("extend rank changes")
        for turn in range(60):
            k = (8, 32)[turn % 2]
            F, fixed, free, r = _chunk(turn, k, 300, [5, 40, 0, 200])
            _set_rank(T, k)
            X = _run(T, F, fixed, free, r, 4, tsid.make_opts(epochs=2, lam=0.1, lr=0.05, step="degree"))
            assert np.all(np.isfinite(X)) and not X[2].any()
    finally:
        T.close()
