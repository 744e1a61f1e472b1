"""The Adam extension's kernels (tsid_extend_chunk_adam) at the sizes where they
can go wrong, and how exact their two contractions are.

One step with beta1 = beta2 = 0, lambda = 0 and lr = eps = 2^60 gives C = -dL/dC to
the bit: the moments are the gradient and its square, the denominator rounds to
2^60, and the factors 2^60 cancel exactly.  From lines of one cell of value 1 the
gradient sums are -2 p, exact as well, so C holds the plain fp32 contraction
B (2 p), and B^T C the plain fp32 contraction of a C that is known to the bit."""
import numpy as np
import pytest

from gpu_util import note

pytestmark = pytest.mark.gpu

BIG = 2.0 ** 60


def _run(k, F, B, fixed, free, r, n_free, opts):
    import torch
    import paper_2608_00977_amd as tsid
    T = tsid.Tsid(0)
    try:
        d = np.arange(8, dtype=np.int32)  # a template of the rank
        T.build_template(8, 8, d, d, np.ones(8, np.float32), d, d, k)
        X = torch.empty((n_free, k), dtype=torch.float32).pin_memory()
        C = torch.empty((n_free, B.shape[0]), dtype=torch.float32).pin_memory()
        Fd, Bd = torch.from_numpy(F).cuda(), torch.from_numpy(B).cuda()
        T.extend_chunk_adam(1, fixed, free, r, n_free, Fd, Bd, X, opts, C)
        T.sync()
        return X.numpy().copy(), C.numpy().copy()
    finally:
        T.close()


def _chain(a, b):
    """fp32 chain of fused multiply-adds over the last axis, from zero."""
    acc = np.zeros(np.broadcast_shapes(a.shape, b.shape)[:-1], np.float32)
    for i in range(a.shape[-1]):
        acc = (a[..., i].astype(np.float64) * b[..., i] + acc).astype(np.float32)
    return acc


def _rms(x):
    return float(np.sqrt(np.mean(np.square(x, dtype=np.float64))))


@pytest.mark.parametrize("k", [8, 16, 32, 64, 128])
def test_contractions_are_as_exact_as_short_chains(k):
    """fp32 sums in long chains lose digits: the error of each contraction stays
    within 5% (the scatter of such a root mean square) of the same sums in chains
    of K / 4 coordinates (four, added in pairs) for the gradient, and of 16 basis
    lines (16 per slice of 256, added in turn) for B^T C."""
    from paper_2608_00977_amd import make_adam_opts
    g = np.random.default_rng(100 + k)
    n_free, n_b = 160, 1024
    F = g.normal(0, k ** -0.25, (n_free, k)).astype(np.float32)
    B = g.normal(0, k ** -0.25, (n_b, k)).astype(np.float32)
    ids = np.arange(n_free, dtype=np.int32)
    note(f"adam contraction errors k={k}")
    X, C = _run(k, F, B, ids, ids, np.ones(n_free, np.float32), n_free, make_adam_opts(1, 0.0, BIG, 0.0, 0.0, BIG))
    want = 2.0 * F.astype(np.float64) @ B.astype(np.float64).T
    parts = [_chain(2 * F[:, None, q * k // 4:(q + 1) * k // 4], B[None, :, q * k // 4:(q + 1) * k // 4])
             for q in range(4)]
    short = (parts[0] + parts[1]) + (parts[2] + parts[3])
    assert _rms(C - want) <= 1.05 * _rms(short - want), (_rms(C - want), _rms(short - want))
    want = C.astype(np.float64) @ B.astype(np.float64)
    short = np.zeros((n_free, k), np.float32)
    for s in range(n_b // 256):
        part = np.zeros((n_free, k), np.float32)
        for lane in range(16):
            at = slice(256 * s + lane, 256 * (s + 1), 16)
            part += _chain(C[:, None, at], B.T[None, :, at])
        short += part
    assert _rms(X - want) <= 1.05 * _rms(short - want), (_rms(X - want), _rms(short - want))
    note(f"gradient and B^T C errors checked at k={k}")


def _lines(k, lengths, n_fixed, n_b, seed):
    """One free line per entry of lengths, of that many cells, in line order."""
    g = np.random.default_rng(seed)
    F = g.normal(0, k ** -0.25, (n_fixed, k)).astype(np.float32)
    B = g.normal(0, k ** -0.25, (n_b, k)).astype(np.float32)
    fixed = np.concatenate([np.sort(g.choice(n_fixed, d, replace=False)) for d in lengths]).astype(np.int32)
    free = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    return F, B, fixed, free, g.standard_normal(fixed.size).astype(np.float32)


def _row_err(x, ref):
    den = np.linalg.norm(ref, axis=1)
    return np.linalg.norm(np.asarray(x, np.float64) - ref, axis=1) / np.where(den > 0, den, 1.0)


def _check_rows(k, lengths, n_fixed, n_b, steps=6):
    """X and C line by line against the oracle in the smooth regime (eps = 10):
    within ten times the oracle's own change, line by line, under 2^-23 relative
    perturbations of F and B, and at least 1e-5."""
    import oracle
    from paper_2608_00977_amd import make_adam_opts
    F, B, fixed, free, r = _lines(k, lengths, n_fixed, n_b, 7 * k + n_b)
    n_free, opt = len(lengths), (0.1, 0.05, 0.9, 0.999, 10.0)
    X, C = _run(k, F, B, fixed, free, r, n_free, make_adam_opts(steps, *opt))
    st, Xo, Co = oracle.extend_adam(fixed, free, r, n_free, F, B, steps, *opt)
    assert st == 0
    g = np.random.default_rng(3)
    Fp, Bp = [a.astype(np.float64) * (1 + 2.0 ** -23 * g.standard_normal(a.shape)) for a in (F, B)]
    _, Xp, Cp = oracle.extend_adam(fixed, free, r, n_free, Fp, Bp, steps, *opt)
    for got, want, moved in ((X, Xo, Xp), (C, Co, Cp)):
        err, bar = _row_err(got, want), np.maximum(1e-5, 10 * _row_err(moved, want))
        assert np.all(err <= bar), (err.max(), int(np.argmax(err - bar)))
    empty = np.asarray(lengths) == 0
    assert not X[empty].any() and not C[empty].any()


# lengths around an item (64 cells) and around a wave's items (4 to 32), one empty line
MIXED = [0, 1, 5, 63, 64, 65, 127, 257, 512, 1025, 3000, 2, 700, 129, 40, 4100]


@pytest.mark.parametrize("k", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("n_free,n_b", [(1, 1), (15, 3), (16, 15), (17, 17), (16, 63), (1, 65), (17, 255), (15, 257),
                                        (33, 301), (16, 520)])
def test_edges_match_oracle_line_by_line(k, n_free, n_b):
    """Basis sizes around a tile of 16, a wave's 64 and a slice of 256 lines, whole
    16-byte words and not; free lines around a workgroup's 16; lines whose items
    lie in one wave and in several."""
    note(f"adam edges k={k} n_free={n_free} n_b={n_b}")
    _check_rows(k, (MIXED * 3)[-n_free:], 4200, n_b)


@pytest.mark.parametrize("k,lines,cells,n_b", [(8, 1, 70_000, 33), (16, 2, 34_000, 260), (32, 2, 18_000, 70),
                                               (64, 3, 9000, 31), (128, 3, 9000, 300), (64, 10, 6400, 68_000),
                                               (128, 10, 6400, 34_001)])
def test_long_lines_match_oracle_line_by_line(k, lines, cells, n_b):
    """Lines whose sums a fixup launch adds: more than 32 a line, or 16 MB of reads
    over the slices of a large basis; short lines among them."""
    note(f"adam long lines k={k} {lines} x {cells} n_b={n_b}")
    _check_rows(k, [cells] * lines + ([3] if lines > 3 else []), max(cells, 6400), n_b, steps=3)
