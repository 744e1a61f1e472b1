"""How exact the two contractions of the Adam extension (tsid_extend_chunk_adam) are.

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
