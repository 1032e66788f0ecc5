"""Coefficients where their kernels change: few patterns (a block each), a region per wave that
does not fit (large m and ell), tables that are not the cyclic ones at ell = 1, rows of 1 to 8
coefficients.

Reference: the pseudo-inverse of every R[:, S_i] in 64 bits.  Bar: one fp32 rounding of an fp64
Cholesky solve, 2 u |ref| + 1e-14 kappa^2 max|B_i|, as for the other coefficient tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2405_19509_amd import gcx  # noqa: E402

pytestmark = pytest.mark.gpu


def tables(m, delta, kind, rng):
    if kind == "cyclic":
        return gcx.gc_assign(gcx.GC_ASSIGN_CYCLIC, m, m, delta - 1)[1:]
    A = np.zeros((m, m), dtype=np.int32)
    rows, cols = rng.permutation(m), rng.permutation(m)
    for o in rng.choice(m, delta, replace=False):
        A[rows[(np.arange(m) + o) % m], cols] = 1
    return gcx.gc_assign(gcx.GC_ASSIGN_REGULAR, m, m, O=A)[1:]


@pytest.mark.parametrize("m,delta,ell,P,kind", [
    (6, 3, 1, 1, "cyclic"), (6, 3, 2, 7, "cyclic"), (37, 7, 3, 5, "regular"), (70, 9, 8, 3, "cyclic"),  # a block each
    (200, 20, 1, 2, "cyclic"), (65, 6, 2, 256, "regular"),
    (70, 9, 2, 300, "regular"), (37, 7, 5, 400, "cyclic"), (20, 4, 4, 600, "cyclic"),  # a wave each
    (64, 8, 1, 300, "regular"), (129, 5, 1, 1000, "regular"),  # not cyclic
    (200, 20, 8, 300, "cyclic"), (137, 12, 6, 520, "regular"), (100, 10, 8, 700, "cyclic"),  # few regions fit
    (200, 20, 4, 1100, "regular"),
])
def test_coefficients(m, delta, ell, P, kind):
    rng = np.random.default_rng(m + 10 * ell + P)
    order, holder, hpos = tables(m, delta, kind, rng)
    psi = rng.integers(0, delta + 1, (P, m)).astype(np.int32)
    psi[:, rng.permutation(m)[: m // 4]] = 0
    psi[P // 2] = rng.integers(0, 2, m)  # most chunks below ell copies
    if P > 2:
        psi[P - 1, m - 1] = delta + 1  # refused, its coefficients zero
    R = rng.standard_normal((ell, m)).astype(np.float32)
    dev = [torch.from_numpy(a).cuda() for a in (psi, order, holder, hpos, R)]
    Bc = torch.full((P, m, delta, ell), float("nan"), device="cuda")
    cov, dec, cerr, _ = gcx.gc_decode_coeffs(*dev, Bc=Bc)
    mask = psi[:, holder] > hpos
    want = mask.sum(2)
    assert np.array_equal(cov.cpu().numpy(), want)
    assert np.array_equal(cerr.cpu().numpy(), np.maximum(ell - want, 0).sum(1))
    state = np.where((want >= ell).all(1), gcx.GC_DEC_YES, gcx.GC_DEC_NO)
    if P > 2:
        state[P - 1] = gcx.GC_DEC_INVALID
    assert np.array_equal(dec.cpu().numpy(), state)
    got = Bc.cpu().numpy()
    assert np.isfinite(got).all()
    for p in sorted({0, P // 2, P // 3, max(0, P - 2)}):
        for i in range(m):
            rows = got[p, holder[i], hpos[i]]  # [gamma][ell]
            on = mask[p, i]
            assert not rows[~on].any()
            if state[p] == gcx.GC_DEC_INVALID or not on.any():
                assert not rows.any()
                continue
            X = R[:, holder[i][on]].astype(np.float64)
            ref = np.linalg.pinv(X, rcond=1e-13)
            kappa = np.linalg.cond(X)
            bar = 2 * 2.0 ** -24 * np.abs(ref) + 1e-14 * kappa ** 2 * np.abs(ref).max()
            assert (np.abs(rows[on] - ref) <= bar).all(), (p, i, kappa)
    if P > 2:
        assert not got[P - 1].any()
