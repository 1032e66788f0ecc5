"""The matrix-core encode against the oracle at the edges of its plan: every count of K steps
(16 rows of chunk blocks) of both storage types, rows of T on and off 16-byte and 64-byte
boundaries, last blocks shorter than the others, fewer positions than a tile, one pattern
(groups of workers), several (fewer workers per group) and more than a window; orders whose
workers share no chunks; gradients that are not finite."""
from __future__ import annotations

import numpy as np
import pytest

import oracle.protocol as OP
import oracle_runs as R_
import test_parity_gpu as TP
from workloads import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2405_19509_amd import gcx  # noqa: E402


def problem(m, delta, d, P, g_dtype, seed=0, cyclic=True):
    rng = np.random.default_rng([seed, m, delta, d, P])
    if cyclic:
        O, order, _, _ = gcx.gc_assign(gcx.GC_ASSIGN_CYCLIC, m, m, delta - 1)
    else:
        A = np.zeros((m, m), dtype=np.int32)
        for j in range(m):
            A[rng.permutation(m)[:delta], j] = rng.permutation(delta) + 1
        O, order, _, _ = gcx.gc_assign(gcx.GC_ASSIGN_ORDER, m, m, O=A)
    G = rng.standard_normal((m, d)).astype(np.float32)
    if g_dtype == "bf16":
        G = gen.f32_to_bf16_bits(G)
    psi = rng.integers(0, delta + 1, size=(P, m)).astype(np.int32)
    psi[:, rng.permutation(m)[: m // 6]] = 0
    return O.astype(np.int64), order, G, psi


# (m, delta, ell): 1 .. 12 K steps of the smallest window; the last of each type goes past them
STEPS = [(100, 4, 1), (50, 16, 2), (34, 14, 3), (34, 14, 4), (26, 16, 5), (26, 16, 6), (26, 16, 7), (26, 16, 8),
         (26, 18, 8), (26, 20, 8), (26, 22, 8), (26, 24, 8), (28, 25, 8)]


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,delta,ell", STEPS)
def test_k_steps(m, delta, ell, g_dtype):
    # 64-byte rows; odd rows with a short last block; rows on 16 but not on 64 bytes
    for d, P in ((ell * 160, 3), (ell * 203 - 1, 7), (ell * 36, 33)):
        O, order, G, psi = problem(m, delta, d, P, g_dtype)
        TP._encode_against_oracle(O, order, psi, gen.shared_R(m, ell), G, g_dtype, ell, d)


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,delta,ell,d,P", [
    (7, 3, 2, 9, 1), (7, 3, 8, 5, 2),        # blocks of a few positions, some of them empty
    (12, 5, 1, 129, 260), (12, 5, 2, 257, 193),  # one row more than a window's
    (110, 2, 1, 131, 5), (110, 2, 1, 128, 64),   # K steps that hold more workers than a window
])
def test_windows(m, delta, ell, d, P, g_dtype):
    O, order, G, psi = problem(m, delta, d, P, g_dtype, seed=1)
    TP._encode_against_oracle(O, order, psi, gen.shared_R(m, ell), G, g_dtype, ell, d)


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P", [1, 6, 40])
@pytest.mark.parametrize("ell", [1, 3])
def test_orders_without_shared_chunks(ell, P, g_dtype):
    m, delta, d = 120, 9, 301
    O, order, G, psi = problem(m, delta, d, P, g_dtype, seed=2, cyclic=False)
    TP._encode_against_oracle(O, order, psi, gen.shared_R(m, ell), G, g_dtype, ell, d)


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_not_finite_gradients(value, g_dtype):
    """A chunk's value that is not finite enters the rows that have processed the chunk, at its
    position, and no other row."""
    m, delta, ell, d, P = 40, 12, 2, 1203, 20
    L = -(-d // ell)
    O, order, G, psi = problem(m, delta, d, P, "f32", seed=3)
    where = [(5, 17), (23, L + 44), (23, d - 1)]
    for c, x in where:
        G[c, x] = 0.0
    bits = np.float32(value).view(np.uint32)
    if g_dtype == "bf16":
        G = gen.f32_to_bf16_bits(G)
        bits = bits >> 16
    Gbad = G.copy()
    for c, x in where:
        Gbad.view(np.uint16 if g_dtype == "bf16" else np.uint32)[c, x] = bits
    wide = OP.widen(G, g_dtype)
    R = gen.shared_R(m, ell)
    Bc, _ = R_.coefficients(O, psi, R)
    Bc32 = Bc.astype(np.float32)
    Gt = TP.dev(Gbad.view(np.int16)).view(torch.bfloat16) if g_dtype == "bf16" else TP.dev(Gbad)
    T = torch.zeros((P, m, L), dtype=torch.float32, device="cuda")
    T = TP.host(gcx.gc_encode(Gt, TP.dev(psi), TP.dev(order), TP.dev(Bc32), T=T))
    ref, M, nterm = R_.encode_ref(Bc32.astype(np.float64), psi, order, wide, ell)
    bound = R_.encode_bound(nterm, M, g_dtype)
    bad = np.zeros(T.shape, dtype=bool)
    for p in range(P):
        for j in range(m):
            for c, x in where:
                if c in order[j, : psi[p, j]]:
                    bad[p, j, x % L] = True
    assert bad.any() and not np.isfinite(T[bad]).any()
    ok = ~bad & (psi > 0)[:, :, None]
    diff = np.where(ok, np.abs(np.where(ok, T, 0).astype(np.float64) - np.where(ok, ref, 0)), 0)
    assert (diff <= np.where(ok, bound, np.inf)).all()


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,delta,d,P", [(50, 3, 40001, 64), (50, 3, 200001, 2), (100, 3, 1 << 16, 64), (37, 10, 20003, 40)])
def test_rows_of_one_term(m, delta, d, P, g_dtype):
    """One product per output is as good as rounded once.  Its rounding to nearest is off by 2.5e-8 on
    the average of squares and by u = 2^-24 at most; the products left out add under 2^-25, the
    coefficient's third part under 2^-25."""
    _, order, _, _ = gcx.gc_assign(gcx.GC_ASSIGN_CYCLIC, m, m, delta - 1)
    g = torch.Generator(device="cuda").manual_seed(d)
    G = torch.randn((m, d), generator=g, device="cuda").to(torch.bfloat16 if g_dtype == "bf16" else torch.float32)
    Bc = torch.randn((P, m, delta, 1), generator=g, device="cuda")
    psi = torch.ones((P, m), dtype=torch.int32, device="cuda")
    T = gcx.gc_encode(G, psi, TP.dev(order), Bc)
    first = torch.from_numpy(order[:, 0]).long().cuda()
    ref = Bc[:, :, 0].double() * G.double()[first]
    err = (T.double() - ref).abs()
    assert float((err / ref.abs().clamp_min(1e-30)).max()) <= 2 * 2.0 ** -24
    assert float(err.norm() / ref.norm()) <= 3.0e-8


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m,delta,ell,d", [(50, 3, 1, 5001), (40, 12, 3, 6003)])
def test_coefficients_at_the_end_of_the_range(m, delta, ell, d, g_dtype):
    """Coefficients that round past the largest bf16 times small gradients give the finite sums of 64
    bits; a coefficient that is not finite makes its row's values not finite, and no other row's."""
    P = 40
    O, order, G, psi = problem(m, delta, d, P, "f32", seed=4)
    psi = np.full_like(psi, delta)
    G *= np.float32(2.0 ** -100)
    if g_dtype == "bf16":
        G = gen.f32_to_bf16_bits(G)
    rng = np.random.default_rng(5)
    Bc = rng.standard_normal((P, m, delta, ell)).astype(np.float32) * np.float32(2.0 ** 120)
    Bc[3, 7, 1, 0] = np.float32(3.4e38)
    Bc[P - 1, m - 1, delta - 1, ell - 1] = -np.finfo(np.float32).max
    Bc[5, 2, 0, 0] = np.float32(np.inf)
    Bc[6, 2, delta - 1, ell - 1] = np.array(0x7fffffff, np.uint32).view(np.float32)
    Bc[6, 3, delta - 1, 0] = np.array(0xffffffff, np.uint32).view(np.float32)
    Gt = TP.dev(G.view(np.int16)).view(torch.bfloat16) if g_dtype == "bf16" else TP.dev(G)
    T = TP.host(gcx.gc_encode(Gt, TP.dev(psi), TP.dev(order), TP.dev(Bc)))
    bad = np.zeros((P, m), dtype=bool)
    bad[5, 2] = bad[6, 2] = bad[6, 3] = True
    assert not np.isfinite(T[bad]).any() and np.isnan(T[6, 2:4]).all()
    fine = np.where(np.isfinite(Bc), Bc, 0).astype(np.float64)
    ref, M, nterm = R_.encode_ref(fine, psi, order, OP.widen(G, g_dtype).astype(np.float64), ell)
    bound = R_.encode_bound(nterm, M, g_dtype)
    assert (np.abs(T[~bad].astype(np.float64) - ref[~bad]) <= bound[~bad]).all()


@pytest.mark.parametrize("g_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("scale", [104, 118])
def test_small_magnitudes(scale, g_dtype):
    """Coefficients, and fp32 gradients, far below 1: parts in full from 2^-108 on, an absolute error of
    2^-126 per value below (magnitudes here mostly from 2^-scale * 2^-4 on)."""
    m, delta, ell, d, P = 50, 16, 2, 4095, 8
    for small_g in (False, True):
        O, order, G, psi = problem(m, delta, d, P, "f32", seed=6)
        rng = np.random.default_rng(7)
        Bc = rng.standard_normal((P, m, delta, ell)).astype(np.float32)
        if small_g:
            G *= np.float32(2.0 ** -scale)
        else:
            Bc *= np.float32(2.0 ** -scale)
        if g_dtype == "bf16":
            G = gen.f32_to_bf16_bits(G)
        Gt = TP.dev(G.view(np.int16)).view(torch.bfloat16) if g_dtype == "bf16" else TP.dev(G)
        T = TP.host(gcx.gc_encode(Gt, TP.dev(psi), TP.dev(order), TP.dev(Bc)))
        wide = OP.widen(G, g_dtype).astype(np.float64)
        ref, M, nterm = R_.encode_ref(Bc.astype(np.float64), psi, order, wide, ell)
        # what the absolute errors of the small operand make of the other one's magnitudes
        other = R_.encode_ref(np.sign(Bc).astype(np.float64) if not small_g else Bc.astype(np.float64), psi, order,
                              np.sign(wide) if small_g else wide, ell)[1]
        sent = psi > 0
        bound = R_.encode_bound(nterm, M, g_dtype) + 2.0 ** -126 * other
        assert (np.abs(T[sent].astype(np.float64) - ref[sent]) <= bound[sent]).all()
