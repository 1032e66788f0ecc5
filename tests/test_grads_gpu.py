"""Chunk gradients where their paths change: column counts that no vector width divides, few and
many rows and points, tile edges, unaligned rows, infinities and NaN.

Reference: the same products in 64 bits.  Bar: relative 2-norm per chunk 1e-6 (measured errors are 0.5
to 5e-7; a product of bf16 parts left out gives 1.4e-6 and more, test_grads_parts.py)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2405_19509_amd import gcx  # noqa: E402

pytestmark = pytest.mark.gpu
BAR = 1e-6


def problem(N, n, d, b, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn((N, n, d), generator=g, device="cuda") * d ** -0.5
    y = (torch.rand((N, n), generator=g, device="cuda") < 0.5).float()
    W = torch.randn((b, d), generator=g, device="cuda")
    return X, y, W[0].contiguous() if b == 1 else W


def reference(X, y, W, loss):
    Wd = W.double().view(-1, X.shape[2])
    G = torch.empty((Wd.shape[0], X.shape[0], X.shape[2]), dtype=torch.float64, device="cuda")
    for i in range(X.shape[0]):
        x = X[i].double()
        z = x @ Wd.t()
        r = (z if loss == gcx.GC_LOSS_LINEAR else torch.sigmoid(z)) - y[i].double()[:, None]
        G[:, i] = r.t().contiguous() @ x
    return G


def check(G, ref):
    G = G.double().view(ref.shape)
    err = (G - ref).norm(dim=-1) / ref.norm(dim=-1).clamp_min(1e-30)
    assert float(err.max()) <= BAR


@pytest.mark.parametrize("N,n,d,b", [
    # streaming: the last one to three columns, fewer than four, one and four rows per wave, split
    # and whole rows per block, more rows than one stage of residuals
    (1, 1, 1, 1), (2, 3, 3, 1), (3, 37, 1001, 1), (2, 9, 1023, 1), (5, 70, 16387, 1), (40, 20, 40002, 1),
    (1, 2100, 1030, 1), (3, 50, 5003, 3),
    # matrix cores: rows, columns and points just past and just short of their tiles of 32, 128,
    # 64, 256, one and several splits of the columns, one to four point tiles per block
    (4, 64, 4096, 4), (3, 33, 8191, 31), (2, 130, 16385, 33), (7, 17, 20001, 64), (1, 128, 32771, 65),
    (5, 100, 2049, 97), (2, 31, 33000, 129), (30, 300, 70, 60), (60, 15, 33, 256), (1, 7, 200003, 5),
    # enough work for the matrix cores where one point at a time takes the smaller calls above
    (20, 33, 8191, 31), (240, 15, 33, 256), (24, 7, 200003, 5),
])
@pytest.mark.parametrize("loss", [gcx.GC_LOSS_LINEAR, gcx.GC_LOSS_LOGISTIC])
def test_shapes(N, n, d, b, loss):
    X, y, W = problem(N, n, d, b)
    G = torch.full((N, d) if b == 1 else (b, N, d), float("nan"), device="cuda")
    gcx.gc_chunk_grads(X, y, W, loss, G=G)
    check(G, reference(X, y, W, loss))


@pytest.mark.parametrize("N,n,d,b", [(3, 50, 40001, 1), (3, 50, 8190, 20)])
def test_rows_on_any_float(N, n, d, b):
    """Every array one float past a 16-byte boundary."""
    X, y, W = problem(N, n, d, b)

    def shifted(t):
        s = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
        return s.copy_(t)

    G = shifted(torch.full((N, d) if b == 1 else (b, N, d), float("nan"), device="cuda"))
    need = gcx.gc_chunk_grads_workspace_size(N, n, d, b)
    ws = torch.empty(need + 4, dtype=torch.uint8, device="cuda")[4:]
    gcx.gc_chunk_grads(shifted(X), shifted(y), shifted(W), gcx.GC_LOSS_LOGISTIC, G=G, workspace=ws)
    check(G, reference(X, y, W, gcx.GC_LOSS_LOGISTIC))


@pytest.mark.parametrize("n", [4, 4000])
def test_whole_quads_off_their_boundary_are_refused(n):
    X, y, W = problem(2, n, 64, 16)
    off = torch.empty(X.numel() + 1, device="cuda")[1:].view(X.shape)
    with pytest.raises(gcx.GcxError):
        gcx.gc_chunk_grads(off.copy_(X), y, W, gcx.GC_LOSS_LINEAR)


@pytest.mark.parametrize("b", [1, 20, 33, 64, 128])
@pytest.mark.parametrize("kind", ["inf in X", "inf in W", "NaN in X", "NaN in W", "near the largest float"])
def test_values_that_are_not_finite(kind, b):
    """They reach the outputs that they reach in 64 bits, and no others."""
    N, n, d = 3, 70, 5001
    X, y, W = problem(N, n, d, b)
    Wv = W.view(b, d)
    if kind == "inf in X":
        X[1, 40, 77] = float("inf")
    elif kind == "inf in W":
        Wv[b - 1, 5000] = -float("inf")
    elif kind == "NaN in X":
        X[2, 0, 5000] = float("nan")
    elif kind == "NaN in W":
        Wv[b // 2, 0] = float("nan")
    else:
        X[0, 69, 4096] = 3.4e38
        Wv[:, 4096] = 2e-38
    G = gcx.gc_chunk_grads(X, y, W, gcx.GC_LOSS_LOGISTIC).double().view(b, N, d)
    ref = reference(X, y, W, gcx.GC_LOSS_LOGISTIC)
    assert torch.equal(G.isnan(), ref.isnan())
    assert torch.equal(G.isinf(), ref.isinf())
    ok = ref.isfinite()
    assert torch.allclose(G[ok].sign() * G[ok].abs().clamp_min(1e-3), ref[ok].sign() * ref[ok].abs().clamp_min(1e-3),
                          rtol=2e-3, atol=2e-5)


@pytest.mark.parametrize("N,n,d,b", [(4, 512, 16384, 6), (2, 512, 16384, 17), (2, 2048, 2048, 8), (1, 8192, 1024, 17),
                                     (3, 150, 4096, 5), (1, 2100, 260, 33), (1, 4096, 8192, 18)])
def test_error_of_short_sums(N, n, d, b):
    """Rows of up to 16384 columns in whole float4 at a few points, or at a number of points that 4 does
    not divide: the error against 64 bits stays below that of the kernel that takes one point at a time
    (sums of a row over a block, of a block's rows; 1.2 to 2e-7 at these sizes, growing with n), where
    one accumulator for a whole sum gave 2.1 to 5e-7."""
    X, y, W = problem(N, n, d, b)
    ref = reference(X, y, W, gcx.GC_LOSS_LINEAR)
    G = gcx.gc_chunk_grads(X, y, W, gcx.GC_LOSS_LINEAR)
    one = torch.stack([gcx.gc_chunk_grads(X, y, w.contiguous(), gcx.GC_LOSS_LINEAR) for w in W])
    err, single = ((g.double() - ref).norm() / ref.norm() for g in (G, one))
    assert float(err) <= float(single)


@pytest.mark.parametrize("N,n,d,b", [
    # one position per lane: columns around its tiles of 128; partials in the workspace (whole quads, and
    # rows of whole float4 at a few points) and in G; segments of both products and their remainders
    (1, 600, 127, 65), (1, 600, 129, 40), (2, 520, 516, 16), (1, 3000, 2052, 20), (3, 700, 260, 132),
    (1, 2100, 1028, 7), (2, 1030, 4100, 9), (1, 129, 16384, 5), (1, 8200, 512, 6),
    (12, 600, 127, 65), (16, 600, 129, 40), (16, 520, 516, 16), (3, 3000, 2052, 20), (9, 700, 260, 132),
])
@pytest.mark.parametrize("loss", [gcx.GC_LOSS_LINEAR, gcx.GC_LOSS_LOGISTIC])
def test_as_many_rows_as_columns(N, n, d, b, loss):
    X, y, W = problem(N, n, d, b)
    G = torch.full((b, N, d), float("nan"), device="cuda")
    need = gcx.gc_chunk_grads_workspace_size(N, n, d, b)
    ws = torch.full((need + 64,), 0xff, dtype=torch.uint8, device="cuda")
    gcx.gc_chunk_grads(X, y, W, loss, G=G, workspace=ws[:need])
    check(G, reference(X, y, W, loss))
    assert bool((ws[need:] == 0xff).all())


@pytest.mark.parametrize("N,n,d,b", [(50, 512, 16, 1), (30, 400, 4, 3), (40, 2100, 32, 9)])
def test_few_columns_on_any_float(N, n, d, b):
    """Every array one float past a 16-byte boundary and a workspace of the size asked for, which holds the
    partials of the kernel for short rows but not the residuals."""
    X, y, W = problem(N, n, d, b)
    need = gcx.gc_chunk_grads_workspace_size(N, n, d, b)
    assert need < 4 * b * N * n

    def shifted(t):
        s = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
        return s.copy_(t)

    G = shifted(torch.full((N, d) if b == 1 else (b, N, d), float("nan"), device="cuda"))
    ws = torch.full((need + 64,), 0xff, dtype=torch.uint8, device="cuda")
    gcx.gc_chunk_grads(shifted(X), shifted(y), shifted(W), gcx.GC_LOSS_LOGISTIC, G=G, workspace=ws[4:4 + need])
    check(G, reference(X, y, W, gcx.GC_LOSS_LOGISTIC))
    assert bool((ws[4 + need:] == 0xff).all())


@pytest.mark.parametrize("N,n,d,b", [(4, 100, 4097, 5), (2, 130, 16384, 20), (3, 70, 4100, 64), (1, 600, 129, 40),
                                     (40, 100, 4097, 5), (16, 600, 129, 40)])
def test_small_residuals(N, n, d, b):
    """Residuals of separated data, far below 2^-108: no larger an error than at ordinary size (sums of up to
    600 products, 2 to 4e-7)."""
    X, y, W = problem(N, n, d, b)
    W *= 0
    y.normal_().mul_(2.0 ** -118)
    ref = reference(X, y, W, gcx.GC_LOSS_LINEAR)
    G = gcx.gc_chunk_grads(X, y, W, gcx.GC_LOSS_LINEAR)
    assert float((G.double() - ref).norm() / ref.norm()) <= 5e-7


@pytest.mark.parametrize("b", [5, 20, 64])
def test_sums_near_the_largest_float(b):
    """A product whose leading parts round up past the largest float while it does not."""
    N, n, d = 2, 40, 5000
    X, y, W = problem(N, n, d, b)
    W *= 0
    y[1, 7] = -(2.0 ** 64)
    X[1, 7, 1234] = 1.998 * 2.0 ** 63
    G = gcx.gc_chunk_grads(X, y, W, gcx.GC_LOSS_LINEAR)
    assert bool(G.isfinite().all())
    check(G, reference(X, y, W, gcx.GC_LOSS_LINEAR))
    ref = 1.998 * 2.0 ** 127
    assert float((G[:, 1, 1234].double() - ref).abs().max()) <= 1e-6 * ref
