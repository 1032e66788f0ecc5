"""The time of chunk gradients at several points against that of the same X at one point, at sizes
where the plan decides between a good and a bad use of the chip.  Bars: about midway between the
two ratios measured."""
import pytest

torch = pytest.importorskip("torch")

from paper_2405_19509_amd import gcx  # noqa: E402
from test_encode_rates_gpu import fastest  # noqa: E402

pytestmark = pytest.mark.gpu


def points_over_one(N, n, d, b):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn((N, n, d), generator=g, device="cuda") * d ** -0.5
    y = (torch.rand((N, n), generator=g, device="cuda") < 0.5).float()
    W = torch.randn((b, d), generator=g, device="cuda")

    def call(W):
        G = torch.empty((N, d) if W.dim() == 1 else (W.shape[0], N, d), device="cuda")
        ws = torch.empty(gcx.gc_chunk_grads_workspace_size(N, n, d, W.shape[0] if W.dim() > 1 else 1),
                         dtype=torch.uint8, device="cuda")
        return fastest(lambda: gcx.gc_chunk_grads(X, y, W, gcx.GC_LOSS_LINEAR, G=G, workspace=ws))
    return call(W) / call(W[0].contiguous())


def test_four_points_of_short_rows():
    """Four passes of the kernel for one point (2.0) against the matrix cores in a long chain (3.9)."""
    assert points_over_one(8, 8192, 2048, 4) < 3


@pytest.mark.parametrize("N,n,d,b,bar", [(10, 512, 1000, 64, 2.2), (2, 4000, 4096, 64, 2.9), (1, 8192, 8192, 16, 2.7)])
def test_chunks_of_as_many_rows_as_columns(N, n, d, b, bar):
    """Column splits that fill the chip (ratios 1.6, 2.0, 1.9), against one split (2.8, 3.8, 3.5)."""
    assert points_over_one(N, n, d, b) < bar


@pytest.mark.parametrize("N,n,d,b,bar", [(5, 200, 1001, 8, 1.7), (1, 1000, 333, 17, 2.7), (2, 12, 100001, 4, 2.2)])
def test_small_calls_at_several_points(N, n, d, b, bar):
    """Rows off float4, one point at a time (ratios 1.2, 1.1, 1.1), against three launches and their
    chains (2.3, 4.4, 3.3)."""
    assert points_over_one(N, n, d, b) < bar
