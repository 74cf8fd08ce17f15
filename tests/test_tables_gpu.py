"""GPU: the small tables that kernels move between page-locked host memory and
the device, at any number of entries: the state of every layer to the host,
the gradient table of an optimizer step to the kernel.  Values are chosen so
that every result is exact."""
import numpy as np
import pytest

from paper_2609_27193_amd import layercheck as LC
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("needs an MI355X")
    LC.load_library()


def tiny_layers(n, **arrays):
    """n layers of one fp32 element each, at elements 0 .. n - 1 of the given arrays."""
    at = lambda a, l: None if a is None else a.data_ptr() + 4 * l  # noqa: E731
    return [LC.Segment(l, 1, *(at(arrays.get(k), l) for k in ("w", "s", "M", "m", "v"))) for l in range(n)]


@pytest.mark.parametrize("n", [1, 256, 257, 8192, 8193, 20001])
def test_state_of_every_layer(n):
    import torch
    idx = torch.arange(n, device="cuda")
    w = torch.ones(n, device="cuda")
    s = torch.empty(n, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    ctx = LC.lc_init_layout(LC.LayoutDesc(tiny_layers(n, w=w, s=s), n, LC.LC_DT_F32, False, LC.LC_MODE_ACCUM,
                                          [1e300 if l % 3 else 0.0 for l in range(n)], s_max=99, eps_w=0.0, stream=stream))
    try:
        w += (idx % 7).float()  # |S| = 1: u is the change itself
        LC.lc_score_layers(ctx, 5)
        LC.lc_select(ctx, 5, 1.0, n)
        u, delta, t_last = LC.lc_read_state(ctx, n)
        l = np.arange(n)
        assert np.array_equal(u, (l % 7).astype(np.float64))
        assert np.array_equal(delta, np.where(l % 3, l % 7, 0).astype(np.float64))
        assert np.array_equal(t_last, np.where(l % 3, 0, 5))
    finally:
        LC.lc_destroy(ctx)
