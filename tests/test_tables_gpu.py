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


@pytest.mark.parametrize("opt", ["sgd", "adamw"])
@pytest.mark.parametrize("n", [223, 224, 225, 300, 1024, 1025, 4096, 4097, 8193])
def test_gradient_tables_back_to_back(n, opt):
    """The gradients' addresses ride in the kernel's arguments up to 224 segments, beyond that in a page-locked table that
    one block or, beyond 4096 segments, several fetch.  The steps follow each other with no read between them, behind a
    stream that is still busy, each with other gradients and other decayed segments: a table that the next call writes too
    early, or that is not read whole, shows in the parameters."""
    import torch
    steps, lr, wd, f = 6, 2.0 ** -4, 2.0, np.float32
    w, m, v = torch.full((n,), 64.0, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    rng = np.random.default_rng(n)
    stream = torch.cuda.current_stream().cuda_stream
    grads = [torch.from_numpy(rng.integers(-8, 8, n).astype(np.float32)).cuda() for _ in range(steps)]
    order = [rng.permutation(n) for _ in range(steps)]  # segment l takes the gradient at order[l]
    decay = [rng.integers(0, 2, n).astype(np.uint8) for _ in range(steps)]
    ptrs = [[g.data_ptr() + 4 * int(k) for k in o] for g, o in zip(grads, order)]
    want = np.full(n, 64.0, np.float32)
    ref_m, ref_v = np.zeros(n, np.float32), np.zeros(n, np.float32)
    ctx = LC.lc_init_layout(LC.LayoutDesc(tiny_layers(n, w=w, m=m, v=v), n, LC.LC_DT_F32, False, LC.LC_MODE_ACCUM,
                                          [1e300] * n, s_max=99, stream=stream))
    try:
        torch.cuda.synchronize()
        busy = torch.zeros(256 << 20, dtype=torch.uint8, device="cuda")
        for _ in range(8):
            busy += 1
        for t in range(steps):
            if opt == "sgd":
                LC.lc_sgd_step_score(ctx, t + 1, ptrs[t], LC.LC_DT_F32, lr, wd, decay[t])
            else:
                LC.lc_adamw_step_score(ctx, t + 1, ptrs[t], LC.LC_DT_F32, lr, 0.5, 0.5, 1e-8, wd, t + 1, decay[t])
        host = [x.cpu().numpy() for x in grads]
        for t in range(steps):
            g = host[t][order[t]]
            d = np.where(decay[t] == 1, want * f(1.0 - lr * wd), want)
            if opt == "sgd":
                want = d - f(lr) * g
            else:
                ref_m = f(0.5) * ref_m + f(0.5) * g
                ref_v = f(0.5) * ref_v + f(0.5) * (g * g)
                c = f(1.0 / (1.0 - 0.5 ** (t + 1)))
                want = d - f(lr) * ((ref_m * c) / (np.sqrt(ref_v * c) + f(1e-8)))
        assert np.array_equal(w.cpu().numpy(), want.astype(np.float32))
        if opt == "adamw":
            assert np.array_equal(m.cpu().numpy(), ref_m) and np.array_equal(v.cpu().numpy(), ref_v)
    finally:
        LC.lc_destroy(ctx)
