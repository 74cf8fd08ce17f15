"""GPU: every chunk and piece of a launch is worked on exactly once, whatever
the number of blocks leaves behind the last runs of the block -> item mapping
(runs of 32 chunks and of 64 pieces per XCD, 8 XCDs), also on a large state."""
import pytest

from paper_2609_27193_amd import layercheck as LC
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("needs an MI355X")
    LC.load_library()


@pytest.mark.parametrize("chunks", [1, 7, 8, 9, 255, 256, 257, 263, 264, 511, 513, 519, 775, 1023, 1025, 2047, 2049, 2600])
def test_each_item_once(chunks):
    import torch
    n = chunks * (LC.lc_query_build()["chunk_bytes"] // 4) - 5
    dev, stream = torch.device("cuda"), torch.cuda.current_stream().cuda_stream
    idx = torch.arange(n, device=dev)
    W = (idx % 1021).float()
    S, m, v = torch.zeros_like(W), (idx % 1019).float(), (idx % 1013).float()
    g = torch.ones_like(W)
    seg = LC.Segment(0, n, W.data_ptr(), S.data_ptr(), None, m.data_ptr(), v.data_ptr())
    ctx = LC.lc_init_layout(LC.LayoutDesc([seg], 1, LC.LC_DT_F32, False, LC.LC_MODE_ACCUM, [0.0], s_max=9, stream=stream))
    try:
        assert torch.equal(S, W)
        W += 1.0
        LC.lc_score_layers(ctx, 1)
        u = LC.lc_read_state(ctx, 1)[0][0]
        assert torch.equal(S, W)
        want = 1.0 / (float((idx % 1021).double().mean()) + 1e-8)
        assert abs(u - want) <= 1e-12 * want, (u, want)  # integers: every fp32 term and pair is exact
        mask, st = LC.lc_select(ctx, 1, 1.0, 1)
        R = LC.lc_record_bytes(ctx, 0)
        staging = torch.full((R + 4096,), 0x5A, dtype=torch.uint8, device=dev)
        assert LC.lc_pack_selected(ctx, staging.data_ptr(), R, 0)["done"] == 1
        torch.cuda.synchronize()
        block = R // 3
        for k, a in enumerate((W, m, v)):
            assert torch.equal(staging[k * block:k * block + 4 * n].view(torch.float32), a)
        assert (staging[R:] == 0x5A).all()
        LC.lc_sgd_step_score(ctx, 2, [g.data_ptr()], LC.LC_DT_F32, 1.0, 0.0)  # p_new = p - 1, exactly
        u = LC.lc_read_state(ctx, 1)[0][0]
        assert torch.equal(W, (idx % 1021).float())
        want = 1.0 / (float((idx % 1021 + 1).double().mean()) + 1e-8)
        assert abs(u - want) <= 1e-12 * want, (u, want)
        versions = [{"step": 1, "mask": mask, "payload": staging.data_ptr(), "payload_bytes": R}]
        for a in (W, S, m, v):
            a.zero_()
        assert LC.lc_restore_composite(ctx, versions, 1, 1).tolist() == [1]
        assert torch.equal(W, (idx % 1021).float() + 1.0) and torch.equal(S, W)
        assert torch.equal(m, (idx % 1019).float()) and torch.equal(v, (idx % 1013).float())
    finally:
        LC.lc_destroy(ctx)


@pytest.mark.parametrize("past", [0, 1, 4096 - (9 << 18) % 4096 + 8])
def test_each_chunk_once_on_a_large_state(past):
    import torch
    n = ((9 << 18) + past) * (LC.lc_query_build()["chunk_bytes"] // 2) - 3
    if torch.cuda.mem_get_info()[0] < 5 * n:
        pytest.skip("needs 48 GB of device memory")
    dev, stream = torch.device("cuda"), torch.cuda.current_stream().cuda_stream
    base = (torch.arange(251 << 16, device=dev) % 251).bfloat16()  # integers below 2^8: exact, also one more
    W = torch.empty(n, dtype=torch.bfloat16, device=dev)
    total = 0.0
    for i in range(0, n, base.numel()):
        part = base[:min(base.numel(), n - i)]
        W[i:i + part.numel()] = part
        total += float(part.double().sum())
    S = torch.zeros_like(W)
    seg = LC.Segment(0, n, W.data_ptr(), S.data_ptr(), None, None, None)
    ctx = LC.lc_init_layout(LC.LayoutDesc([seg], 1, LC.LC_DT_BF16, False, LC.LC_MODE_ACCUM, [0.0], s_max=9, stream=stream))
    try:
        W += 1.0
        LC.lc_score_layers(ctx, 1)
        u = LC.lc_read_state(ctx, 1)[0][0]
        want = 1.0 / (total / n + 1e-8)
        assert abs(u - want) <= 1e-12 * want, (u, want)  # a chunk left out or taken twice is 4e-7 of it
        assert torch.equal(S, W)
    finally:
        LC.lc_destroy(ctx)
