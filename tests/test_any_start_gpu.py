"""GPU: segments that start at any element, as the pieces of a ZeRO-3 rank
do, with every array of a segment at an element offset of its own against a
128-byte line (the weights, the shadow, the fp32 arrays and the gradient may
all differ), and lengths around a head, a tile and the first chunk's edge.
Every array lies between guard bytes, which stay as they were.  Scores to
1e-5 (fp64 sums), everything else exact, against the CPU oracle."""
import numpy as np
import pytest

from oracle import layercheck_oracle as O
from paper_2609_27193_amd import layercheck as LC
from tests.conftest import gpu_available
from tests.gpu_harness import rel_ok

pytestmark = pytest.mark.gpu
GUARD = 512  # bytes on each side of an array


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not gpu_available():
        pytest.skip("needs an MI355X")
    LC.load_library()


class Arr:
    """One array of one segment at byte ``off`` past a 128-byte line, with its host copy."""

    def __init__(self, host, off):
        import torch
        self.host, self.off = host, GUARD + off
        self.buf = torch.full((2 * GUARD + host.nbytes + 128,), 0xA5, dtype=torch.uint8, device="cuda")
        assert self.buf.data_ptr() % 128 == 0
        self.ptr = self.buf.data_ptr() + self.off
        self.put()

    def put(self):
        import torch
        b = torch.from_numpy(self.host.view(np.uint8).copy())
        self.buf[self.off:self.off + b.numel()].copy_(b)

    def check(self, what):
        g = self.buf.cpu().numpy()
        n = self.host.nbytes
        assert np.array_equal(g[self.off:self.off + n], self.host.view(np.uint8)), what
        assert (g[:self.off] == 0xA5).all() and (g[self.off + n:] == 0xA5).all(), f"{what}: guard bytes written"


def bf16(x):
    """Round-to-nearest-even bf16 bits of finite fp32 values."""
    u = x.astype(np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def lengths(esz):
    tile, line = LC.lc_query_build()["chunk_bytes"] // esz, 128 // esz
    return [1, line - 1, line, line + 1, tile - 1, tile, tile + 1, tile + line - 1, tile + line, 2 * tile, 2 * tile + 5,
            3 * tile + line - 1]


# element offsets of (weights, shadow, fp32 arrays, gradient), taken in turn by the segments
ALIKE = [(e, e, e, e) for e in (1, 7, 8, 33, 0)]
APART = [(1, 0, 0, 2), (0, 1, 3, 1), (5, 2, 1, 0), (0, 0, 1, 3), (8, 16, 4, 8), (3, 3, 0, 3), (0, 8, 0, 0)]
GRAD = [(0, 0, 0, 1), (0, 0, 0, 2), (0, 1, 0, 3), (8, 8, 8, 7), (0, 0, 0, 0)]  # the gradient alone


@pytest.mark.parametrize("offsets", [ALIKE, APART, GRAD], ids=["alike", "apart", "gradient"])
@pytest.mark.parametrize("dtype,master,op", [("bf16", True, "accum"), ("bf16", False, "snapshot"), ("f32", False, "accum"),
                                             ("f32", True, "snapshot"), ("bf16", True, "adamw"), ("bf16", False, "adamw"),
                                             ("f32", False, "adamw"), ("bf16", True, "sgd"), ("f32", False, "sgd")])
def test_segments_at_any_element(dtype, master, op, offsets):
    import torch
    rng = np.random.default_rng(17)
    esz = 2 if dtype == "bf16" else 4
    wbits = bf16 if dtype == "bf16" else (lambda x: x.astype(np.float32))
    draw = lambda n, s: (rng.standard_normal(n) * s).astype(np.float32)  # noqa: E731
    sizes = lengths(esz)
    layer_of = [i // 3 for i in range(len(sizes))]
    N = layer_of[-1] + 1
    segs, grad_dt = [], "f32" if master else "bf16"
    for i, n in enumerate(sizes):
        ow, os_, of, og = offsets[i % len(offsets)]
        p = draw(n, 0.02)
        d = {"w": Arr(wbits(p), ow * esz), "s": Arr(np.zeros(n, wbits(p).dtype), os_ * esz),
             "M": Arr(p.copy(), of * 4) if master else None, "m": Arr(draw(n, 1e-3), of * 4),
             "v": Arr(np.abs(draw(n, 1e-6)), of * 4)}
        g = draw(n, 1.0)
        d["g"] = Arr(g if grad_dt == "f32" else bf16(g), og * (4 if grad_dt == "f32" else 2))
        segs.append(d)
    arrays = ["w", "s", "m", "v"] + ["M"] * master
    osegs = [O.OSegment(l, d["w"].host, d["s"].host, d["M"].host if master else None, d["m"].host, d["v"].host)
             for l, d in zip(layer_of, segs)]
    lsegs = [LC.Segment(l, n, d["w"].ptr, d["s"].ptr, d["M"].ptr if master else None, d["m"].ptr, d["v"].ptr)
             for l, n, d in zip(layer_of, sizes, segs)]
    mode = LC.LC_MODE_SNAPSHOT if op == "snapshot" else LC.LC_MODE_ACCUM
    lc_dt = LC.LC_DT_BF16 if esz == 2 else LC.LC_DT_F32
    k0 = [0.0 if l % 2 else 1e300 for l in range(N)]  # every second layer at each step, the others by age
    orc = O.LayerCheckOracle(osegs, N, lc_dt, master, mode, k0, 2, eps_w=1e-8, t_base=0)
    stream = torch.cuda.current_stream().cuda_stream
    ctx = LC.lc_init_layout(LC.LayoutDesc(lsegs, N, lc_dt, master, mode, k0, 2, eps_w=1e-8, stream=stream))
    decay = [i % 2 for i in range(len(sizes))]

    def check(what):
        torch.cuda.synchronize()
        for i, d in enumerate(segs):
            for a in arrays:
                d[a].check(f"{what}: {a} of segment {i} ({sizes[i]} elements, offsets {offsets[i % len(offsets)]})")

    def pack():
        total = sum(LC.lc_record_bytes(ctx, l) for l in range(N))
        staging = torch.full((total,), 0x5A, dtype=torch.uint8, device="cuda")
        got = LC.lc_pack_selected(ctx, staging.data_ptr(), total, 0)
        want, res = orc.pack(0, total)
        assert got == res
        h = staging.cpu().numpy()
        k = got["bytes_written"]
        assert np.array_equal(h[:k], want) and (h[k:] == 0x5A).all()
        return staging, k

    try:
        check("init")
        versions, host = [], []
        b, k = pack()
        versions.append({"step": 0, "mask": np.ones(N, np.uint8), "payload": b.data_ptr(), "payload_bytes": k, "keep": b})
        host.append({"step": 0, "mask": np.ones(N, np.uint8), "payload": b.cpu().numpy()[:k]})
        for t in (1, 2):
            if op in ("adamw", "sgd"):
                gdt = LC.LC_DT_F32 if grad_dt == "f32" else LC.LC_DT_BF16
                ptrs = [d["g"].ptr for d in segs]
                gf = [d["g"].host if grad_dt == "f32" else (d["g"].host.astype(np.uint32) << 16).view(np.float32)
                      for d in segs]
                if op == "adamw":
                    LC.lc_adamw_step_score(ctx, t, ptrs, gdt, 1e-3, 0.9, 0.95, 1e-8, 0.1, t, decay)
                    orc.adamw_step_score(t, gf, 1e-3, 0.9, 0.95, 1e-8, 0.1, t, decay)
                else:
                    LC.lc_sgd_step_score(ctx, t, ptrs, gdt, 1e-3, 0.1, decay)
                    orc.sgd_step_score(t, gf, 1e-3, 0.1, decay)
            else:
                for d in segs:
                    x = d["M"].host if master else (d["w"].host if esz == 4 else
                                                    (d["w"].host.astype(np.uint32) << 16).view(np.float32))
                    x = (x + draw(len(x), 1e-3)).astype(np.float32)
                    d["w"].host[...] = wbits(x)
                    d["w"].put()
                    if master:
                        d["M"].host[...] = x
                        d["M"].put()
                LC.lc_score_layers(ctx, t)
                orc.score(t)
            u, delta, _ = LC.lc_read_state(ctx, N)
            assert rel_ok(u, orc.u) and rel_ok(delta, orc.delta), (u, orc.u)
            check(f"step {t}")
            mask, _ = LC.lc_select(ctx, t, 1.0, N)
            orc.select(t, 1.0)
            assert np.array_equal(mask, orc.mask)
            b, k = pack()
            check(f"pack {t}")
            versions.append({"step": t, "mask": mask, "payload": b.data_ptr(), "payload_bytes": k, "keep": b})
            host.append({"step": t, "mask": mask, "payload": b.cpu().numpy()[:k]})
        chosen = LC.lc_restore_composite(ctx, versions, 1, N)
        assert chosen.tolist() == orc.restore(host, 1).tolist()
        check("restore")
        # the same from host memory: page-locked (a kernel reads it), at odd places of one allocation, and pageable
        pinned = torch.empty(sum(h["payload"].nbytes + 256 for h in host), dtype=torch.uint8, pin_memory=True)
        for where in ("pinned", "pageable", "mixed"):
            at, hv = 2, []
            for h in host:
                k = h["payload"].nbytes
                if where == "pinned" or where == "mixed" and h["step"] == 1:
                    buf = pinned[at:at + k]
                    buf.copy_(torch.from_numpy(h["payload"].copy()))
                    at += k + 254
                else:
                    buf = torch.from_numpy(h["payload"].copy())
                hv.append({"step": h["step"], "mask": h["mask"], "payload": buf.data_ptr(), "payload_bytes": k, "keep": buf})
            for d in segs:
                for a in arrays:
                    d[a].buf[d[a].off:d[a].off + d[a].host.nbytes] = 0x33
            assert LC.lc_restore_composite(ctx, hv, 1, N).tolist() == chosen.tolist()
            check(f"restore from {where} memory")
    finally:
        LC.lc_destroy(ctx)


@pytest.mark.parametrize("N", [1, 107, 108, 109, 300])
def test_restore_of_any_number_of_layers(N):
    """The ranks of a restore ride in the kernel's arguments up to 108 layers, beyond that in a table."""
    import torch
    sizes = [1 + l % 7 * 50 for l in range(N)]
    arrs = [torch.arange(sum(sizes), device="cuda").float() + k for k in range(4)]  # w, s, m, v
    segs, at = [], 0
    for l, n in enumerate(sizes):
        w, s, m, v = (a.data_ptr() + 4 * at for a in arrs)
        segs.append(LC.Segment(l, n, w, s, None, m, v))
        at += n
    stream = torch.cuda.current_stream().cuda_stream
    ctx = LC.lc_init_layout(LC.LayoutDesc(segs, N, LC.LC_DT_F32, False, LC.LC_MODE_ACCUM,
                                          [0.0 if l % 3 == 0 else 1e300 for l in range(N)], s_max=99, stream=stream))
    try:
        total = sum(LC.lc_record_bytes(ctx, l) for l in range(N))
        bufs, versions = [], []
        for t in (0, 1):
            if t:
                for a in (arrs[0], arrs[2], arrs[3]):
                    a += 0.5
                LC.lc_score_layers(ctx, t)
                mask, _ = LC.lc_select(ctx, t, 1.0, N)
                assert mask.tolist() == [int(l % 3 == 0) for l in range(N)]
            else:
                mask = np.ones(N, np.uint8)
            bufs.append(torch.empty(total, dtype=torch.uint8, device="cuda"))
            r = LC.lc_pack_selected(ctx, bufs[t].data_ptr(), total, 0)
            assert r["done"] == 1
            versions.append({"step": t, "mask": mask, "payload": bufs[t].data_ptr(), "payload_bytes": r["bytes_written"]})
        later = torch.repeat_interleave(torch.tensor([0.5 * (l % 3 == 0) for l in range(N)], device="cuda"),
                                        torch.tensor(sizes, device="cuda"))
        want = [torch.arange(sum(sizes), device="cuda").float() + k + later for k in range(4)]
        for a in arrs:
            a.fill_(-1.0)
        assert LC.lc_restore_composite(ctx, versions, 3, N).tolist() == [int(l % 3 == 0) for l in range(N)]
        for k in (0, 2, 3):
            assert torch.equal(arrs[k], want[k]), k
        assert torch.equal(arrs[1], want[0])
        _, delta, t_last = LC.lc_read_state(ctx, N)
        assert not delta.any() and t_last.tolist() == [int(l % 3 == 0) for l in range(N)]
        with pytest.raises(LC.LCError):
            LC.lc_score_layers(ctx, 3)  # the next step must exceed t_fail
        LC.lc_score_layers(ctx, 4)
    finally:
        LC.lc_destroy(ctx)


@pytest.mark.parametrize("where", ["pinned", "device"])
@pytest.mark.parametrize("place", [0, 2, 16, 64])
@pytest.mark.parametrize("first", [0, 4, 5])
def test_records_written_again_between_restores(first, place, where):
    """Records at, beside and off a line, arrays too; the second restore reads what the host wrote into the same memory."""
    import torch
    n = 2 * 2048 + 77  # fp32: whole pieces and a tail
    arrs = [torch.zeros(n + 64, device="cuda") for _ in range(4)]  # w, s, m, v
    seg = LC.Segment(0, n, *(a.data_ptr() + 4 * first if a is not None else None for a in (*arrs[:2], None, *arrs[2:])))
    ctx = LC.lc_init_layout(LC.LayoutDesc([seg], 1, LC.LC_DT_F32, False, LC.LC_MODE_ACCUM, [1.0], s_max=9,
                                          stream=torch.cuda.current_stream().cuda_stream))
    try:
        size = LC.lc_record_bytes(ctx, 0)
        host = torch.empty(size + 256, dtype=torch.uint8, pin_memory=True)
        buf = host if where == "pinned" else torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        v = [{"step": 3, "mask": np.ones(1, np.uint8), "payload": buf.data_ptr() + place, "payload_bytes": size}]
        rng = np.random.default_rng(first)
        for _ in range(3):
            rec = rng.integers(0, 2 ** 16, (3, size // 12), dtype=np.uint32)
            host.numpy()[place:place + size] = rec.view(np.uint8).reshape(-1)
            if where == "device":
                buf.copy_(host)
            assert LC.lc_restore_composite(ctx, v, 3, 1).tolist() == [3]
            for a, r in zip(arrs, (rec[0], rec[0], rec[1], rec[2])):
                got = a.cpu().numpy().view(np.uint32)
                assert np.array_equal(got[first:first + n], r[:n])
                assert not got[:first].any() and not got[first + n:].any()
    finally:
        LC.lc_destroy(ctx)
