"""Operands whose two passes share a launch, and operands that go along in one: the same outputs as each of them gives alone launch by launch; also where
no wave waits to be told and all of them take the figures themselves, and from a replayed graph."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

# sizes at the edges of the first pass's tiles (64 x 256, pieces of 4096 of a row, four to a workgroup) and of the groups of eight workgroups
BLOCKS = [(128, 128), (128, 8320), (1152, 640), (1024, 2048), (2176, 1152), (896, 384)]
ROWS = [(1, 4096), (333, 4104), (1027, 1000), (512, 4096), (250, 14336), (5, 16384), (64, 8)]
NAMES = ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask", "scale_e8m0", "group_mantissa")


def _operands(gran, dev):
    """Operands that stay in E4M3, that fall back with and without a proof, and with an infinity."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(7)
    xs = []
    for k, (rows, cols) in enumerate(ROWS if gran == "channel_row" else BLOCKS):
        x = torch.randn((rows, cols), generator=gen, device=dev)
        if k % 3 == 1:
            x *= torch.where(torch.rand((rows, cols), generator=gen, device=dev) < 0.3, 1e-9, 1.0)
        if k % 3 == 2:
            x *= torch.where(torch.rand((rows, cols), generator=gen, device=dev) < 0.035, 1e-9, 1.0)
        x = x.to(torch.bfloat16)
        if k == 4:
            x[rows // 2, cols // 2] = float("inf")
        xs.append(x)
    return xs


def _entry(B, x, gran, scope, fake, dev):
    p = B.make_params(*x.shape, gran, scope, "mean_rel_err", 0.045, scaling="gam")
    out = B.alloc_outputs(p, dev, want_bf16=not fake, want_fp8=not fake, bf16_fill=0x1234)
    out.workspace = None
    for n in NAMES:
        t = getattr(out, n)
        if t is not None and n != "bf16":
            t.view(torch.uint8).fill_(0x5A)
    y = torch.full(x.shape, 3.0, dtype=torch.bfloat16, device=dev) if fake else None
    st = torch.full((B.STATS_BYTES,), 0x5A, dtype=torch.uint8, device=dev) if not fake else None
    return p, x, out, st, y


def _same(want, got, case):
    for k, (a, b) in enumerate(zip(want, got)):
        for n in NAMES:
            u, v = getattr(a[2], n), getattr(b[2], n)
            assert (u is None) == (v is None) and (u is None or torch.equal(u.view(torch.uint8), v.view(torch.uint8))), (case, k, n)
        for u, v in ((a[3], b[3]), (a[4], b[4])):
            assert u is None or torch.equal(u.view(torch.uint8), v.view(torch.uint8)), (case, k)


def _run(B, entries, polls=None):
    items = B.make_batch(entries)
    ws = torch.full((max(16, B.mor_batch_workspace_bytes(items)),), 0xA7, dtype=torch.uint8, device=entries[0][1].device)
    if polls is None:
        B.mor_analyze_quantize_batch(items, 1e-5, ws)
    else:
        lib = B.load()
        lib.mor_test_batch.argtypes = [C.POINTER(B.MorBatchItem), C.c_int32, C.c_float, C.c_void_p, C.c_size_t, C.c_void_p, C.c_int32]
        assert lib.mor_test_batch(items, len(items), 1e-5, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, polls) == 0
    torch.cuda.synchronize()
    return ws


@pytest.mark.parametrize("fake", [False, True])
@pytest.mark.parametrize("scope", ["tensor", "partition"])
@pytest.mark.parametrize("gran", ["block128", "block64", "channel_row"])
def test_both_passes_in_a_launch(gran, scope, fake):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    xs = _operands(gran, dev)
    assert sum(x.numel() for x in xs) * 2 >= 8 << 20
    want = [_entry(B, x, gran, scope, fake, dev) for x in xs]
    for e in want:
        _run(B, [e])
    assert {int(e[2].mask.max()) for e in want} == {0, 1}
    for polls in (None, 0):
        print(f"[stream] {gran} {scope} fake={fake} polls={polls}", flush=True)
        got = [_entry(B, x, gran, scope, fake, dev) for x in xs]
        _run(B, got, polls)
        _same(want, got, (gran, scope, fake, polls))
    # captured and replayed, with other work between the replays
    got = [_entry(B, x, gran, scope, fake, dev) for x in xs]
    items = B.make_batch(got)
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0x3C, dtype=torch.uint8, device=dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.mor_analyze_quantize_batch(items, 1e-5, ws)
    for replay in range(3):
        for e in got:
            for t in (e[2].scale, e[2].err_sum, e[4] if fake else e[2].fp8):
                t.view(torch.uint8).fill_(0x33)
        graph.replay()
        torch.cuda.synchronize()
        _same(want, got, (gran, scope, fake, "replay", replay))


@pytest.mark.parametrize("gran, rows, cols", [("block64", 4096, 4096), ("channel_row", 8192, 4096), ("channel_row", 2048, 14336), ("block128", 8192, 8192)])
def test_a_large_operand_alone(gran, rows, cols):
    """Against two smaller halves of its rows as bands would be wrong (one group), so against the same operand beside 300 MB of others,
    where two or three operands are taken launch by launch."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(11)
    x = torch.randn((rows, cols), generator=gen, device=dev)
    x = (x * torch.where(torch.rand((rows, cols), generator=gen, device=dev) < 0.1, 1e-8, 1.0)).to(torch.bfloat16)
    other = torch.ones((16384, 8192), dtype=torch.bfloat16, device=dev)
    print(f"[stream] alone {gran} {rows}x{cols}", flush=True)
    want = [_entry(B, x, gran, "tensor", False, dev), _entry(B, other, gran, "tensor", False, dev)]
    _run(B, want)
    for polls in (None, 0):
        got = [_entry(B, x, gran, "tensor", False, dev)]
        _run(B, got, polls)
        _same(want[:1], got, (gran, rows, cols, polls))


# tile edges of per-tensor operands (2048 chunks of 8 elements): one chunk, a whole tile, a chunk more, ragged ones, and one that fills the launch
TENSORS = [(8192, 2568), (1, 8), (1, 16384), (1, 16392), (333, 1000), (700, 4096)]


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("fake, lean", [(False, False), (True, False), (False, True)])
def test_per_tensor_operands(fake, lean, pad):
    """Against the oracle, and bit for bit against workgroups that do not wait."""
    import numpy as np
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(17)
    bufs = []
    for k, (rows, cols) in enumerate(TENSORS):
        x = torch.randn((rows, cols + pad), generator=gen, device=dev)
        share = (0.3, 0.0, 0.035, 0.3, 0.0, 0.3)[k]       # proven to fall back, E4M3, falling back without a proof
        x = (x * torch.where(torch.rand(x.shape, generator=gen, device=dev) < share, 1e-9, 1.0)).to(torch.bfloat16)
        if k == 4:
            x[rows // 2, cols // 2] = float("nan")
        bufs.append(x)
    results = []
    for polls in (None, 0):
        print(f"[stream] per tensor fake={fake} lean={lean} pad={pad} polls={polls}", flush=True)
        entries, guards = [], []
        for x, (rows, cols) in zip(bufs, TENSORS):
            p = B.make_params(rows, cols, "tensor", ld=cols + pad, lean_fp8=lean)
            out, g = parity.guarded_outputs(p, dev, want_bf16=not fake, bf16_fill=parity.FILL, want_fp8=not fake)
            out.workspace = None
            if not fake:
                out.fp8.fill_(0xA7)
            y = g.carve("y", (rows, cols), torch.int16, 0x1111) if fake else None
            st = g.carve("stats", (B.STATS_BYTES,), torch.uint8, 0x5A)
            entries.append((p, x[:, :cols], out, st, y.view(torch.bfloat16) if fake else None))
            guards.append(g)
        _run(B, entries, polls)
        for g in guards:
            g.check()
        results.append(entries)
    _same(*results, ("per tensor", fake, lean, pad))
    flags = [B.read_stats(e[3])["flags"] for e in results[0]]
    proven = [k for k in range(len(TENSORS)) if k in (0, 3, 5)]
    assert flags == [0 if pad or k not in proven else B.MOR_STATS_FLAG_FUSED_FALLBACK for k in range(len(TENSORS))]
    for k, (p, x, out, st, y) in enumerate(results[0]):
        rows, cols = TENSORS[k]
        bits = bufs[k].view(torch.int16).cpu().numpy().view(np.uint16)
        want = parity.O.analyze_quantize(bits, "tensor", "partition", "mean_rel_err", 0.045, bf16_fill=parity.FILL, ld=cols + pad, cols=cols)
        if lean and not pad and k in proven:
            assert bool((out.fp8 == 0xA7).all())
            out.fp8.copy_(torch.from_numpy(want.fp8.reshape(rows, cols)))
        if not fake:
            parity.compare(bits, "tensor", cols=cols, gpu=(p, out), label=f"stream {k}")
        else:
            alone, _ = parity.guarded_outputs(p, dev, want_bf16=False, want_fp8=False)
            y1 = torch.zeros((rows, cols), dtype=torch.bfloat16, device=dev)
            B.mor_fake_quantize(p, bufs[k], y1, alone)
            assert torch.equal(y1.view(torch.int16), y.view(torch.int16))
        assert int(out.mask[0]) == int(want.mask[0])


@pytest.mark.parametrize("gran, rows, cols, pad", [("tensor", 8192, 4096, 0), ("tensor", 8192, 8192, 8), ("block128", 8192, 8192, 0)])
def test_waves_that_are_not_told_share_the_operand(gran, rows, cols, pad):
    """Where no wave waits, all of them go for the operand's figures themselves, and together read it about once: 0.26 to 0.33 ms for these
    calls.  Each on its own, 8192 waves would read 64 MB in the smallest: more than 25 ms at 20 TB/s."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    x = torch.randn((rows, cols + pad), generator=gen, device=dev)
    x = (x * torch.where(torch.rand(x.shape, generator=gen, device=dev) < 0.1, 1e-8, 1.0)).to(torch.bfloat16)[:, :cols]
    scaling = "fp32_amax" if gran == "tensor" else "gam"
    entries = []
    for polls in (None, 0):
        p = B.make_params(rows, cols, gran, "partition" if gran == "tensor" else "tensor", ld=cols + pad, scaling=scaling)
        out = B.alloc_outputs(p, dev, bf16_fill=0x1234)
        out.workspace = None
        out.fp8.view(torch.uint8).fill_(0x5A)
        entries.append((p, x, out, None, None))
    _run(B, entries[:1])
    for _ in range(3):
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        print(f"[stream] untold {gran} {rows}x{cols}", flush=True)
        start.record()
        _run(B, entries[1:], 0)
        stop.record()
        stop.synchronize()
        assert start.elapsed_time(stop) < 5.0
        _same(entries[:1], entries[1:], (gran, rows, cols))


# (granularity, rows, cols, row padding, scaling): per-tensor operands first, then what goes along; edges of the 1 x 128 operand's units of 32 blocks and
# of the number that its waves take (one up to 6144 units, then two), of its two forms, and of groups of eight 128 x 128 blocks
ALONG = [
    [("tensor", 300, 1000, 0, "fp32_amax"), ("sub1x128", 33, 128, 0, "fp32_amax")],
    [("tensor", 1, 8, 0, "fp32_amax"), ("tensor", 2000, 4096, 0, "fp32_amax"), ("sub1x128", 6160, 4096, 0, "e8m0"), ("block128", 1152, 128, 0, "fp32_amax"),
     ("block128", 128, 1024, 0, "e8m0")],
    [("tensor", 300, 1000, 1000, "fp32_amax"), ("sub1x128", 301, 1000, 1000, "fp32_amax"), ("block128", 256, 256, 0, "fp32_amax")],
    [("tensor", 700, 4096, 8, "gam"), ("tensor", 64, 8, 8, "fp32_amax"), ("sub1x128", 65, 4104, 0, "e8m0"), ("block128", 8320, 8064, 128, "fp32_amax"),
     ("block128", 200, 256, 0, "fp32_amax"), ("block64", 128, 128, 0, "fp32_amax")],
    [("tensor", 4096, 4096, 0, "fp32_amax"), ("block128", 8192, 8192, 0, "fp32_amax")],
    [("tensor", 512, 2048, 0, "fp32_amax"), ("sub1x128", 64, 2048, 0, "fp32_amax"), ("sub1x128", 65, 2048, 0, "fp32_amax"), ("channel_col", 256, 384, 0, "fp32_amax")],
    # padded rows with blocks alone, and with 1 x 128 operands that keep their own launch: a dense one, two
    [("tensor", 4200, 2048, 2048, "fp32_amax"), ("block128", 1024, 1024, 0, "fp32_amax"), ("block128", 128, 128, 0, "e8m0")],
    [("tensor", 1000, 4096, 4096, "gam"), ("tensor", 1100, 1000, 8, "fp32_amax"), ("sub1x128", 256, 1024, 0, "fp32_amax"), ("block128", 1152, 640, 0, "fp32_amax")],
    [("tensor", 4200, 2048, 8, "fp32_amax"), ("sub1x128", 64, 2048, 0, "fp32_amax"), ("sub1x128", 65, 2056, 0, "fp32_amax"), ("block128", 256, 384, 0, "fp32_amax")],
    # as many operands with statistics as the finish pass has room for, and one more
    [("tensor", 300, 1000, 8, "fp32_amax"), ("sub1x128", 64, 256, 0, "fp32_amax"), ("block128", 256, 128, 0, "fp32_amax")] + [("block64", 64, 192, 0, "fp32_amax")] * 10,
    [("tensor", 300, 1000, 8, "fp32_amax"), ("sub1x128", 64, 256, 0, "fp32_amax"), ("block128", 256, 128, 0, "fp32_amax")] + [("block64", 64, 192, 0, "fp32_amax")] * 11,
]


@pytest.mark.parametrize("counted", [True, False])
@pytest.mark.parametrize("case", range(len(ALONG)))
def test_operands_that_go_along(case, counted):
    """1 x 128 and 128 x 128 operands in the launch of per-tensor ones: the outputs of each alone, and its statistics."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(100 + case)

    def entries():
        got = []
        for x, (gran, rows, cols, pad, scaling) in zip(xs, ALONG[case]):
            ragged = gran in ("sub1x128", "block128") and bool(cols % 128 or (gran == "block128" and rows % 128))
            p = B.make_params(rows, cols, gran, ld=cols + pad, scaling=scaling, ragged=ragged)
            out = B.alloc_outputs(p, dev, bf16_fill=0x1234)
            out.workspace = None
            for n in NAMES:
                t = getattr(out, n)
                if t is not None and n != "bf16":
                    t.view(torch.uint8).fill_(0x5A)
            got.append((p, x, out, torch.full((B.STATS_BYTES,), 0x5A, dtype=torch.uint8, device=dev) if counted else None, None))
        return got

    xs = []
    for k, (gran, rows, cols, pad, scaling) in enumerate(ALONG[case]):
        x = torch.randn((rows, cols + pad), generator=gen, device=dev)
        tiny = torch.rand((rows, (cols + pad + 127) // 128), generator=gen, device=dev).repeat_interleave(128, 1)[:, :cols + pad] < 0.2
        x = torch.where(tiny & (torch.rand(x.shape, generator=gen, device=dev) < 0.5), x * 1e-8, x).to(torch.bfloat16)
        if gran == "sub1x128":
            x[rows // 2, cols // 2] = float("inf")
        xs.append(x[:, :cols])
    want = entries()
    for e in want:
        _run(B, [e])
    for polls in (None, 0):
        print(f"[stream] along {case} counted={counted} polls={polls}", flush=True)
        got = entries()
        _run(B, got, polls)
        for k, (a, b) in enumerate(zip(want, got)):
            for n in NAMES:
                u, v = getattr(a[2], n), getattr(b[2], n)
                if u is None:
                    continue
                if n == "err_sum":      # other kernels alone, so another order: binary32 chains of up to 32 terms and steps in each
                    assert torch.allclose(u, v, rtol=32 * 2.0 ** -24, atol=0.0), (case, k)
                else:
                    assert torch.equal(u.view(torch.uint8), v.view(torch.uint8)), (case, k, n)
            if counted:
                s, t = B.read_stats(a[3]), B.read_stats(b[3])
                for key in s:
                    if key in ("err_sum_total", "mean_err"):
                        assert s[key] == t[key] or abs(s[key] - t[key]) <= 32 * 2.0 ** -24 * abs(s[key]), (case, k, key)
                    elif key != "flags":                                                    # (which says how, not what)
                        assert s[key] == t[key], (case, k, key)


# rows and columns of linear layers: waves, workgroups, one row; whole tiles, ragged ones, a single column chunk
PAIRS = [[(64, 256), (256, 256)], [(333, 4104), (1, 8), (512, 1000)], [(5, 16384), (1027, 1000), (128, 128), (1280, 640)], [(2048, 4096), (4096, 2048)]]


@pytest.mark.parametrize("fake", [False, True])
@pytest.mark.parametrize("scope", ["tensor", "partition"])
@pytest.mark.parametrize("scaling", ["gam", "fp32_amax", "e8m0"])
@pytest.mark.parametrize("case", range(len(PAIRS)))
def test_rows_and_columns_together(case, scaling, scope, fake):
    """Every operand by rows and by columns in one call: the outputs of each alone."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(31 + case)
    ops = []
    for k, (rows, cols) in enumerate(PAIRS[case]):
        x = torch.randn((rows, cols), generator=gen, device=dev)
        x = (x * torch.where(torch.rand(x.shape, generator=gen, device=dev) < (0.0, 0.3, 0.035)[k % 3], 1e-9, 1.0)).to(torch.bfloat16)
        if k == 1:
            x[0, cols // 2] = float("inf")
        ops += [(x, "channel_row"), (x, "channel_col")]

    def entries():
        got = []
        for x, gran in ops:
            p = B.make_params(*x.shape, gran, scope, "mean_rel_err", 0.045, scaling=scaling)
            out = B.alloc_outputs(p, dev, want_bf16=not fake, want_fp8=not fake, bf16_fill=0x1234)
            out.workspace = None
            for n in NAMES:
                t = getattr(out, n)
                if t is not None and n != "bf16":
                    t.view(torch.uint8).fill_(0x5A)
            got.append((p, x, out, None if fake else torch.full((B.STATS_BYTES,), 0x5A, dtype=torch.uint8, device=dev),
                        torch.full(x.shape, 3.0, dtype=torch.bfloat16, device=dev) if fake else None))
        return got

    want = entries()
    for e in want:
        _run(B, [e])
    for polls in (None, 0):
        print(f"[stream] rows and columns {case} {scaling} {scope} fake={fake} polls={polls}", flush=True)
        got = entries()
        _run(B, got, polls)
        for k, (a, b) in enumerate(zip(want, got)):
            for n in NAMES:
                u, v = getattr(a[2], n), getattr(b[2], n)
                assert (u is None) == (v is None) and (u is None or torch.equal(u.view(torch.uint8), v.view(torch.uint8))), (case, k, n)
            if fake:
                assert torch.equal(a[4].view(torch.int16), b[4].view(torch.int16)), (case, k)
            else:
                s, t = B.read_stats(a[3]), B.read_stats(b[3])
                for key in s:
                    assert s[key] == t[key] or (isinstance(s[key], float) and abs(s[key] - t[key]) <= 1e-12 * abs(s[key])), (case, k, key)
