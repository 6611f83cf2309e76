"""Operands whose rows are longer than the operand is wide, and 1x128 operands with ragged edges: the chunk and block
addresses of these kernels come from divisions by the row's length, so the sizes are those where a tile (2048 16-byte chunks)
or a unit (32 blocks) ends inside a row, spans many rows, or ends at the operand's last element.  Everything is compared with
the oracle, bit for bit but for the error sums; outputs with padded rows of their own must leave the padding alone."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu

# rows, cols, ld: one chunk per row; rows shorter and longer than the 256 chunks of one step; a tile that ends with a row;
# one element more than a tile; rows longer than a tile
SHAPES = [(5000, 8, 16), (700, 24, 40), (1030, 136, 272), (257, 2040, 4096), (256, 2048, 2056), (9, 2056, 2064), (33, 16384, 16392),
          (3, 40000, 40008)]


def _operand(rows, cols, ld, kind, seed=5):
    width = -(-ld // 128) * 128
    if kind == "grad":
        return W.gradient(rows, width, seed)[:, :ld].copy()
    if kind == "half":
        return W.gradient(rows, width, seed, tiny_frac=0.3, tiny_half=True)[:, :ld].copy()
    x = W.outlier_normal(rows, ld, seed)
    if kind == "large":                    # amax >= 2^25: the element path that needs no assumption
        x[rows // 2, cols // 2] = 0x4D00
    if kind == "inf":
        x[0, cols - 1] = 0x7F80
    return x


@pytest.mark.parametrize("gran", ["tensor", "sub1x128"])
@pytest.mark.parametrize("rows, cols, ld", SHAPES)
def test_padded_rows(gran, rows, cols, ld):
    import parity
    ragged = gran == "sub1x128" and cols % 128 != 0
    for kind in ("normal", "grad", "half", "large", "inf"):
        parity.compare(_operand(rows, cols, ld, kind), gran, cols=cols, ragged=ragged, label=kind)
    parity.compare(_operand(rows, cols, ld, "half"), gran, crit="e4m3_vs_e5m2", cols=cols, ragged=ragged, scaling="gam")
    parity.compare_fake(_operand(rows, cols, ld, "half"), gran, cols=cols, ragged=ragged)


@pytest.mark.parametrize("rows, cols", [(1, 8), (1, 136), (31, 128), (33, 128), (3, 1400), (65, 4104), (127, 16)])
def test_ragged_sub_rows(rows, cols):
    """Dense 1x128 operands whose last block or last unit is not whole, with bands of rows as GAM groups too."""
    import parity
    for kind in ("half", "large"):
        x = _operand(rows, cols, cols, kind)
        parity.compare(x, "sub1x128", cols=cols, ragged=cols % 128 != 0, label=kind)
        parity.compare(x, "sub1x128", scope="tensor", cols=cols, ragged=cols % 128 != 0, scaling="gam", gam_group_rows=7)


@pytest.mark.parametrize("gran", ["tensor", "sub1x128"])
@pytest.mark.parametrize("cols, ld", [(8, 4194304), (8, 2097152), (136, 3000000)])
def test_rows_too_long_for_tile_offsets(gran, cols, ld):
    """A few columns of very long rows: a tile of the operand spans 2 GB or more, or a row is 2^22 elements."""
    import parity
    rows = 5 if ld == 4194304 else 520
    dev = torch.device("cuda:0")
    from paper_2512_22804_amd import binding as B
    small = _operand(rows, cols, cols, "half")
    buf = torch.zeros(rows * ld, dtype=torch.int16, device=dev).view(rows, ld)
    buf[:, :cols] = parity.to_dev(small)
    p = B.make_params(rows, cols, gran, ld=ld, ragged=gran == "sub1x128")
    q = B.make_params(rows, cols, gran, ld=cols, ragged=gran == "sub1x128")
    a, b = (B.alloc_outputs(x, dev, bf16_fill=parity.FILL) for x in (p, q))
    B.mor_analyze_quantize(p, buf, a)
    B.mor_analyze_quantize(q, parity.to_dev(small), b)
    torch.cuda.synchronize()
    for f in ("fp8", "bf16", "scale", "amax", "nnz", "mask"):
        assert torch.equal(getattr(a, f), getattr(b, f)), f
    assert torch.allclose(a.err_sum, b.err_sum, rtol=1e-5, atol=0)      # the error sums' own bound


@pytest.mark.parametrize("gran", ["tensor", "sub1x128"])
@pytest.mark.parametrize("rows, cols", [(300, 200), (70, 3000)])
def test_padded_outputs_and_statistics(oracle, gran, rows, cols):
    """Payload and fallback buffers with rows of their own length; statistics of the lone operand (ragged blocks counted with
    their real sizes) and of two operands in one call."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    near = 1e-2
    entries, keep = [], []
    for seed in (1, 2):
        xb = _operand(rows, cols, cols + 24, "half", seed)
        p = B.make_params(rows, cols, gran, ld=cols + 24, ragged=True)
        out = B.alloc_outputs(p, dev)
        wide8 = torch.full((rows, cols + 8), 0xA5, dtype=torch.uint8, device=dev)
        wideb = torch.full((rows, cols + 16), 0x5A5A, dtype=torch.int16, device=dev)
        out.fp8, out.bf16 = wide8[:, :cols], wideb[:, :cols]
        st = torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)
        entries.append((p, parity.to_dev(xb), out, st))
        keep.append((xb, wide8, wideb))
    for group in ([0], [0, 1]):
        items = B.make_batch([entries[i] for i in group])
        ws = torch.full((max(16, B.mor_batch_workspace_bytes(items)),), 0xA7, dtype=torch.uint8, device=dev)
        for i in group:
            keep[i][1].fill_(0xA5); keep[i][2].fill_(0x5A5A); entries[i][3].fill_(0xEE)
        B.mor_analyze_quantize_batch(items, near, ws)
        torch.cuda.synchronize()
        for i in group:
            xb, wide8, wideb = keep[i]
            p, x, out, st = entries[i]
            a = oracle.analyze_quantize(xb, gran, "partition", "mean_rel_err", 0.045, bf16_fill=0x5A5A, ld=cols + 24, cols=cols, ragged=True)
            assert np.array_equal(out.mask.cpu().numpy(), a.mask)
            assert np.array_equal(wide8[:, :cols].cpu().numpy(), a.fp8) and bool((wide8[:, cols:] == 0xA5).all())
            assert np.array_equal(wideb[:, :cols].cpu().numpy().view(np.uint16), a.bf16) and bool((wideb[:, cols:] == 0x5A5A).all())
            got = B.read_stats(st)
            want = oracle.select_stats(out.err_sum.cpu().numpy(), a.nnz, a.mask, rows, cols, gran, 0.045, near, ragged=True)
            for k in ("n_part", "n_fp8_part", "n_bf16_part", "n_e5m2_part", "n_elem_fp8", "n_elem_bf16", "n_elem_e5m2", "nnz_total", "hist"):
                if k in want:
                    assert got[k] == want[k], (k, got[k], want[k])


@pytest.mark.parametrize("rows, cols, ld", SHAPES + [(1, 8, 8), (33, 128, 128), (65, 4104, 4104), (31, 1400, 1400)])
def test_rows_form_of_the_unit_kernel(rows, cols, ld):
    """Two or more such 1x128 operands in a call share launches of the kernel that works through units of 32 blocks (a small
    operand alone takes the general kernel); payload with both criteria, fake quantization, bands of rows as GAM groups."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for kind in ("half", "large", "inf"):
        xb = _operand(rows, cols, ld, kind)
        for kw in ({}, {"crit": "e4m3_vs_e5m2"}, {"scaling": "gam", "gam_group_rows": 5}, {"scaling": "e8m0", "scope": "tensor"}):
            p = B.make_params(rows, cols, "sub1x128", ld=ld, ragged=cols % 128 != 0, threshold=0.045, **kw)
            outs = [parity.guarded_outputs(p, dev, bf16_fill=parity.FILL) for _ in range(2)]
            fakes = [parity.guarded_outputs(p, dev, want_bf16=False, want_fp8=False) for _ in range(2)]
            ys = [torch.full((rows, cols), 0x5A5A, dtype=torch.int16, device=dev) for _ in range(2)]
            x = parity.to_dev(xb)
            items = B.make_batch([(p, x, o, None) for o, _ in outs] + [(p, x, o, None, y) for (o, _), y in zip(fakes, ys)])
            ws = torch.full((max(16, B.mor_batch_workspace_bytes(items)),), 0xFF, dtype=torch.uint8, device=dev)
            B.mor_analyze_quantize_batch(items, 1e-2, ws)
            torch.cuda.synchronize()
            for _, guards in outs + fakes:
                guards.check()
            parity.compare(xb, "sub1x128", cols=cols, ragged=cols % 128 != 0, label=kind, gpu=(p, outs[1][0]), **kw)
            o, f = outs[0][0], fakes[1][0]
            y = torch.full_like(ys[0], 0x1111)
            B.mor_dequantize(p, o.fp8, o.scale, o.mask, o.bf16, y)
            assert torch.equal(ys[1], y) and torch.equal(f.mask, o.mask) and torch.equal(f.err_sum, o.err_sum)


def test_rows_form_alone_with_statistics(oracle):
    """One operand large enough for that kernel alone, ragged, with statistics (BF16 blocks of the last column are narrower)."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    rows, cols = 24581, 520
    xb = _operand(rows, cols, cols, "half")
    p = B.make_params(rows, cols, "sub1x128", ragged=True)
    out = B.alloc_outputs(p, dev, bf16_fill=parity.FILL)
    st = torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)
    items = B.make_batch([(p, parity.to_dev(xb), out, st)])
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
    B.mor_analyze_quantize_batch(items, 1e-2, ws)
    torch.cuda.synchronize()
    r = parity.compare(xb, "sub1x128", cols=cols, ragged=True, gpu=(p, out))
    got, a = B.read_stats(st), r["oracle"]
    assert 0 < got["n_bf16_part"] < got["n_part"]
    want = oracle.select_stats(out.err_sum.cpu().numpy(), a.nnz, out.mask.cpu().numpy(), rows, cols, "sub1x128", 0.045, 1e-2, ragged=True)
    for k in ("n_part", "n_fp8_part", "n_bf16_part", "n_e5m2_part", "n_elem_fp8", "n_elem_bf16", "n_elem_e5m2", "nnz_total", "hist"):
        if k in want:
            assert got[k] == want[k], (k, got[k], want[k])


@pytest.mark.parametrize("rows, cols, ld", [(1, 8, 16), (63, 8, 16), (64, 8, 16), (65, 64, 72), (1, 4096, 8192), (1, 4104, 8208), (2, 4088, 4096),
                                            (512, 8192, 8200), (513, 8192, 8200)])
def test_small_lone_operands(rows, cols, ld):
    """Per-tensor operands with padded rows up to 2^19 chunks have kernels of their own where they are alone in the call: tiles of 512
    chunks, one chunk to many tiles, the largest of the range and the next larger one; with and without statistics."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for kind, kw in (("normal", {}), ("grad", {}), ("half", {"crit": "e4m3_vs_e5m2", "formats": "e4m3|e5m2|bf16"}), ("large", {"scaling": "gam"}),
                     ("half", {"crit": "e4m3_vs_e5m2"}), ("inf", {"scaling": "e8m0"})):
        x = _operand(rows, cols, ld, kind)
        r = parity.compare(x, "tensor", cols=cols, label=kind, **kw)
        if "formats" not in kw:
            parity.compare_fake(x, "tensor", cols=cols, **kw)
        p = r["params"]
        out = B.alloc_outputs(p, dev, bf16_fill=parity.FILL)
        st = [torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev) for _ in range(2)]
        xd = parity.to_dev(x)
        items = B.make_batch([(p, xd, out, st[0])])
        ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
        B.mor_analyze_quantize_batch(items, 1e-2, ws)
        B.mor_select_stats(p, out.err_sum, out.nnz, out.mask, 1e-2, st[1])
        got, want = (B.read_stats(s) for s in st)
        assert got == want
        for f in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask"):
            assert torch.equal(getattr(out, f), getattr(r["gpu"], f)), (kind, f)


@pytest.mark.parametrize("rows, cols, ld, frac, proven", [(520, 1024, 1032, 0.2, 1), (520, 1024, 1032, 0.0, 0), (4096, 2048, 2056, 0.2, 1),
                                                          (4096, 2048, 2056, 0.0, 0)])
def test_padded_rows_prove_their_decision(rows, cols, ld, frac, proven):
    """The statistics of operands with padded rows do not report whether the BF16 decision was proven by the amax pass, so the
    workspace is looked at: behind its partial records stand the operand's amax pattern and the outcome of the proof."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(int(frac * 10))
    v = np.exp2(rng.uniform(-3.0, 3.0, size=(rows, ld))).astype(np.float32)
    v[rng.random((rows, ld)) < frac] = np.float32(2.0 ** -40)
    v[3, 5] = 8.0
    x = torch.from_numpy(W.f32_to_bf16_bits(v).view(np.int16)).to(dev)
    p = B.make_params(rows, cols, "tensor", ld=ld)
    out = B.alloc_outputs(p, dev, bf16_fill=0x5A5A)
    B.mor_analyze_quantize(p, x[:, :cols], out)
    at = (4 * 768 + 3 * 4 * 16384) // 4                    # 768 amax records, 16 384 of each of three sums
    words = out.workspace.view(torch.int32)[at:at + 2].tolist()
    assert words == [0x4100, proven] and int(out.mask[0]) == proven


@pytest.mark.parametrize("rows, cols, ld", SHAPES)
def test_grouped_padded_tensors(rows, cols, ld):
    """Two or more per-tensor operands with padded rows in a call, however small, share the grouped kernels (tiles of 2048 chunks)."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for kind in ("normal", "grad", "half", "large", "inf"):
        xb = _operand(rows, cols, ld, kind)
        for kw in ({}, {"crit": "e4m3_vs_e5m2", "scaling": "gam"}, {"crit": "e4m3_vs_e5m2", "formats": "e4m3|e5m2|bf16"}):
            p = B.make_params(rows, cols, "tensor", ld=ld, threshold=0.045, **kw)
            outs = [parity.guarded_outputs(p, dev, bf16_fill=parity.FILL) for _ in range(2)]
            fakes = [parity.guarded_outputs(p, dev, want_bf16=False, want_fp8=False) for _ in range(2)]
            ys = [torch.full((rows, cols), 0x5A5A, dtype=torch.int16, device=dev) for _ in range(2)]
            x = parity.to_dev(xb)
            items = B.make_batch([(p, x, o, None) for o, _ in outs] + [(p, x, o, None, y) for (o, _), y in zip(fakes, ys)])
            ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xFF, dtype=torch.uint8, device=dev)
            B.mor_analyze_quantize_batch(items, 1e-2, ws)
            torch.cuda.synchronize()
            for _, guards in outs + fakes:
                guards.check()
            for o, _ in outs:
                parity.compare(xb, "tensor", cols=cols, label=kind, gpu=(p, o), **kw)
            o = outs[0][0]
            want = torch.full_like(ys[0], 0x1111)
            B.mor_dequantize(p, o.fp8, o.scale, o.mask, o.bf16, want)
            for (f, _), y in zip(fakes, ys):
                assert torch.equal(y, want) and torch.equal(f.mask, o.mask) and torch.equal(f.err_sum, o.err_sum)


@pytest.mark.parametrize("cols, ld", [(8, 2097152), (136, 3000000)])
def test_grouped_rows_too_long_for_tile_offsets(cols, ld):
    import parity
    from paper_2512_22804_amd import binding as B
    rows = 520
    dev = torch.device("cuda:0")
    small = parity.to_dev(_operand(rows, cols, cols, "half"))
    buf = torch.zeros(rows * ld, dtype=torch.int16, device=dev).view(rows, ld)
    buf[:, :cols] = small
    p, q = (B.make_params(rows, cols, "tensor", ld=n) for n in (ld, cols))
    a = [B.alloc_outputs(p, dev, bf16_fill=parity.FILL) for _ in range(2)]
    b = B.alloc_outputs(q, dev, bf16_fill=parity.FILL)
    items = B.make_batch([(p, buf, o, None) for o in a])
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xFF, dtype=torch.uint8, device=dev)
    B.mor_analyze_quantize_batch(items, 1e-2, ws)
    B.mor_analyze_quantize(q, small, b)
    torch.cuda.synchronize()
    for o in a:
        for f in ("fp8", "bf16", "scale", "amax", "nnz", "mask"):
            assert torch.equal(getattr(o, f), getattr(b, f)), f
        assert torch.allclose(o.err_sum, b.err_sum, rtol=1e-5, atol=0)      # the error sums' own bound
