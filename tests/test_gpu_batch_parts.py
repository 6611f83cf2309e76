"""Batches whose twice-read operands exceed the Infinity Cache are mostly taken in parts of at most 256 MB: every operand must come out
as from a call of its own, whichever part it falls into and whatever shares its launches."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _operand(rows, cols, seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x = torch.randn((rows, cols), generator=g, device=dev) * 1e-3
    x.mul_(torch.where(torch.rand((rows, cols // 128, 1), generator=g, device=dev) < 0.1 * (seed % 2), 1e-6, 1.0).expand(-1, -1, 128).reshape(rows, cols))
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("scaling, scope", [("gam", "tensor"), ("gam", "partition"), ("fp32_amax", "partition")])
def test_parts_equal_single_calls(scaling, scope):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    # two parts of the GAM operands and of the per-tensor ones: 117 + 100 MB fit one part, the third does not; columns share one set of launches
    shapes = [("block128", 4096, 14336), ("channel_row", 12288, 4096), ("block64", 4096, 8192), ("sub1x128", 8192, 8192),
              ("channel_col", 4096, 14336), ("channel_col", 8192, 8192), ("channel_col", 1024, 8192),
              ("tensor", 4096, 14336), ("tensor", 12288, 4096), ("tensor", 8192, 4096), ("tensor", 128, 256)]
    entries, singles = [], []
    for i, (gran, rows, cols) in enumerate(shapes):
        x = _operand(rows, cols, i, dev)
        p = B.make_params(rows, cols, gran, scope, "mean_rel_err", 0.045, scaling=scaling)
        outs = [B.alloc_outputs(p, dev, bf16_fill=0x5A5A) for _ in range(2)]
        st = [torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev) for _ in range(2)]
        entries.append((p, x, outs[0], st[0]))
        singles.append((p, x, outs[1], st[1]))
    items = B.make_batch(entries)
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
    for _ in range(2):
        B.mor_analyze_quantize_batch(items, 1e-2, ws)
    for p, x, out, st in singles:
        B.mor_analyze_quantize(p, x, out)
        B.mor_select_stats(p, out.err_sum, out.nnz, out.mask, 1e-2, st)
    torch.cuda.synchronize()
    kept = 0
    for (gran, rows, cols), (_, _, a, sa), (_, _, b, sb) in zip(shapes, entries, singles):
        for f in ("fp8", "bf16", "scale", "amax", "nnz", "mask", "scale_e8m0", "group_mantissa"):
            u, v = getattr(a, f), getattr(b, f)
            assert (u is None and v is None) or torch.equal(u.view(torch.uint8), v.view(torch.uint8)), (gran, rows, cols, f)
        # binary32 sums of at most 2^24 terms each rounded once per addition of a lane's chain (<= 4096 long), then binary64
        assert torch.allclose(a.err_sum.double(), b.err_sum.double(), rtol=1e-6, atol=0), (gran, rows, cols)
        got, want = B.read_stats(sa), B.read_stats(sb)
        for k in want:
            if k not in ("flags", "err_sum_total", "mean_err"):
                assert got[k] == want[k], (gran, rows, cols, k)
        kept += int((b.mask == 1).sum())
    assert kept > 0


@pytest.mark.parametrize("crit", ["mean_rel_err", "e4m3_vs_e5m2"])
@pytest.mark.parametrize("rows, cols", [(1, 128), (255, 128), (256, 128), (257, 128), (1025, 128), (2048, 128 * 129)])
def test_tensor_level_statistics(crit, rows, cols):
    """Statistics gathered by the reduce pass of a tensor-level decision: one block, a last lane or wave that is not full, one and
    more than one workgroup, more blocks than one round of all workgroups."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for seed in (0, 1):                    # kept in E4M3 and in BF16 under Eq. 2
        x = _operand(rows, cols, seed, dev)
        p = B.make_params(rows, cols, "sub1x128", "tensor", crit, 0.0238)
        out = B.alloc_outputs(p, dev, bf16_fill=0x5A5A)
        st = [torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev) for _ in range(2)]
        items = B.make_batch([(p, x, out, st[0])])
        ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
        B.mor_analyze_quantize_batch(items, 0.05, ws)
        B.mor_select_stats(p, out.err_sum, out.nnz, out.mask, 0.05, st[1])
        got, want = (B.read_stats(s) for s in st)
        for k in want:
            if k in ("err_sum_total", "mean_err"):       # binary64 sums of the same terms in another order
                assert got[k] == pytest.approx(want[k], rel=1e-12)
            else:
                assert got[k] == want[k], (k, got[k], want[k])
