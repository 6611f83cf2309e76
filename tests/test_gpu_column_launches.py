"""Per-channel columns: the quantize pass of a launch of at most 2048 workgroups forms the column scales itself, those of a larger one come
from a launch of their own; a tensor-level decision takes its sums from the strips in the reduce pass of all such operands.  Sizes on
both sides of the line and where the number of strips fills or crosses a round of 16 (scales) or 8 (sums) loads.  Tall operands, whose strips take long to read one after another, get launches of their own for the sums
and, where many workgroups would repeat the reads, for the scales."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu

# strips x tiles: 1 x 1, one row short of two strips, 8, 9, 16, 17, 33 strips; then 2048 and 2049 workgroups in the launch
SHAPES = [(8, 8), (128, 128), (255, 136), (1024, 128), (1025, 72), (2048, 256), (2049, 128), (4224, 128), (16, 2048 * 128), (16, 2049 * 128)]


def _input(rows, cols, kind):
    if kind == "grad":
        return W.gradient(rows, -(-cols // 128) * 128, 7)[:, :cols].copy()
    x = W.outlier_normal(rows, cols, 7)
    x[:, ::5] = np.where(np.arange(rows)[:, None] % 9 == 0, 0x0100, x[:, ::5])          # every fifth column: a ninth of it flushes
    x[:, 3] = 0
    return x


@pytest.mark.parametrize("rows, cols", SHAPES)
@pytest.mark.parametrize("scope, crit, scaling, formats", [("partition", "mean_rel_err", "fp32_amax", "e4m3|bf16"), ("partition", "mean_rel_err", "gam", "e4m3|bf16"),
                                                           ("partition", "e4m3_vs_e5m2", "e8m0", "e4m3|e5m2|bf16"), ("tensor", "mean_rel_err", "gam", "e4m3|bf16"),
                                                           ("tensor", "e4m3_vs_e5m2", "fp32_amax", "e4m3|bf16")])
def test_columns(rows, cols, scope, crit, scaling, formats):
    import parity
    for kind in ("normal", "grad"):
        x = _input(rows, cols, kind)
        parity.compare(x, "channel_col", scope, crit, scaling=scaling, formats=formats, ragged=True, label=kind)
        if rows * cols <= 1 << 20:
            parity.compare_fake(x, "channel_col", scope, crit, scaling=scaling, formats=formats, ragged=True)


@pytest.mark.parametrize("rows, cols", [(255, 136), (1025, 72), (2049, 384)])
@pytest.mark.parametrize("crit", ["mean_rel_err", "e4m3_vs_e5m2"])
def test_tensor_level_sums_with_and_without_statistics(oracle, rows, cols, crit):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    x = torch.from_numpy(_input(rows, cols, "normal").view(np.int16)).to(dev)
    p = B.make_params(rows, cols, "channel_col", "tensor", crit, scaling="gam", ragged=True)
    bare, told = B.alloc_outputs(p, dev, bf16_fill=0), B.alloc_outputs(p, dev, bf16_fill=0)
    st = torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)
    for out, s in ((bare, None), (told, st)):
        items = B.make_batch([(p, x, out, s)])
        ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
        B.mor_analyze_quantize_batch(items, 1e-2, ws)
    torch.cuda.synchronize()
    for k in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask") + (("err5_sum",) if bare.err5_sum is not None else ()):
        assert torch.equal(getattr(bare, k), getattr(told, k)), k
    got = B.read_stats(st)
    want = oracle.select_stats(told.err_sum.cpu().numpy(), told.nnz.cpu().numpy().view(np.uint32), told.mask.cpu().numpy(), rows, cols,
                               "channel_col", 0.045, 1e-2, ragged=True)
    for k in ("n_part", "n_fp8_part", "n_bf16_part", "n_elem_fp8", "n_elem_bf16", "nnz_total", "hist", "n_near_threshold"):
        assert got[k] == want[k], k
    assert got["err_sum_total"] == pytest.approx(want["err_sum_total"], rel=1e-12)


# 96 and 97 strips, 128 strips in 640 workgroups, 129 strips in 129 and in 645, two operands of the latter
@pytest.mark.parametrize("rows, cols, k, combines", [(12288, 128, 1, (0, 1)), (12289, 128, 1, (1, 1)), (16384, 640, 1, (1, 1)), (16385, 128, 1, (1, 1)),
                                                     (16385, 640, 1, (2, 1)), (16385, 640, 2, (2, 2))])
@pytest.mark.parametrize("crit, scaling", [("mean_rel_err", "gam"), ("mean_rel_err", "fp32_amax"), ("e4m3_vs_e5m2", "fp32_amax")])
@pytest.mark.parametrize("scope", ["tensor", "partition"])
def test_tall_columns(rows, cols, k, combines, crit, scaling, scope):
    """combines: launches that combine strips (scales, sums) with a tensor-level decision, and with decisions and flush counts per column."""
    import parity
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for kind in ("normal", "grad"):
        x = _input(rows, cols, kind)
        xd = torch.from_numpy(x.view(np.int16)).to(dev)
        p = B.make_params(rows, cols, "channel_col", scope, crit, scaling=scaling, ragged=True)
        entries = [(p, xd, B.alloc_outputs(p, dev, bf16_fill=parity.FILL), torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)) for _ in range(k)]
        items = B.make_batch(entries)
        ev = B.HipEvents()
        prof = ev.new_profile(B.MOR_PROFILE_MAX)
        B.mor_analyze_quantize_batch(items, 1e-5, torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev), prof)
        torch.cuda.synchronize()
        names = [B.KERNEL_NAMES[prof.kernel[i]] for i in range(prof.count)]
        ev.destroy()
        counts = scope == "partition" and crit == "mean_rel_err"          # else a tall operand's scales are as with a tensor-level decision
        want = combines[1] if counts else combines[0] + (1 if scope == "partition" and combines[0] == 0 else 0)
        assert names.count("column_combine") == want, names
        parity.compare(x, "channel_col", scope, crit, scaling=scaling, ragged=True, label=kind, gpu=(p, entries[0][2]))
        for _, _, out, st in entries[1:]:
            for name in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask"):
                assert torch.equal(getattr(out, name), getattr(entries[0][2], name)), name
            assert torch.equal(st, entries[0][3])
        parity.compare_fake(x[:, :128], "channel_col", scope, crit, scaling=scaling, ragged=True)
