"""A small per-tensor operand alone in its call takes two launches: the workgroup of the quantize pass that finishes last decides, and the
others, which hold their tile in registers, copy it (or rewrite it in E5M2) when they are told.  The sizes are those where the number
of tiles, of first tickets or the tile size changes; the decision falls each way, with and without a proof from the amax pass."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu

# chunks of 8 elements: one; a tile of 512 and one more; 16 tiles (one first ticket) and one chunk more; Eq. 3's and Eq. 2's changes of
# the tile size and of the kernels
SHAPES = [(1, 8), (8, 512), (9, 456), (512, 128), (513, 128), (683, 3072), (1024, 2056), (1024, 4096), (1025, 4096), (2048, 4096), (2049, 4096)]


@pytest.mark.parametrize("rows, cols", SHAPES)
@pytest.mark.parametrize("kind, crit, th", [("normal", "mean_rel_err", 0.045),        # kept in E4M3
                                            ("normal", "mean_rel_err", 0.001),        # BF16 without a proof
                                            ("grad", "mean_rel_err", 0.045),          # BF16, proven where the operand is large enough
                                            ("grad", "e4m3_vs_e5m2", 0.045), ("large", "e4m3_vs_e5m2", 0.045)])
def test_lone_small_operand(rows, cols, kind, crit, th):
    import parity
    x = W.gradient(rows, -(-cols // 128) * 128, 3)[:, :cols].copy() if kind == "grad" else W.outlier_normal(rows, cols, 3)
    if kind == "large":
        x[rows // 2, cols // 2] = 0x4D00
    parity.compare(x, "tensor", crit=crit, threshold=th, label=f"{kind} {crit} {th}", scaling="gam" if kind == "large" else "fp32_amax")
    if rows * cols <= 1 << 22:
        parity.compare_fake(x, "tensor", crit=crit, threshold=th)


@pytest.mark.parametrize("rows, cols", [(9, 456), (512, 128), (1024, 2056), (1025, 4096)])
@pytest.mark.parametrize("kind, crit", [("normal", "mean_rel_err"), ("grad", "e4m3_vs_e5m2"), ("large", "e4m3_vs_e5m2")])
def test_alone_as_in_a_batch(rows, cols, kind, crit):
    """Dense operands give the same bits alone as beside another one, in whose call the kernels for several operands take them."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    x = W.gradient(rows, -(-cols // 128) * 128, 6)[:, :cols].copy() if kind == "grad" else W.outlier_normal(rows, cols, 6)
    if kind == "large":
        x[0, 3] = 0x4D00
    xd = torch.from_numpy(x.view(np.int16)).to(dev)
    p = B.make_params(rows, cols, "tensor", crit=crit)
    alone, beside, other = (B.alloc_outputs(p, dev, bf16_fill=0) for _ in range(3))
    B.mor_analyze_quantize(p, xd, alone)
    items = B.make_batch([(p, xd, beside, None), (p, xd.clone(), other, None)])
    ws = torch.empty(B.mor_batch_workspace_bytes(items), dtype=torch.uint8, device=dev)
    B.mor_analyze_quantize_batch(items, 1e-5, ws)
    torch.cuda.synchronize()
    for k in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask") + (("err5_sum",) if alone.err5_sum is not None else ()):
        assert torch.equal(getattr(alone, k), getattr(beside, k)), k


@pytest.mark.parametrize("rows, cols, ld", [(513, 128, 128), (1024, 2056, 2064)])
def test_three_types(rows, cols, ld):
    import parity
    wide = W.outlier_normal(rows, ld, 4)
    wide[::7] = (wide[::7] & 0x8000) | 0x3200           # magnitudes E4M3 flushes and E5M2 holds
    for x in (wide, W.gradient(rows, -(-ld // 128) * 128, 4)[:, :ld].copy()):
        parity.compare(x, "tensor", crit="e4m3_vs_e5m2", formats="e4m3|e5m2|bf16", cols=cols)
        parity.compare_fake(x, "tensor", crit="e4m3_vs_e5m2", formats="e4m3|e5m2|bf16", cols=cols)


def test_on_a_busy_chip_and_in_a_graph():
    """The workgroups that wait to be told find their places late while another stream keeps the chip busy; a captured call runs again
    and again on one workspace."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    x = torch.from_numpy(W.outlier_normal(2048, 4096, 5).view(np.int16)).to(dev)
    p = B.make_params(2048, 4096, "tensor", threshold=0.001)
    want = B.alloc_outputs(p, dev, bf16_fill=0)
    B.mor_analyze_quantize(p, x, want)
    outs = [B.alloc_outputs(p, dev, bf16_fill=0) for _ in range(8)]
    big = torch.empty(1 << 28, dtype=torch.int32, device=dev)
    other = torch.empty_like(big)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(20):
            other.copy_(big)
    for out in outs:
        B.mor_analyze_quantize(p, x, out)
    torch.cuda.synchronize()
    same = lambda o: all(torch.equal(getattr(o, k), getattr(want, k)) for k in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask"))      # noqa: E731
    assert int(want.mask[0]) == 1 and torch.equal(want.bf16, x)
    assert all(same(o) for o in outs)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.mor_analyze_quantize(p, x, outs[0])
    for _ in range(3):
        outs[0].bf16.zero_()
        outs[0].mask.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert same(outs[0])
