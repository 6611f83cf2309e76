"""A small per-tensor operand alone in its call.  Most tests here: operands that end inside a wave of the amax pass.  Under Eq. 2 with a BF16 output that
pass also counts elements that are certain to flush, against the amax of a whole wave: lanes beyond the operand's end take part in that
reduction and bring nothing, and the amax itself comes from every lane that holds data."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu
LARGE = 0x4300                                            # 128.0, far above the rest


def _normal(rows, cols, ld, seed):
    x = W.outlier_normal(rows, ld, seed)
    x[(x & 0x7FFF) >= 0x4200] = 0x3F80                    # nothing else of that size (32 and above)
    return x


def _run(B, p, x, fake=False):
    out = B.alloc_outputs(p, x.device, bf16_fill=0)
    if fake:
        B.mor_fake_quantize(p, x, torch.empty_like(x), out)
    else:
        B.mor_analyze_quantize(p, x, out)
    return out


# an amax tile is 512 chunks of 8 elements, a wave takes 64 of the first 256 and the same of the second; above 768 tiles a workgroup
# takes several, and what it found in the first must not stand for the last
@pytest.mark.parametrize("tiles", [0, 20, 800])
@pytest.mark.parametrize("r", [1, 5, 7, 9, 15, 17, 63, 65, 255])
@pytest.mark.parametrize("padded", [False, True])
def test_largest_value_in_the_last_tile(tiles, r, padded):
    import parity
    from paper_2512_22804_amd import binding as B
    n = 512 * tiles + 256 + r
    rows, cols, ld = (n, 8, 24) if padded else (1, 8 * n, 8 * n)
    x = _normal(rows, cols, ld, r)
    xd = parity.to_dev(x)
    p = B.make_params(rows, cols, "tensor", ld=ld)
    last = 512 * tiles
    for at in sorted({last, last + min(4, r), last + r - 1, last + r, last + 255, last + 256, last + 256 + r // 2, n - 1}):
        pos = (at, 7) if padded else (0, 8 * at + 7)
        old = x[pos]
        x[pos] = LARGE
        xd[pos] = LARGE
        out = _run(B, p, xd)
        assert float(out.amax[0]) == 128.0 and float(out.scale[0]) == 3.5, (n, at)
        if at == n - 1 or (tiles == 20 and at >= n - r):
            parity.compare(x, "tensor", cols=cols, label=f"chunk {at} of {n}")
        x[pos] = old
        xd[pos] = int(old.view(np.int16))


@pytest.mark.parametrize("rows, cols, pad", [(1500, 2880, 0), (2049, 2304, 0), (4000, 1000, 0), (1000, 5000, 0), (1500, 2880, 40), (1000, 5000, 8)])
def test_largest_value_is_the_last(rows, cols, pad):
    import parity
    x = _normal(rows, cols, cols + pad, 2)
    x[rows - 1, cols - 1] = LARGE | 0x8000
    if pad:
        x[:, cols:] = 0x7F80                              # what lies between the rows is not the operand's
    parity.compare(x, "tensor", cols=cols)
    parity.compare_fake(x, "tensor", cols=cols)


@pytest.mark.parametrize("rows, cols, pad", [(700, 1000, 0), (700, 1000, 24), (1, 8, 0), (1500, 2880, 0)])
def test_all_zero(rows, cols, pad):
    import parity
    from paper_2512_22804_amd import binding as B
    x = np.zeros((rows, cols + pad), np.uint16)
    x[:, 1::2] = 0x8000                                   # both signs
    xd = parity.to_dev(x)
    for fake in (False, True):
        out = _run(B, B.make_params(rows, cols, "tensor", ld=cols + pad), xd, fake)
        assert float(out.amax[0]) == 0.0 and float(out.scale[0]) == 1.0 and int(out.nnz[0]) == 0 and int(out.mask[0]) == 0
    parity.compare(x, "tensor", cols=cols)


# 2^22 elements and more do not fit the rows of the kernels for lone operands; 2^23 are as many as those take
@pytest.mark.parametrize("cols", [(1 << 22) - 8, 1 << 22, (1 << 22) + 8, 5000 * 1000, 1 << 23])
@pytest.mark.parametrize("kind", ["normal", "grad"])
def test_one_long_row(cols, kind):
    """The same bits, and the same proof of a BF16 decision, as in rows of eight and as beside another operand."""
    import parity
    from paper_2512_22804_amd import binding as B
    x = W.gradient(1, -(-cols // 128) * 128, 8)[:, :cols].copy() if kind == "grad" else W.outlier_normal(1, cols, 8)
    xd = parity.to_dev(x)
    p, short = B.make_params(1, cols, "tensor"), B.make_params(cols // 8, 8, "tensor")

    def call(*operands):
        entries = []
        for q in operands:
            st = torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=xd.device)
            entries.append((q, xd, B.alloc_outputs(q, xd.device, bf16_fill=0), st))
        items = B.make_batch(entries)
        B.mor_analyze_quantize_batch(items, 1e-5, torch.empty(B.mor_batch_workspace_bytes(items), dtype=torch.uint8, device=xd.device))
        torch.cuda.synchronize()
        return entries[0][2], B.read_stats(entries[0][3])
    alone, stats = call(p)
    for other, other_stats in (call(short), call(p, p)):
        for k in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask"):
            assert torch.equal(getattr(alone, k).flatten(), getattr(other, k).flatten()), k
        assert stats == other_stats
    assert int(alone.mask[0]) == (kind == "grad") and stats["flags"] == (B.MOR_STATS_FLAG_FUSED_FALLBACK if kind == "grad" else 0)
    parity.compare(x, "tensor")


# small values in whole lanes (chunk modulo 256) of the amax pass have no large neighbour in their lane: no flush is certain, whatever their
# wave holds; small values in single chunks have one
@pytest.mark.parametrize("rows, cols", [(1, 2400), (128, 128), (255, 72), (600, 1000), (1024, 1024), (1500, 2880), (2048, 4096)])
@pytest.mark.parametrize("kind", ["lanes", "chunks", "few"])
def test_proof_alone_as_in_a_batch(rows, cols, kind):
    """The proof of a BF16 decision, which the statistics report and which leaves out a lean operand's payload."""
    import parity
    from paper_2512_22804_amd import binding as B
    n = rows * cols // 8
    x = _normal(rows, cols, cols, 11)
    chunks = x.reshape(n, 8)
    at = np.arange(n)
    small = at % 8 == 5 if kind == "lanes" else at // 256 % 8 == 3 if kind == "chunks" else at % 293 < 14
    chunks[small] = (chunks[small] & 0x8000) | 0x0110
    xd = parity.to_dev(x)
    p = B.make_params(rows, cols, "tensor", lean_fp8=True)

    def call(k):
        entries = []
        for _ in range(k):
            out = B.alloc_outputs(p, xd.device, bf16_fill=0)
            out.fp8.fill_(0xA7)
            entries.append((p, xd, out, torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=xd.device)))
        items = B.make_batch(entries)
        B.mor_analyze_quantize_batch(items, 1e-5, torch.empty(B.mor_batch_workspace_bytes(items), dtype=torch.uint8, device=xd.device))
        torch.cuda.synchronize()
        return entries[0][2], B.read_stats(entries[0][3])
    (alone, stats), (beside, beside_stats) = call(1), call(2)
    assert stats == beside_stats
    for k in ("fp8", "bf16", "scale", "amax", "err_sum", "nnz", "mask"):
        assert torch.equal(getattr(alone, k), getattr(beside, k)), k
    proven = stats["flags"] == B.MOR_STATS_FLAG_FUSED_FALLBACK
    assert bool((alone.fp8 == 0xA7).all()) == proven
    assert int(alone.mask[0]) == bool(small.any())
    if kind != "few":
        assert proven == (kind == "chunks" and n >= 2048)


# rows of 2^22 elements: chunk by chunk; 2^18 chunks, one more, 2^19 and one more
@pytest.mark.parametrize("chunks", [(1 << 18), (1 << 18) + 1, 1 << 19, (1 << 19) + 1])
@pytest.mark.parametrize("crit, formats, kind", [("mean_rel_err", "e4m3|bf16", "normal"), ("mean_rel_err", "e4m3|bf16", "grad"),
                                                 ("e4m3_vs_e5m2", "e4m3|bf16", "grad"), ("e4m3_vs_e5m2", "e4m3|e5m2|bf16", "grad")])
def test_rows_beyond_the_row_map(chunks, crit, formats, kind):
    import parity
    cols, ld = 8 * chunks, (1 << 22) + 128
    x = W.gradient(1, ld, 9) if kind == "grad" else W.outlier_normal(1, ld, 9)
    parity.compare(x, "tensor", crit=crit, formats=formats, cols=cols)
    parity.compare_fake(x, "tensor", crit=crit, formats=formats, cols=cols)


@pytest.mark.parametrize("rows", [512, 513, 1023, 1024, 1025])      # 4096 of 4104 columns: two chunks per lane of 256, of 512, eight of 256
@pytest.mark.parametrize("crit", ["mean_rel_err", "e4m3_vs_e5m2"])
@pytest.mark.parametrize("special", [None, 0x7F80, 0xFFC1])
def test_padded_rows_at_the_edges_of_the_shapes(rows, crit, special):
    import parity
    x = W.outlier_normal(rows, 4104, 12)
    if special is not None:
        x[rows // 2, 4095] = special
    parity.compare(x, "tensor", crit=crit, cols=4096)
    parity.compare_fake(x, "tensor", crit=crit, cols=4096)
