"""De-quantization in tiles of 1024 consecutive 16-byte chunks: operands smaller than a tile, one chunk beyond a tile, rows shorter
and longer than a tile, padded rows on either side, mixed masks with and without a fallback buffer, and rows too long for the
tiles' 32-bit offsets.  Every value against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8), (3, 24), (1025, 8), (64, 128), (127, 136), (5, 8200), (130, 2048), (2, 16384)]


def _analysed(oracle, rows, cols, gran, formats="e4m3|bf16", seed=3, **kw):
    x = W.gradient(rows, -(-cols // 128) * 128, seed, tiny_frac=0.4, tiny_half=True)[:, :cols].copy()
    crit = "e4m3_vs_e5m2" if formats != "e4m3|bf16" else "mean_rel_err"
    a = oracle.analyze_quantize(x, gran, "partition", crit, 0.045, bf16_fill=0x5A5A, ld=cols, cols=cols, ragged=True, formats=formats, **kw)
    return x, a, crit


@pytest.mark.parametrize("gran", ["tensor", "sub1x128", "block128", "block64", "channel_row"])
@pytest.mark.parametrize("formats", ["e4m3|bf16", "e4m3|e5m2|bf16"])
def test_tile_edges(oracle, gran, formats):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    for rows, cols in SHAPES:
        print(f"[dequant tiles] {gran} {formats} {rows}x{cols}", flush=True)
        x, a, crit = _analysed(oracle, rows, cols, gran, formats)
        p = B.make_params(rows, cols, gran, "partition", crit, 0.045, ragged=True, formats=formats)
        want = oracle.dequantize(a.fp8, a.scale, a.mask, a.bf16, gran, ragged=True)
        rng = np.random.default_rng(rows)
        for pad in (0, 8, 24):
            fp8 = torch.from_numpy(rng.integers(0, 256, (rows, cols + pad), dtype=np.uint8)).to(dev)
            bf16 = torch.full((rows, cols + 2 * pad), 0x1234, dtype=torch.int16, device=dev)
            y = torch.full((rows, cols + pad), 0x5A5A, dtype=torch.int16, device=dev)
            fp8[:, :cols] = torch.from_numpy(a.fp8).to(dev)
            bf16[:, :cols] = torch.from_numpy(a.bf16.view(np.int16)).to(dev)
            scale, mask = torch.from_numpy(a.scale).to(dev), torch.from_numpy(a.mask).to(dev)
            B.mor_dequantize(p, fp8[:, :cols], scale, mask, bf16[:, :cols], y[:, :cols])
            got = y[:, :cols].cpu().numpy().view(np.uint16)
            assert np.array_equal(got, want)
            assert bool((y[:, cols:] == 0x5A5A).all())
            y.fill_(0x5A5A)
            B.mor_dequantize(p, fp8[:, :cols], scale, mask, None, y[:, :cols])      # BF16 blocks stay as they are
            blank = oracle.dequantize(a.fp8, a.scale, a.mask, np.full((rows, cols), 0x5A5A, np.uint16), gran, ragged=True)
            assert np.array_equal(y[:, :cols].cpu().numpy().view(np.uint16), blank)


@pytest.mark.parametrize("gran, band", [("sub1x128", 1), ("sub1x128", 7), ("block64", 64), ("block128", 256)])
def test_stored_scales_with_bands(oracle, gran, band):
    """E8M0 bytes and one mantissa per band of rows: tiles that start and end inside a band."""
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    rows, cols = 300, 264
    x, a, _ = _analysed(oracle, rows, cols, gran, scaling="gam", gam_group_rows=band)
    p = B.make_params(rows, cols, gran, ragged=True, scaling="gam", gam_group_rows=band)
    want = oracle.dequantize(a.fp8, a.scale, a.mask, a.bf16, gran, ragged=True)
    t = lambda v: torch.from_numpy(v).to(dev)                              # noqa: E731
    y = torch.zeros((rows, cols), dtype=torch.int16, device=dev)
    B.mor_dequantize_e8m0(p, t(a.fp8), t(a.e8m0), t(np.ascontiguousarray(a.group_mantissas.reshape(-1)).view(np.int32)), t(a.mask),
                          t(a.bf16.view(np.int16)), y)
    assert np.array_equal(y.cpu().numpy().view(np.uint16), want)


def test_rows_too_long_for_tile_offsets(oracle):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    rows, cols, ld = 520, 16, 2097152
    x, a, _ = _analysed(oracle, rows, cols, "channel_row")
    p = B.make_params(rows, cols, "channel_row")
    want = oracle.dequantize(a.fp8, a.scale, a.mask, a.bf16, "channel_row")
    y = torch.zeros(rows * ld, dtype=torch.int16, device=dev).view(rows, ld)
    t = lambda v: torch.from_numpy(v).to(dev)                              # noqa: E731
    B.mor_dequantize(p, t(a.fp8), t(a.scale), t(a.mask), t(a.bf16.view(np.int16)), y[:, :cols])
    assert np.array_equal(y[:, :cols].cpu().numpy().view(np.uint16), want)
    assert int(torch.count_nonzero(y)) == int(np.count_nonzero(want))


def test_conversion_agrees_on_every_code():
    """All 256 codes of both formats under scales of every kind: finite, subnormal, infinite, zero."""
    from paper_2512_22804_amd import binding as B
    from oracle import mor_oracle as O
    dev = torch.device("cuda:0")
    scales = np.array([1.0, 3.14159, 1e-38, 1e-45, 3.4e38, 0.0, -0.0, np.inf, -np.inf, 448.0 / 3, 57344.0 / 7], np.float32)
    rows, cols = len(scales), 256
    fp8 = np.tile(np.arange(256, dtype=np.uint8), (rows, 1))
    p = B.make_params(rows, cols, "channel_row")
    for code in (0, 2):
        mask = np.full(rows, code, np.uint8)
        with np.errstate(all="ignore"):
            want = O.dequantize(fp8, scales, mask, np.zeros((rows, cols), np.uint16), "channel_row")
        y = torch.zeros((rows, cols), dtype=torch.int16, device=dev)
        B.mor_dequantize(p, torch.from_numpy(fp8).to(dev), torch.from_numpy(scales).to(dev), torch.from_numpy(mask).to(dev), None, y)
        got = y.cpu().numpy().view(np.uint16)
        nan = (want & 0x7FFF) > 0x7F80
        assert np.array_equal(got[~nan], want[~nan])
        assert ((got[nan] & 0x7FFF) == 0x7FC0).all()      # (the sign of a NaN product is the operand's that the hardware picks)
