"""Selection statistics of operands in a batch call, at block counts that fill or cross a wave, a workgroup's round and a workgroup's
share: the counters come from ballots and the records are read by neighbouring lanes, so a lane beyond the last block must count nothing."""
import numpy as np
import pytest
import torch

from paper_2512_22804_amd import workloads as W

pytestmark = pytest.mark.gpu
INT_KEYS = ("n_part", "n_fp8_part", "n_bf16_part", "n_e5m2_part", "n_elem_fp8", "n_elem_bf16", "n_elem_e5m2", "nnz_total", "hist", "n_near_threshold")
COUNTS = [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4097, 16384, 16385, 70001]


@pytest.mark.parametrize("n", COUNTS)
@pytest.mark.parametrize("crit, formats", [("mean_rel_err", "e4m3|bf16"), ("e4m3_vs_e5m2", "e4m3|e5m2|bf16")])
def test_counts(oracle, n, crit, formats):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    cols = 120                                            # ragged blocks: 120 elements each, the last row's included
    x = W.gradient(n, 128, n, tiny_frac=0.3, tiny_half=True)[:, :cols].copy()
    x[::7] = (x[::7] & 0x8000) | 0x3200                   # constant magnitude
    x[n // 2, 5] = 0x7F80                                 # a block with an infinity, one with NaN, one without a value
    x[n // 3, 9] = 0x7FC1
    x[n // 5] = 0
    xd = torch.from_numpy(x.view(np.int16)).to(dev)
    p = B.make_params(n, cols, "sub1x128", crit=crit, formats=formats, ragged=True)
    entries = []
    for _ in range(2):                                    # beside another operand: the statistics launches of several operands
        entries.append((p, xd, B.alloc_outputs(p, dev, bf16_fill=0), torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)))
    items = B.make_batch(entries)
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
    B.mor_analyze_quantize_batch(items, 1e-2, ws)
    alone = torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev)
    out = entries[0][2]
    B.mor_select_stats(p, out.err_sum, out.nnz, out.mask, 1e-2, alone)
    torch.cuda.synchronize()
    want = oracle.select_stats(out.err_sum.cpu().numpy(), out.nnz.cpu().numpy().view(np.uint32), out.mask.cpu().numpy(), n, cols, "sub1x128",
                               0.045, 1e-2, ragged=True)
    for got in (B.read_stats(entries[0][3]), B.read_stats(entries[1][3]), B.read_stats(alone)):
        for k in INT_KEYS:
            if k in want:
                assert got[k] == want[k], (k, got[k], want[k])
        if np.isfinite(want["err_sum_total"]):
            assert got["err_sum_total"] == pytest.approx(want["err_sum_total"], rel=1e-12)
        else:
            assert not np.isfinite(got["err_sum_total"])
