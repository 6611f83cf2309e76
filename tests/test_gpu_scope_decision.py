"""Tensor-level decisions at block counts around those up to which one launch takes them (2048 blocks with statistics, 4096 without):
decision, mask and copied fallback against the oracle, statistics against the oracle's count of the call's own sums."""
import numpy as np
import pytest
import torch

import parity
from paper_2512_22804_amd import workloads as W
from test_gpu_stats_counts import INT_KEYS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stats, n", [(s, n) for s in (True, False) for n in (1, 255, 257, 2047, 2048, 2049, 4095, 4096, 4097)])
def test_decisions(oracle, n, stats):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    entries, cases = [], []
    # two operands of the call, BF16 and FP8; padded rows in the first; under Eq. 3 the sums of both types decide
    for k, (cols, ld, tiny, crit) in enumerate([(128, 144, 0.5, "mean_rel_err"), (120, 120, 0.0, "mean_rel_err"), (128, 128, 0.3, "e4m3_vs_e5m2")]):
        x = W.gradient(n, 256, n + k, tiny_frac=tiny, tiny_half=True)[:, :ld].copy()
        if k == 0 and n > 1:
            x[n // 2, 5] = 0x7F80                          # a block with an infinity
        for scaling in ("fp32_amax", "gam"):
            p = B.make_params(n, cols, "sub1x128", "tensor", crit, 0.045, ld=ld, scaling=scaling, ragged=True)
            out = B.alloc_outputs(p, dev, bf16_fill=parity.FILL)
            entries.append((p, parity.to_dev(x), out, torch.full((B.STATS_BYTES,), 0xEE, dtype=torch.uint8, device=dev) if stats else None))
            cases.append((x, cols, crit, scaling))
    print(f"[scope] {n} blocks, statistics {stats}", flush=True)
    items = B.make_batch(entries)
    ws = torch.full((B.mor_batch_workspace_bytes(items),), 0xA7, dtype=torch.uint8, device=dev)
    B.mor_analyze_quantize_batch(items, 1e-2, ws)
    torch.cuda.synchronize()
    for (p, _, out, st), (x, cols, crit, scaling) in zip(entries, cases):
        parity.compare(x, "sub1x128", "tensor", crit, cols=cols, scaling=scaling, ragged=True, gpu=(p, out))
        if not stats:
            continue
        want = oracle.select_stats(out.err_sum.cpu().numpy(), out.nnz.cpu().numpy().view(np.uint32), out.mask.cpu().numpy(), n, cols, "sub1x128",
                                   0.045, 1e-2, ragged=True)
        got = B.read_stats(st)
        for k in INT_KEYS:
            if k in want:
                assert got[k] == want[k], (k, got[k], want[k])
        if np.isfinite(want["err_sum_total"]):             # up to 4097 binary32 sums added in binary64, in any order
            assert got["err_sum_total"] == pytest.approx(want["err_sum_total"], rel=1e-12)
