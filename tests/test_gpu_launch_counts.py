"""How many kernels a call of several operands launches, from the library's own profile: operands that are read twice are taken in
parts of at most 256 MB only where the second read gains more than the launches of each part cost."""
import collections

import pytest
import torch

pytestmark = pytest.mark.gpu


def _kernels(gran, scope, scaling, shapes, fake=False):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1)
    entries = []
    for rows, cols in shapes:
        x = torch.randn((rows, cols), generator=gen, device=dev).to(torch.bfloat16)
        p = B.make_params(rows, cols, gran, scope, "mean_rel_err", 0.045, scaling=scaling)
        out = B.alloc_outputs(p, dev, want_bf16=not fake, want_fp8=not fake)
        entries.append((p, x, out, None, torch.empty_like(x) if fake else None))
    items = B.make_batch(entries)
    ws = torch.empty(max(16, B.mor_batch_workspace_bytes(items)), dtype=torch.uint8, device=dev)
    ev = B.HipEvents()
    prof = ev.new_profile(B.MOR_PROFILE_MAX)
    B.mor_analyze_quantize_batch(items, 1e-5, ws, prof)
    torch.cuda.synchronize()
    names = [B.KERNEL_NAMES[prof.kernel[k]] for k in range(prof.count)]
    ev.destroy()
    assert len(names) < B.MOR_PROFILE_MAX
    return collections.Counter(names)


THREE = [(4096, 14336)] * 3          # 117 MB each


@pytest.mark.parametrize("scaling", ["fp32_amax", "gam"])
def test_columns_share_their_launches(scaling):
    got = _kernels("channel_col", "partition", scaling, THREE)
    assert got == {"column_tile": 2, "column_combine": 2, "fallback_copy": 1}
