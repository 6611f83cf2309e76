"""Per-tensor operands of 2^34 elements (34 GB): 2^20 tiles, so that a workgroup of the amax pass counts elements over 2048 tiles.
A count that wraps there would claim that every element flushes to zero, and an operand kept in E4M3 would be handled as one
proven to stay in BF16.  The operand repeats one slab, so that every slab of its outputs is that of the slab alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS, COLS, SLAB = 131072, 131072, 1024


@pytest.mark.parametrize("pad", [0, 8])
def test_no_false_proof(pad):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    if torch.cuda.mem_get_info(dev)[0] < 100 << 30:
        pytest.skip("needs 100 GiB of device memory")
    torch.cuda.empty_cache()
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    base = (1.0 + torch.rand((SLAB, COLS), generator=gen, device=dev)).to(torch.bfloat16)      # one binade: E4M3's mean error is below 3 %
    base[0, 0] = 2.0
    p1 = B.make_params(SLAB, COLS, "tensor")
    out1 = B.alloc_outputs(p1, dev, bf16_fill=0x5A5A)
    y1 = torch.empty_like(base)
    B.mor_analyze_quantize(p1, base, out1)
    B.mor_fake_quantize(p1, base, y1, out1)
    assert int(out1.mask[0]) == 0 and not torch.equal(y1, base)

    x = torch.empty((ROWS, COLS + pad), dtype=torch.bfloat16, device=dev)
    x.view(ROWS // SLAB, SLAB, COLS + pad)[:, :, :COLS] = base
    p = B.make_params(ROWS, COLS, "tensor", ld=COLS + pad, lean_fp8=True)
    out = B.alloc_outputs(p, dev, want_bf16=False)
    y = torch.empty((ROWS, COLS), dtype=torch.bfloat16, device=dev)
    B.mor_fake_quantize(p, x[:, :COLS], y, out)
    assert int(out.mask[0]) == 0 and float(out.scale[0]) == float(out1.scale[0])
    for r in range(0, ROWS, SLAB):
        assert torch.equal(y[r:r + SLAB], y1), r
    # the payload call: codes are stored although a lean operand need not have any, the BF16 buffer is left alone
    out.bf16 = y.view(torch.int16)
    out.bf16.fill_(0x5A5A)
    out.fp8.fill_(0xA5)
    B.mor_analyze_quantize(p, x[:, :COLS], out)
    assert int(out.mask[0]) == 0
    for r in range(0, ROWS, SLAB):
        assert torch.equal(out.fp8[r:r + SLAB], out1.fp8), r
        assert bool((out.bf16[r:r + SLAB] == 0x5A5A).all()), r
    del x, y, out
    torch.cuda.empty_cache()
