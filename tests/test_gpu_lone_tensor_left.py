"""The bounded wait of a small per-tensor operand alone in its call: a workgroup that is not told the decision in time marks its tile as left
and ends, and the workgroup that decides sees to it.  Here nobody looks more than the once after leaving, so that nearly every tile is
left; every output must be what a call that waits gives, bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# threads x chunks of the kernels: 512 x 4 (dense), 256 x 8, 512 x 4 (one tile), 256 x 2, 512 x 2, 256 x 8, 512 x 2 (rows beyond the row map)
OPERANDS = [(1000, 1048, 0), (2048, 4096, 0), (1, 8, 0), (1000, 1048, 8), (700, 4096, 4096), (1500, 4096, 64), (1, 2500000, 1700000)]


def _values(rows, ld, kind):
    """BF16 bits in [1, 2), for "e5m2" and "bf16" three in ten below what E4M3 holds under the operand's
    scale (E5M2 holds all of them, or half)."""
    rng = np.random.default_rng(rows + ld)
    x = (0x3F80 | rng.integers(0, 128, (rows, ld))).astype(np.uint16) | (rng.integers(0, 2, (rows, ld)) << 15).astype(np.uint16)
    if kind != "e4m3":
        small = rng.random((rows, ld)) < 0.3
        small[0, :3] = (True, False, True)
        x[small] = (x[small] & 0x807F) | 0x3480           # 2^-22
        if kind == "bf16":
            x[:, ::2][small[:, ::2]] -= 33 << 7           # half of them 2^-55
    return x


@pytest.mark.parametrize("rows, cols, pad", OPERANDS)
@pytest.mark.parametrize("crit, formats, kind, mask", [("mean_rel_err", "e4m3|bf16", "e4m3", 0), ("mean_rel_err", "e4m3|bf16", "e4m3", 1),
                                                       ("mean_rel_err", "e4m3|bf16", "bf16", 1), ("e4m3_vs_e5m2", "e4m3|bf16", "bf16", 1),
                                                       ("mean_rel_err", "e4m3|e5m2|bf16", "e5m2", 2), ("e4m3_vs_e5m2", "e4m3|e5m2|bf16", "e5m2", 2),
                                                       ("e4m3_vs_e5m2", "e4m3|e5m2|bf16", "bf16", 1)])
@pytest.mark.parametrize("fake", [False, True])
def test_tiles_that_are_left(rows, cols, pad, crit, formats, kind, mask, fake):
    import parity
    from paper_2512_22804_amd import binding as B
    lib = B.load()
    lib.mor_test_lone_tensor.argtypes = [C.POINTER(B.MorParams), C.c_void_p, C.POINTER(B.MorOutputs), C.c_void_p, C.c_int64, C.c_void_p, C.c_size_t,
                                         C.c_void_p, C.c_int32, C.POINTER(C.c_int64)]
    print(f"[left] {rows}x{cols}+{pad} {crit} {formats} {kind} fake={fake}", flush=True)
    x = _values(rows, cols + pad, kind)
    xd = parity.to_dev(x)
    threshold = 0.001 if (kind, mask) == ("e4m3", 1) else 0.045
    p = B.make_params(rows, cols, "tensor", crit=crit, formats=formats, threshold=threshold, ld=cols + pad)
    results, left = [], (C.c_int64 * 2)()
    for polls in (None, 0):
        out, guards = parity.guarded_outputs(p, xd.device, want_bf16=not fake, bf16_fill=parity.FILL, want_fp8=not fake)
        y = guards.carve("y", (rows, cols), torch.int16, 0x1111) if fake else None
        if polls is None:
            B.mor_fake_quantize(p, xd, y, out) if fake else B.mor_analyze_quantize(p, xd, out)
        else:
            o = B._outputs_struct(out)
            rc = lib.mor_test_lone_tensor(C.byref(p), xd.data_ptr(), C.byref(o), y.data_ptr() if fake else None, cols, out.workspace.data_ptr(),
                                          out.workspace.numel(), torch.cuda.current_stream().cuda_stream, polls, left)
            assert rc == 0
        torch.cuda.synchronize()
        guards.check()
        results.append((out, y))
    (want, y0), (got, y1) = results
    assert int(want.mask[0]) == mask
    for k in ("fp8", "bf16", "scale", "amax", "err_sum", "err5_sum", "nnz", "mask", "amin"):
        a, b = getattr(want, k), getattr(got, k)
        assert (a is None) == (b is None) and (a is None or torch.equal(a, b)), k
    assert not fake or torch.equal(y0, y1)
    words = got.workspace[left[0]:left[0] + 4 * left[1]].view(torch.int32).cpu().numpy()
    if crit == "mean_rel_err" or rows * cols <= 1 << 22:          # (else the kernels for several operands take it)
        assert set(words.tolist()) <= {0, 1}
        proven = kind == "bf16" and crit == "mean_rel_err" and rows > 1      # nobody waits then (rows beyond the row map prove nothing)
        assert bool(words.any()) == (not proven and rows * cols >= 1 << 19)
    if not fake and kind != "e4m3":
        parity.compare(x, "tensor", crit=crit, formats=formats, threshold=threshold, cols=cols, gpu=(p, got))
