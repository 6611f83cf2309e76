"""Error sums of large per-tensor operands against 64 bits.  The sum is stored in binary32, which rounds it by up to 2^-24; the
additions that lead to it must not add more than that, in the root mean square over a few operands (BF16 inputs have few distinct
error terms, so the roundings of a long chain of additions are alike in all lanes and do not average out)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS, COLS = 8192, 14336


def _exact(x, scale):
    total = torch.zeros((), dtype=torch.float64, device=x.device)
    for r in range(0, x.shape[0], 1024):
        v = x[r:r + 1024].float()
        y = v * scale
        q = y.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double()
        y = y.double()
        total += torch.where(v != 0, (y - q).abs() / y.abs(), torch.zeros_like(y)).sum()
    return float(total)


@pytest.mark.parametrize("pad", [0, 8, COLS])
def test_error_sums_of_large_operands(pad):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    squares = []
    for seed in range(6):
        gen.manual_seed(seed)
        x = torch.empty((ROWS, COLS + pad), dtype=torch.bfloat16, device=dev)[:, :COLS]
        chan = torch.exp(torch.randn((1, COLS), generator=gen, device=dev)) if seed % 2 else 0.02          # activations, weights
        for r in range(0, ROWS, 1024):
            x[r:r + 1024] = torch.randn((1024, COLS), generator=gen, device=dev) * chan
        p = B.make_params(ROWS, COLS, "tensor", ld=COLS + pad)
        out = B.alloc_outputs(p, dev)
        B.mor_analyze_quantize(p, x, out)
        want = _exact(x, out.scale[0])
        squares.append((float(out.err_sum[0]) / want - 1.0) ** 2)
        print(f"[sums] pad={pad} seed={seed} relative error {squares[-1] ** 0.5:.2e}", flush=True)
    assert (sum(squares) / len(squares)) ** 0.5 <= 2.0 ** -24
