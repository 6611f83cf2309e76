"""The de-quantized values are rounded to BF16 by a conversion instruction: compared with round-to-nearest-even in integer arithmetic
on the products of sixteen codes with the inverse of scales of all 2^23 mantissas, at exponents that give large, ordinary and
subnormal products.  A row of eight columns is one 1x128 block, so that every row has a scale of its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CODES = [[0x38, 0x39, 0x3F, 0xB8, 0x01, 0x08, 0x7E, 0xFE], [0x3A, 0xBB, 0x02, 0x03, 0x87, 0x0F, 0x00, 0x80]]      # E4M3: 1, 1.125, 1.875, -1, 2^-9, 2^-6, 448, ...
ROWS = 1 << 21


@pytest.mark.parametrize("exponent", [1, 64, 127, 128, 200, 252, 253, 254])
def test_rounding(exponent):
    from paper_2512_22804_amd import binding as B
    dev = torch.device("cuda:0")
    p = B.make_params(ROWS, 8, "sub1x128", ragged=True)
    mask = torch.zeros(ROWS, dtype=torch.uint8, device=dev)
    y = torch.empty((ROWS, 8), dtype=torch.int16, device=dev)
    ties = subnormals = 0
    for first in range(0, 1 << 23, ROWS):
        bits = torch.arange(first, first + ROWS, dtype=torch.int32, device=dev) | (exponent << 23)
        scale = bits.view(torch.float32)
        inverse = (1.0 / scale.double()).float().double()          # binary64 holds enough digits for the second rounding to be harmless
        for codes in CODES:
            row = torch.tensor(codes, dtype=torch.uint8, device=dev)
            B.mor_dequantize(p, row.repeat(ROWS, 1), scale, mask, None, y)
            v = row.view(torch.float8_e4m3fn).double()
            u = (v[None, :] * inverse[:, None]).float().view(torch.int32)
            want = (u + 0x7FFF + ((u >> 16) & 1)) >> 16
            assert torch.equal(y.int() & 0xFFFF, want & 0xFFFF)
            ties += int(((u & 0xFFFF) == 0x8000).sum())
            subnormals += int((((u & 0x7F800000) == 0) & ((u & 0x7FFFFF) != 0)).sum())
    assert ties > 0
    assert exponent < 250 or subnormals > 0
