"""FP8 conversion of words that mix NaN of both signs, infinities and finite
values in every position, at lengths around a block's last unit: the codes and
the bf16 results equal the oracle's."""
import numpy as np
import pytest
import torch

import paper_2606_20537_amd as cap

pytestmark = pytest.mark.gpu

SPECIAL = np.array([0x7F81, 0xFF81, 0x7FC0, 0xFFC0, 0x7FFF, 0xFFFF, 0x7F80, 0xFF80, 0x0000, 0x8000, 0x3F80, 0xBF80,
                    0x43E0, 0xC3E8, 0x0001, 0x8001], dtype=np.uint16)


@pytest.mark.parametrize("n", [16, 4080, 4096, 4112, 3 * 4096 + 16])
@pytest.mark.parametrize("scale", [1.0, 0.0125])
def test_mixed_specials(orc, n, scale):
    rng = np.random.default_rng(n)
    bits = SPECIAL[rng.integers(0, SPECIAL.size, n)]
    src = torch.from_numpy(bits.view(np.int16).copy()).cuda()
    dst = torch.full((n + 16,), 0xAA, dtype=torch.uint8, device="cuda")
    cap.kv_fp8_quantize([(src, dst, n, scale)])
    codes = rng.choice(np.array([0x7F, 0xFF, 0x7E, 0xFE, 0x00, 0x80, 0x08, 0x7F], dtype=np.uint8), n)
    out = torch.full((n + 8,), 0x1234, dtype=torch.int16, device="cuda")
    cap.kv_fp8_dequantize([(torch.from_numpy(codes).cuda(), out, n, scale)])
    torch.cuda.synchronize()
    got, back = dst.cpu().numpy(), out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:n], orc.fp8_quantize(bits, scale)) and np.all(got[n:] == 0xAA)
    assert np.array_equal(back[:n], orc.fp8_dequantize(codes, scale)) and np.all(back[n:] == 0x1234)


@pytest.mark.parametrize("scale", [1e-39, 1e-45, 3e-39])
def test_reciprocal_out_of_range(orc, scale):
    """1 / scale is infinite for the first two: zeros become NaN with the sign
    of the product (not the input's), everything else saturates."""
    bits = np.arange(65536, dtype=np.uint32).astype(np.uint16)
    dst = torch.full((65536,), 0xAA, dtype=torch.uint8, device="cuda")
    cap.kv_fp8_quantize([(torch.from_numpy(bits.view(np.int16).copy()).cuda(), dst, 65536, scale)])
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy(), orc.fp8_quantize(bits, scale))


def test_every_value_in_every_position(orc):
    """A unit converts eight elements with packed instructions: every code, and
    every bf16 pattern, in each of the eight positions."""
    codes = np.concatenate([np.roll(np.arange(256, dtype=np.uint8), i) for i in range(8)])
    bits = np.concatenate([np.roll(np.arange(65536, dtype=np.uint32), i).astype(np.uint16) for i in range(8)])
    out = torch.zeros(codes.size, dtype=torch.int16, device="cuda")
    dst = torch.zeros(bits.size, dtype=torch.uint8, device="cuda")
    cap.kv_fp8_dequantize([(torch.from_numpy(codes).cuda(), out, codes.size, 0.3)])
    cap.kv_fp8_quantize([(torch.from_numpy(bits.view(np.int16).copy()).cuda(), dst, bits.size, 0.3)])
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint16), orc.fp8_dequantize(codes, 0.3))
    want = orc.fp8_quantize(np.arange(65536, dtype=np.uint32).astype(np.uint16), 0.3)
    assert np.array_equal(dst.cpu().numpy(), np.concatenate([np.roll(want, i) for i in range(8)]))
