"""The row quantiser's division by a two-float reciprocal against the oracle's float32 quotient, bit for bit: every
mantissa that a row's scale can have (128: amax is a bf16 value) times every bf16 x down to 2^-20 of the row's largest, both
signs, zeros of both signs; rows that take the division itself (NaN, infinite, very small elements); row lengths at the
edges of what a thread holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_backend
    return gpu_backend


def _check(oracle, G, bits):
    import torch
    from paper_2509_16495_amd import binding as B
    want_codes, want_scales = oracle.quantize_rows_e4m3(bits, "bf16")
    codes = torch.full(bits.shape, 0x55, dtype=torch.uint8, device=G.DEV)
    scales = torch.zeros(bits.shape[0], dtype=torch.float32, device=G.DEV)
    B.quantize_rows_fp8(G.t(bits, "bf16"), codes, scales)
    torch.cuda.synchronize()
    got_scales = scales.cpu().numpy()
    assert np.array_equal(got_scales.view(np.uint32)[~np.isnan(want_scales)], want_scales.view(np.uint32)[~np.isnan(want_scales)])
    assert np.array_equal(codes.cpu().numpy(), want_codes)


@pytest.mark.parametrize("exponent", [127 - 40, 127, 127 + 3, 127 + 50])
def test_every_scale_and_element(oracle, G, exponent):
    top = (np.arange(128) + (exponent << 7)).astype(np.uint16)                        # the row's largest element
    below = np.arange((exponent - 20) << 7, (exponent + 1) << 7, dtype=np.int64)      # 21 octaves of magnitudes
    mags = np.minimum(below[None, :], top[:, None].astype(np.int64)).astype(np.uint16)
    zeros = np.tile(np.array([0, 0x8000, 0, 0x8000, 0, 0, 0x8000, 0x8000], dtype=np.uint16), (128, 1))
    _check(oracle, G, np.concatenate([mags, mags | 0x8000, zeros], axis=1))


@pytest.mark.parametrize("cols", [8, 2040, 2048, 2056, 4104, 6152, 8184, 8200, 12296, 16384, 16392])
def test_row_lengths(oracle, G, cols):
    rng = np.random.Generator(np.random.PCG64(7))
    x = rng.standard_normal((3, cols), dtype=np.float32)
    x[2] *= np.float32(1e-30)                                                          # a scale too small for the reciprocal
    x[0, -1] = 9.0                                                                     # the largest element is the last one
    _check(oracle, G, (x.view(np.uint32) >> 16).astype(np.uint16))


def test_nan_elements(oracle, G):
    rng = np.random.Generator(np.random.PCG64(8))
    bits = (rng.standard_normal((4, 4104), dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    bits[1, 5] = 0x7FC0
    bits[2, 4103] = 0xFFC1
    import torch
    from paper_2509_16495_amd import binding as B
    want_codes, want_scales = oracle.quantize_rows_e4m3(bits, "bf16")
    codes = torch.zeros(bits.shape, dtype=torch.uint8, device=G.DEV)
    scales = torch.zeros(4, dtype=torch.float32, device=G.DEV)
    B.quantize_rows_fp8(G.t(bits, "bf16"), codes, scales)
    torch.cuda.synchronize()
    got, nan = codes.cpu().numpy(), (bits & 0x7FFF) > 0x7F80
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), want_scales.view(np.uint32))
    assert np.array_equal(got[~nan], want_codes[~nan])
    assert np.all((got[nan] & 0x7F) == 0x7F) and np.all((want_codes[nan] & 0x7F) == 0x7F)
