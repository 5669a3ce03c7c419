"""Rows whose scale lies around the range in which the quantiser works from a shared reciprocal (2^-80 .. 2^80), rows of
zeros of either sign, and row counts around the four row groups a wave takes: codes and scales bit for bit as the
float32 scheme of the oracle."""
import numpy as np
import pytest
import torch

from oracle import fp8_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 3, 15, 16, 17, 64, 131])
def test_scales_around_the_fast_range(dtype, d, n):
    import paper_2502_17599_amd as pkg
    rng = np.random.default_rng(n * 1000 + d)
    x = rng.standard_normal((n, d)).astype(np.float32)
    exps = np.array([0, -79, -80, -81, 79, 80, 81, -100, 100, 3], dtype=np.float64)
    x *= np.float32(2.0) ** exps[np.arange(n) % len(exps)][:, None].astype(np.float32)
    x[rng.random(x.shape) < 0.1] = -0.0
    x[:, 1] *= np.float32(1e-5)                # elements that round to zero or to subnormal codes
    if n > 2:
        x[2] = -0.0
    t = torch.from_numpy(x).to(dtype)
    codes, scales = pkg.meda_quantize_fp8(t.to("cuda:0"))
    torch.cuda.synchronize()
    ref_codes, ref_scales = fp8_oracle.quantize_rows(t.double().numpy())
    assert np.array_equal(scales.cpu().numpy(), ref_scales.astype(np.float32))
    assert np.array_equal(codes.cpu().numpy(), ref_codes)
