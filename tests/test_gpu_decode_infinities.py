"""Infinite values in the value cache of a decoding step: a column of out is +inf (-inf) where some row with a nonzero
weight holds +inf (-inf) in it, NaN where rows hold both, and every other column keeps its bound (parity.decode_error).
The logits stay within +-20, so no weight underflows.  Rows that hold them: the first, the last of the layer (which the
kernels repeat to fill their last step), one in the middle, and one of the appended rows."""
import numpy as np
import pytest
import torch

from oracle import decode_oracle as D

from parity import decode_error

pytestmark = pytest.mark.gpu
LENS = [1, 33, 128, 300, 1000]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (2, 1), (3, 1), (4, 1), (5, 1), (8, 1)])
@pytest.mark.parametrize("n_new", [0, 5, 150])
def test_infinite_values(dtype, d, hq, hkv, n_new):
    import paper_2502_17599_amd as pkg
    print(f"\n[decode infinities] {dtype} d={d} Hq={hq} Hkv={hkv} n_new={n_new}", flush=True)
    dev, L = torch.device("cuda:0"), len(LENS)
    g = torch.Generator().manual_seed(hq * 10 + d)
    rows = sum(LENS) * hkv
    k, v = (torch.randn(rows, d, generator=g).to(dtype) for _ in range(2))
    q = torch.randn(L, hq, d, generator=g).to(dtype)
    kn = vn = None
    if n_new:
        kn, vn = (torch.randn(L, hkv, n_new, d, generator=g).to(dtype) for _ in range(2))
    off = np.concatenate([[0], np.cumsum(LENS)])
    inf = float("inf")
    for l, s in enumerate(LENS):
        for h in range(hkv):
            row = off[l] * hkv + h * s
            v[row, 3] = inf
            v[row + s // 2, d // 2] = -inf
            v[row + s - 1, d - 1] = inf
            v[row, 7] = inf
            v[row + s - 1, 7] = -inf  # the same row in the layer of one row: -inf alone
            if n_new:
                vn[l, h, n_new - 1, 9] = -inf
    s_dev = torch.tensor(LENS, dtype=torch.int32, device=dev)
    off_dev = torch.tensor(off, dtype=torch.int64, device=dev)
    dec = pkg.Decoder(pkg.make_decode_params(L, hq, hkv, d, sum(LENS), dtype, n_new), dev)
    args = [x if x is None else x.to(dev) for x in (kn, vn)]
    out = dec(q.to(dev), k.to(dev), v.to(dev), s_dev, off_dev, *args)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = D.decode_step(q.double().numpy(), k.double().numpy(), v.double().numpy(), np.array(LENS), off, hkv,
                            None if kn is None else kn.double().numpy(), None if vn is None else vn.double().numpy())
    assert np.isnan(ref).any() and np.isposinf(ref).any() and np.isneginf(ref).any()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    finite = np.isfinite(ref)
    decode_error(got[finite], ref[finite], 6.0, dtype == torch.bfloat16)
