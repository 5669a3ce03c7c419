"""How a decoding step cuts the rows into chunks: lengths around the 32-row step of a wave, the 128-row workgroup
step and the chunk size, very uneven layers, more than 64 layers, appended rows with and without chunks of their own,
and lengths whose sum exceeds the budget the launch was sized for.  Against the fp64 oracle; the bound is that of
parity.decode_error (exact products, fp32 sums, one rounding)."""
import numpy as np
import pytest
import torch

from oracle import decode_oracle as D
from oracle import fp8_oracle

from parity import decode_error

pytestmark = pytest.mark.gpu


def _case(lens, hq, hkv, d, dtype, n_new, budget=None, fp8=False, seed=0):
    import paper_2502_17599_amd as pkg
    print(f"\n[decode split] L={len(lens)} Hq={hq} Hkv={hkv} d={d} {dtype} n_new={n_new} fp8={fp8}", flush=True)
    dev = torch.device("cuda:0")
    L, rows = len(lens), sum(lens) * hkv
    g = torch.Generator().manual_seed(seed)
    k = torch.randn(rows, d, generator=g).to(dtype).to(dev)
    v = torch.randn(rows, d, generator=g).to(dtype).to(dev)
    q = (3 * torch.randn(L, hq, d, generator=g)).to(dtype).to(dev)
    kn = vn = None
    if n_new:
        kn = torch.randn(L, hkv, n_new, d, generator=g).to(dtype).to(dev)
        vn = torch.randn(L, hkv, n_new, d, generator=g).to(dtype).to(dev)
    s = torch.tensor(lens, dtype=torch.int32, device=dev)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64, device=dev)
    dec = pkg.Decoder(pkg.make_decode_params(L, hq, hkv, d, sum(lens) if budget is None else budget, dtype, n_new), dev)
    if fp8:
        kc, ks = pkg.meda_quantize_fp8(k)
        vc, vs = pkg.meda_quantize_fp8(v)
        out = dec.fp8(q, kc, vc, ks, vs, s, off, kn, vn)
        kr = fp8_oracle.dequantize_rows(kc.cpu().numpy(), ks.cpu().numpy())
        vr = fp8_oracle.dequantize_rows(vc.cpu().numpy(), vs.cpu().numpy())
    else:
        out = dec(q, k, v, s, off, kn, vn)
        kr, vr = k.double().cpu().numpy(), v.double().cpu().numpy()
    torch.cuda.synchronize()
    ref = D.decode_step(q.double().cpu().numpy(), kr, vr, np.array(lens), off.cpu().numpy(), hkv,
                        None if kn is None else kn.double().cpu().numpy(), None if vn is None else vn.double().cpu().numpy())
    vmax = max(np.abs(vr).max(), 0.0 if vn is None else float(vn.abs().max()))
    decode_error(out.double().cpu().numpy(), ref, vmax, dtype == torch.bfloat16)


EDGES = [1, 31, 32, 33, 127, 128, 129, 255, 257, 1000]


@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (3, 1), (8, 2), (5, 1), (8, 1)])
@pytest.mark.parametrize("d", [64, 128])
def test_lengths_around_the_steps(hq, hkv, d):
    for n_new in (0, 1, 33, 128, 129, 300):
        _case(EDGES, hq, hkv, d, torch.bfloat16, n_new)
    _case(EDGES, hq, hkv, d, torch.bfloat16, 5, fp8=True)
    _case(EDGES, hq, hkv, d, torch.bfloat16, 140, fp8=True)
    for n_new in (5, 32, 33, 140):
        _case(EDGES, hq, hkv, d, torch.float32, n_new)


def test_more_layers_than_lanes_and_uneven_lengths():
    lens = [1 + (37 * i * i) % 400 for i in range(130)]
    lens[70] = 9000
    _case(lens, 4, 1, 64, torch.bfloat16, 2)
    _case(lens, 2, 1, 64, torch.float32, 0)


@pytest.mark.parametrize("L", [63, 64, 65, 511, 512, 513, 1030])
def test_layers_around_the_steps_of_the_chunk_search(L):
    lens = [1 + (53 * i * i) % 300 for i in range(L)]
    lens[L - 1], lens[L // 2] = 700, 1
    _case(lens, 2, 1, 64, torch.bfloat16, 0)
    _case(lens, 2, 1, 64, torch.bfloat16, 140, budget=L)       # R doubled until the chunks fit, appended rows of their own
    _case(lens, 2, 1, 64, torch.float32, 2)


def test_lengths_beyond_the_budget_of_the_launch():
    # 20 layers of up to 2000 rows, sized for 20 rows: the chunks grow until their number fits
    lens = [2000, 1, 700] * 6 + [129, 128]
    _case(lens, 4, 2, 128, torch.bfloat16, 3, budget=20)
    _case(lens, 2, 2, 64, torch.float32, 200, budget=20)


def test_rows_enough_for_chunks_of_several_hundred_rows():
    # 2 kv heads, 500000 rows: chunks of 384 rows at 1536 workgroups
    _case([120000, 70000, 33333, 26667], 8, 2, 64, torch.bfloat16, 0)


@pytest.mark.parametrize("fp8,dtype,d,rows", [(False, torch.bfloat16, 128, 1 << 24), (True, torch.bfloat16, 128, 1 << 25),
                                              (False, torch.float32, 64, 1 << 24)])
def test_a_chunk_of_more_than_4_gib(fp8, dtype, d, rows):
    # One layer sized for one row is one chunk: its rows from the 2^32nd byte on are the only ones with keys, values and a
    # weight; rows read from anywhere else give zero.  The softmax over them is uniform: out = 1.
    import paper_2502_17599_amd as pkg
    print(f"\n[decode split] {rows} rows and 40 more, d={d} {dtype} fp8={fp8}", flush=True)
    dev, tail = torch.device("cuda:0"), 40
    el = torch.uint8 if fp8 else dtype
    k, v = (torch.zeros(rows + tail, d, dtype=el, device=dev) for _ in range(2))
    k[rows:] = 0x38 if fp8 else 1.0   # 0x38 is the code of 1
    v[rows:] = 0x38 if fp8 else 1.0
    q = torch.full((1, 1, d), 4.0, dtype=dtype, device=dev)       # logits of 4 sqrt(d): the others' weights vanish
    s = torch.tensor([rows + tail], dtype=torch.int32, device=dev)
    off = torch.tensor([0, rows + tail], dtype=torch.int64, device=dev)
    p = pkg.make_decode_params(1, 1, 1, d, 1, dtype, 0)
    dec = pkg.Decoder(p, dev)
    if fp8:
        ones = torch.ones(rows + tail, device=dev)
        out = dec.fp8(q, k, v, ones, ones, s, off)
    else:
        out = dec(q, k, v, s, off)
    torch.cuda.synchronize()
    # the 2^24 and more other rows weigh exp(-4 sqrt(d)) each: 2^25 * exp(-45.2) and 2^24 * exp(-32) over 40 rows
    assert (out.float() - 1).abs().max() < 1e-6 + (2.0 ** -8 if dtype == torch.bfloat16 else 0.0)


def test_chunks_made_longer_to_fit_the_built_in_scratch():
    # 150 layers, 512 query heads: 157 partials per head fit, 174 would be cut without that bound.  The entry point without
    # a workspace gives the same bits.
    import paper_2502_17599_amd as pkg
    lens = [200 if l % 9 == 0 else 10 + l % 7 for l in range(150)]
    p = pkg.make_decode_params(150, 512, 64, 128, sum(lens), torch.bfloat16, 0)
    assert pkg.DECODE_NOALLOC_MAX_BYTES - 512 * 130 * 4 < pkg.meda_decode_workspace_bytes(p) <= pkg.DECODE_NOALLOC_MAX_BYTES
    _case(lens, 512, 64, 128, torch.bfloat16, 0)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(0)
    k, v = (torch.randn(sum(lens) * 64, 128, generator=g, device=dev).bfloat16() for _ in range(2))
    q = torch.randn(150, 512, 128, generator=g, device=dev).bfloat16()
    s = torch.tensor(lens, dtype=torch.int32, device=dev)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64, device=dev)
    out = pkg.Decoder(p, dev)(q, k, v, s, off).clone()
    got = torch.empty_like(out)
    pkg.meda_decode_attention_noalloc(p, q, k, v, s, off, got)
    torch.cuda.synchronize()
    assert torch.equal(out, got)
