"""The sort of the dropped positions by the slot they merge into, at its edges: one to three passes (slots below and
above 256 and 65536), slot and position bits that do and do not fit one word, parts of a wave that are empty or
ragged, and lists of thousands.  The assignment the pass reports has to reproduce the merged rows: every output row is
the mean of its conserved row and its members, in fp64 and rounded once (which is what the kernels do)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(T, B, d, dtype, n_layers=1, hkv=1, one_cluster=False, seed=0):
    import paper_2502_17599_amd as pkg
    print(f"\n[segment sort] T={T} B={B} d={d} {dtype} one_cluster={one_cluster}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(seed)
    k = torch.randn(n_layers, hkv, T, d, generator=g, device=dev)
    if one_cluster:                      # every key close to one direction: few slots take nearly everything
        k[:, :, :] = k[:, :, :1] + 0.01 * k
    k = k.to(dtype)
    v = torch.randn(n_layers, hkv, T, d, generator=g, device=dev).to(dtype)
    q = torch.randn(n_layers, hkv, 16, d, generator=g, device=dev).to(dtype)
    mask = torch.ones(T, dtype=torch.uint8, device=dev)
    mask[:T // 3] = 0
    comp = pkg.Compressor(pkg.make_params(n_layers, hkv, hkv, d, T, 16, B, dtype), dev, want_merge_assign=True)
    out = comp(q, k, v, mask)
    torch.cuda.synchronize()
    for l in range(n_layers):
        k_l, v_l, idx = out.layer(l)
        s = int(out.layer_len[l])
        for h in range(hkv):
            slot = out.merge_assign[l, h].long()
            assert int(slot.min()) >= 0 and int(slot.max()) < s
            assert torch.equal(slot[idx[h].long()], torch.arange(s, device=dev))
            n = torch.zeros(s, dtype=torch.float64, device=dev).index_add_(0, slot, torch.ones(T, dtype=torch.float64, device=dev))
            for src, got in ((k[l, h], k_l[h]), (v[l, h], v_l[h])):
                mean = torch.zeros(s, d, dtype=torch.float64, device=dev).index_add_(0, slot, src.double()) / n[:, None]
                # fp64 sums in another order, then one rounding to the storage type: at most one ulp of it
                ulp = 2.0 ** (-7 if dtype == torch.bfloat16 else -23)
                assert ((got.double() - mean).abs() <= ulp * mean.abs().clamp_min(2.0 ** -126)).all()
                exact = (got == mean.to(dtype)).double().mean()
                assert exact > 0.9999, float(exact)


@pytest.mark.parametrize("T,B", [(65, 17), (100, 99), (1000, 16), (1025, 257), (1100, 256), (1104, 80), (5000, 600),
                                 (20000, 257)])
@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 128)])
def test_passes_and_ragged_parts(T, B, dtype, d):
    _case(T, B, d, dtype)


@pytest.mark.parametrize("T,B,L,hkv", [(129, 33, 2, 3), (128, 33, 2, 3), (700, 100, 32, 16), (300, 90, 64, 16), (2000, 300, 64, 16)])
def test_waves_chosen_by_length_and_pairs(T, B, L, hkv):
    _case(T, L * B, 64, torch.bfloat16, n_layers=L, hkv=hkv)


def test_long_lists():
    _case(6000, 300, 64, torch.bfloat16, one_cluster=True)
    _case(3000, 40, 64, torch.float32, one_cluster=True)


def test_many_slots_and_words_that_do_not_fit():
    _case(140000, 66000, 64, torch.bfloat16)       # 17 + 18 bits: slot and position apart, three passes
    _case(70000, 30000, 64, torch.bfloat16)        # 15 + 17 bits: exactly one word, two passes
    _case(70000, 40000, 64, torch.bfloat16)        # 16 + 17 bits: apart, two passes
