"""Selection and budgets at their edges.  Selection: lengths around the sizes at which a workgroup changes its shape
(1024, 4096, 8192, 16384 positions) and beyond, text or vision cuts, many equal scores; the reference is a sort of the
kernel's own column scores (text candidates first, then by score, equal scores by position), so it is exact.
Budgets: one layer to more layers than a wave has lanes, with and without active bounds; the reference is the oracle's
allocator on the kernel's own entropies.
Nearest neighbours of the kernel that works without an LDS copy of the conserved set: against float64 cosines; a
slot counts as right if its cosine is within 1e-5 of the best (sums of up to 128 exact products in fp32, times 1/|k|).
The same where layers with conserved sets held whole in LDS (512 pairs and more) lie between layers with longer ones.
Merged rows: the mean of the members in float64, for outputs below and above 65536 rows; bf16 may differ by one unit in
the last place (2^-7 of the value) because the reference rounds twice.
Row statistics: column scores against a float64 softmax, for 16 to 2052 partials per row; a logit is a sum of 64
products with a magnitude of up to 30, so its error is below 64 * 30 * 2^-24 = 1.2e-4, which is the relative error of
the probability; twice that for both passes."""
import numpy as np
import pytest
import torch

from oracle import meda_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(T, L, hkv, d, dtype, B, W=16, p_text=0.3, duplicates=0, flat=False, seed=0):
    import paper_2502_17599_amd as pkg
    print(f"\n[select/allocate] T={T} L={L} Hkv={hkv} d={d} {dtype} B={B} W={W} text={p_text} dup={duplicates}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(seed)
    k = torch.randn(L, hkv, T, d, generator=g, device=DEV)
    if duplicates:
        k[:, :, torch.randperm(T, generator=g, device=DEV)[:duplicates]] = k[:, :, :1]
    q = torch.randn(L, hkv, W, d, generator=g, device=DEV)
    if not flat:
        q *= torch.linspace(0.2, 6.0, L, device=DEV)[:, None, None, None]
    mask = (torch.rand(T, generator=g, device=DEV) >= p_text).to(torch.uint8)
    comp = pkg.Compressor(pkg.make_params(L, hkv, hkv, d, T, W, B, dtype), DEV, want_merge_assign=True)
    k = k.to(dtype)
    out = comp(q.to(dtype), k, k.clone(), mask)
    torch.cuda.synchronize()
    S, M, N, off = meda_oracle.allocate_budgets(out.entropy.cpu().numpy(), B, T, W)
    assert out.layer_len.cpu().tolist() == S.tolist() and out.layer_off.cpu().tolist() == off.tolist()
    scores = comp.region("col_scores", torch.float32).view(L, hkv, T)
    for l in range(L):
        _, _, idx = out.layer(l)
        s, m = int(S[l]), int(M[l])
        order_class = mask[:T - m].long()
        for h in range(hkv):
            cand = scores[l, h, :T - m]
            order = torch.sort(-cand, stable=True).indices                  # by score, equal ones by position
            order = order[torch.sort(order_class[order], stable=True).indices]  # text first
            want = torch.cat([order[:s - m].sort().values, torch.arange(T - m, T, device=DEV)])
            assert torch.equal(idx[h].long(), want), (l, h)
    return out, k, S, comp


@pytest.mark.parametrize("T", [33, 1023, 1024, 1025, 4095, 4097, 8192, 8193, 16384, 16385, 40001])
@pytest.mark.parametrize("p_text", [0.02, 0.6])
def test_selection_around_the_shapes(T, p_text):
    _run(T, 2, 2, 64, torch.bfloat16, 2 * max(16, T // 5), p_text=p_text)
    _run(T, 2, 1, 64, torch.bfloat16, 2 * max(16, T // 5), p_text=p_text, duplicates=T // 3)


# short prompts, and the workgroups chosen for more than 256 and 512 pairs
@pytest.mark.parametrize("T,L,hkv", [(17, 2, 2), (256, 2, 2), (257, 2, 2), (512, 2, 2), (513, 2, 2), (2048, 3, 1), (2049, 3, 1),
                                     (300, 33, 20), (1025, 33, 20), (2048, 33, 20), (4097, 33, 20), (4100, 20, 20), (16385, 33, 20),
                                     (12000, 3, 1)])
@pytest.mark.parametrize("duplicates", [False, True])
def test_selection_of_short_prompts_and_many_pairs(T, L, hkv, duplicates):
    _run(T, L, hkv, 64, torch.bfloat16, L * max(16, T // 5), p_text=0.1, duplicates=T // 3 if duplicates else 0)


def test_selection_of_one_modality_and_of_nearly_everything():
    for p in (0.0, 1.0):
        _run(1500, 2, 1, 64, torch.float32, 2 * 300, p_text=p)
    _run(5000, 2, 1, 64, torch.bfloat16, 2 * 4999)
    _run(5000, 2, 1, 64, torch.bfloat16, 2 * 16)


@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 200])
def test_budgets(L):
    _run(200, L, 1, 64, torch.bfloat16, L * 60 + L // 2)
    _run(200, L, 1, 64, torch.bfloat16, L * 60 + L // 2, flat=True)
    _run(100, L, 1, 64, torch.bfloat16, L * 90 + L // 3)       # layers at the cap
    _run(200, L, 1, 64, torch.bfloat16, L * 17)                # layers at the floor


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 64), (torch.bfloat16, 128)])
@pytest.mark.parametrize("T,L,hkv", [(40, 1, 1), (97, 2, 3), (1000, 2, 1), (2048, 3, 1), (2049, 3, 1), (700, 5, 8)])
def test_nearest_neighbours(dtype, d, T, L, hkv):
    out, k, _, _ = _run(T, L, hkv, d, dtype, L * max(17, T // 4))
    _check_neighbours(out, k)


# fp32 keys of many positions over all pairs: the kernel that splits them
MANY_FP32 = [(64, 1500, 32, 8, 150), (64, 701, 33, 9, 97), (64, 257, 40, 16, 50), (128, 1500, 16, 8, 300), (128, 385, 13, 11, 40),
             (128, 6500, 3, 2, 1300)]


@pytest.mark.parametrize("d,T,L,hkv,kept", MANY_FP32)
def test_nearest_neighbours_of_many_fp32_pairs(d, T, L, hkv, kept):
    out, k, _, _ = _run(T, L, hkv, d, torch.float32, L * kept)
    _check_neighbours(out, k)
    _check_merged(out, k)


# Ties: one key stands at four conserved positions more than 32 slots apart (different blocks, and different waves of the
# kernels whose waves share the blocks) and at five dropped ones, which have to go to the lowest of the four slots.
# Kept are exactly the text positions and the window (uniform budgets, no recent part), so the slots are known.
TIES = [
    (torch.float32, 64, 1000, 2, 2, 300, "direct"),       # one fragment per wave
    (torch.float32, 64, 990, 8, 8, 300, "direct"),        # two
    (torch.float32, 128, 1000, 2, 2, 300, "direct"),
    (torch.float32, 64, 1000, 8, 8, 300, "split"),
    (torch.float32, 64, 600, 32, 16, 200, "split"),
    (torch.float32, 128, 600, 16, 8, 200, "split"),
    (torch.float32, 128, 600, 48, 8, 200, "split"),       # eight waves
    (torch.bfloat16, 64, 1000, 2, 2, 300, "direct"),
    (torch.bfloat16, 128, 1000, 2, 2, 300, "direct"),
    (torch.bfloat16, 64, 1000, 8, 8, 300, "tiled"),
    (torch.bfloat16, 128, 1000, 8, 8, 300, "tiled"),
    (torch.bfloat16, 64, 600, 32, 8, 200, "tiled"),       # in the order of the sums of sets in LDS
    (torch.bfloat16, 128, 600, 32, 8, 200, "tiled"),
    (torch.bfloat16, 64, 600, 64, 8, 200, "resident"),    # the whole set in LDS
    (torch.bfloat16, 128, 600, 64, 8, 200, "resident")]


@pytest.mark.parametrize("dtype,d,T,L,hkv,kept,kernel", TIES)
def test_equal_keys_go_to_the_lowest_slot(dtype, d, T, L, hkv, kept, kernel):
    import paper_2502_17599_amd as pkg
    print(f"\n[ties] {dtype} d={d} T={T} L={L} Hkv={hkv} kept={kept}", flush=True)
    W = 16
    g = torch.Generator().manual_seed(d + L)
    k = torch.randn(L, hkv, T, d, generator=g).to(dtype)
    text = torch.randperm(T - W, generator=g)[:kept - W].sort().values    # slots 0 .. kept - W - 1
    mask = torch.ones(T, dtype=torch.uint8)
    mask[text] = 0
    dropped = torch.tensor(sorted(set(range(T - W)) - set(text.tolist())))
    lowest = torch.empty(L, hkv, dtype=torch.int64)
    copies = torch.empty(L, hkv, 5, dtype=torch.int64)
    for l in range(L):
        for h in range(hkv):
            first = int(torch.randint(0, kept - W - 3 * 50, (1,), generator=g))
            slots = torch.tensor([first, first + 33, first + 83, first + 3 * 50 - 1])
            copies[l, h] = dropped[torch.randperm(len(dropped), generator=g)[:5]]
            key = torch.randn(d, generator=g).to(dtype)
            k[l, h, text[slots]] = key
            k[l, h, copies[l, h]] = key
            lowest[l, h] = first
    q = torch.randn(L, hkv, W, d, generator=g).to(dtype)
    p = pkg.make_params(L, hkv, hkv, d, T, W, L * kept, dtype, 0, 1, flags=pkg.FLAG_UNIFORM_BUDGET)
    comp = pkg.Compressor(p, DEV, want_merge_assign=True)
    k = k.to(DEV)
    out = comp(q.to(DEV), k, k.clone(), mask.to(DEV))
    torch.cuda.synchronize()
    for l in range(L):
        _, _, idx = out.layer(l)
        assert torch.equal(idx[:, :kept - W].cpu().long(), text.expand(hkv, -1))
    got = out.merge_assign.cpu().long().gather(2, copies)
    assert torch.equal(got, lowest[:, :, None].expand_as(got))


def _check_neighbours(out, k):
    L, hkv = k.shape[:2]
    for l in range(L):
        _, _, idx = out.layer(l)
        for h in range(hkv):
            u = k[l, h].double()
            u = u / u.norm(dim=1, keepdim=True)
            cos = u @ u[idx[h].long()].T
            got = cos.gather(1, out.merge_assign[l, h].long()[:, None])[:, 0]
            assert (got >= cos.max(dim=1).values - 1e-5).all()


SETS_IN_LDS = [(1500, 64, 8, 560), (1500, 130, 4, 300), (700, 64, 8, 33), (3000, 28, 16, 64)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,L,hkv,kept", SETS_IN_LDS)
def test_conserved_sets_in_lds_between_longer_ones(T, L, hkv, kept, d):
    out, k, S, _ = _run(T, L, hkv, d, torch.bfloat16, L * kept)
    if kept == 560 and d == 128:
        assert S.min() <= 576 < S.max()  # rows of 256 bytes and one 1/|k| each: 576 of them fit
    _check_neighbours(out, k)
    _check_merged(out, k)


def _check_merged(out, k):
    L, hkv, T, _ = k.shape
    for l in range(L):
        k_out, v_out, idx = out.layer(l)
        for h in range(hkv):
            pos = idx[h].long()
            slot = out.merge_assign[l, h].long().clone()
            slot[pos] = torch.arange(len(pos), device=DEV)
            x = k[l, h].double()
            n = torch.zeros(len(pos), dtype=torch.float64, device=DEV).index_add_(0, slot, torch.ones(T, dtype=torch.float64, device=DEV))
            want = torch.zeros(len(pos), x.shape[1], dtype=torch.float64, device=DEV).index_add_(0, slot, x) / n[:, None]
            bound = 2.0 ** -7 if k.dtype == torch.bfloat16 else 2.0 ** -23
            for got in (k_out[h], v_out[h]):
                assert ((got.double() - want).abs() <= bound * want.abs() + 1e-12).all(), (l, h)


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 64), (torch.bfloat16, 128)])
@pytest.mark.parametrize("T,L,hkv,kept", [(50, 1, 1, 17), (1001, 3, 5, 203), (700, 33, 8, 250)])
def test_merged_rows(dtype, d, T, L, hkv, kept):
    out, k, _, _ = _run(T, L, hkv, d, dtype, L * kept)
    _check_merged(out, k)


@pytest.mark.parametrize("tiles", [1, 4, 5, 37, 512, 513])
def test_column_scores_with_many_partials(tiles):
    T, L, W = tiles * 128 - 3, 2, 16
    _, k, _, comp = _run(T, L, 1, 64, torch.bfloat16, L * max(W, T // 5), W=W)
    g = torch.Generator(device=DEV).manual_seed(0)
    torch.randn(L, 1, T, 64, generator=g, device=DEV)                       # the keys come first in _run
    q = torch.randn(L, 1, W, 64, generator=g, device=DEV) * torch.linspace(0.2, 6.0, L, device=DEV)[:, None, None, None]
    logits = q.bfloat16().double() @ k.double().transpose(-1, -2) / 8.0
    rows = torch.arange(T - W, T, device=DEV)[:, None]
    logits = logits.masked_fill(torch.arange(T, device=DEV)[None, :] > rows, float("-inf"))
    want = torch.softmax(logits, dim=-1).sum(dim=2)
    got = comp.region("col_scores", torch.float32).view(L, 1, T).double()
    assert ((got - want).abs() <= 2.4e-4 * want + 1e-30).all()
