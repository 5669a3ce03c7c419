"""Nearest conserved key of fp32 keys against float64, and near ties against the fp32 instruction, at sizes of the direct
kernel and of the kernel that multiplies the keys in three bf16 parts: one and several tiles, a part of a tile, rows that do
not fill a block."""
import pytest
import torch

import paper_2502_17599_amd as pkg

pytestmark = pytest.mark.gpu


def _run(L, hkv, T, d, kept, k, q0, scale=1.0):
    dev = torch.device("cuda:0")
    W = min(T, 16)
    B = max(L * W, int(kept * L * T))
    g = torch.Generator().manual_seed(5)
    q = torch.randn(L, hkv, W, d, generator=g) * torch.linspace(0.3, 3.0, L)[:, None, None, None]
    q[..., 0] *= q0
    q *= scale
    mask = torch.zeros(T, dtype=torch.uint8)
    mask[T // 4:T // 2] = 1
    comp = pkg.Compressor(pkg.make_params(L, hkv, hkv, d, T, W, B, torch.float32), dev, want_merge_assign=True)
    out = comp(q.to(dev), k.to(dev), k.to(dev), mask.to(dev))
    S, off = out.layer_len.cpu().tolist(), out.layer_off.cpu().tolist()
    sel, slot = out.sel_idx.cpu().long(), out.merge_assign.cpu().long().reshape(L, hkv, T)
    for l in range(L):
        for h in range(hkv):
            at = off[l] * hkv + h * S[l]
            yield l, h, sel[at:at + S[l]], slot[l, h]


DIRECT = [  # layers, kv heads, positions, head dimension, share kept
    (1, 1, 33, 64, 0.5), (2, 4, 257, 64, 0.3), (3, 8, 700, 64, 0.25), (2, 20, 300, 64, 0.2), (1, 2, 65, 128, 0.5), (4, 16, 520, 64, 0.3),
]
SPLIT = [  # sets of one and of many tiles, row blocks of 128 and 256 with a remainder, few and many pairs
    (2, 24, 500, 128, 0.1), (8, 32, 600, 128, 0.12), (32, 32, 65, 64, 0.5), (1, 4, 9001, 64, 0.05), (8, 8, 1111, 64, 0.35),
    (48, 32, 33, 128, 0.55), (2, 24, 553, 128, 0.15),
]
SHAPES = DIRECT + SPLIT


@pytest.mark.parametrize("near", [0.0, 5e-2], ids=["spread", "near"])
@pytest.mark.parametrize("L,hkv,T,d,kept", SHAPES)
def test_nearest_key_of_fp32_keys(L, hkv, T, d, kept, near):
    k = torch.randn(L, hkv, T, d, generator=torch.Generator().manual_seed(T))
    if near:
        k = torch.randn(L, hkv, 1, d, generator=torch.Generator().manual_seed(T + 7)) + near * k
    # Two similarities, each with d fused multiply-adds and 12 more roundings (norm, root, reciprocal, scaling) of 2^-24
    bound = 2 * (d + 12) * 2.0 ** -24
    for l, h, sel, slot in _run(L, hkv, T, d, kept, k, 1.0):
        u = torch.nn.functional.normalize(k[l, h].double(), dim=1)
        less = torch.ones(T, dtype=torch.bool)
        less[sel] = False
        if not bool(less.any()):
            continue
        sim = u[less] @ u[sel].T
        got = sim.gather(1, slot[less][:, None])[:, 0]
        assert float((sim.max(1).values - got).max()) <= bound, (l, h)
        # (no one slot would do for all rows)
        assert float((sim.max(1, keepdim=True).values - sim).max(0).values.min()) > 3 * bound


@pytest.mark.parametrize("near", [0.0, 3e-4, 3e-3], ids=["spread", "all_near", "many_near"])
@pytest.mark.parametrize("L,hkv,T,d,kept", SHAPES)
def test_near_ties_fall_as_with_the_fp32_instruction(L, hkv, T, d, kept, near):
    """The same keys twice: as they are, and with a last key (always conserved) that has no three parts and is the nearest
    of no row, which sends every workgroup over the whole set with the fp32 instruction."""
    g = torch.Generator().manual_seed(3 * T)
    centres = torch.randn(L, hkv, 1 if near else 4, d, generator=g)
    k = centres.repeat(1, 1, T // centres.shape[2] + 1, 1)[:, :, :T] + (near or 0.3) * torch.randn(L, hkv, T, d, generator=g)
    if not near:  # copies of two keys, as the selection finds them, and of one that is the nearest of many rows
        k[:, :, 5::7], k[:, :, 6::11] = k[:, :, 5:6], k[:, :, 6:7]
        k[:, :, 3::9] = centres[:, :, 3:4]
    k[..., 0] = 0.1
    k[:, :, -1] = -3.0 * centres.sum(2)
    plain, fp32 = k.clone(), k.clone()
    plain[:, :, -1, 0] = -0.1
    fp32[:, :, -1, 0] = 3.4e38
    for (l, h, sel, slot), (_, _, sel32, slot32) in zip(_run(L, hkv, T, d, kept, plain, 0.0), _run(L, hkv, T, d, kept, fp32, 0.0)):
        assert torch.equal(sel, sel32) and int(sel[-1]) == T - 1
        assert torch.equal(slot, slot32), (l, h, int((slot != slot32).sum()))


@pytest.mark.parametrize("L,hkv,T,d,kept", SHAPES)
def test_keys_that_have_no_three_parts(L, hkv, T, d, kept):
    """An element that rounds to an infinite bf16: its (finite) products still decide where the row goes."""
    # elements of 0.1: the raw product with a large row, at most 3.4e38 * 0.6, stays below the largest float
    k = 0.1 * torch.randn(L, hkv, T, d, generator=torch.Generator().manual_seed(T + 1))
    big = torch.arange(0, T, 5)
    k[:, :, big, 0] = 3.4e38
    for l, h, sel, slot in _run(L, hkv, T, d, kept, k, 0.0):
        x = k[l, h].double()
        # 1 / |k| of a key whose sum of squares overflows is 0: it can win only where every other similarity is negative
        inv = x[sel].norm(dim=1).reciprocal() * (x[sel, 0] < 1e38)
        less = torch.ones(T, dtype=torch.bool)
        less[sel] = False
        rows = torch.nonzero(less & (x[:, 0] > 1e38)).flatten()
        for r in rows.tolist():
            sim = (x[sel] @ x[r]) * inv
            sim[x[sel, 0] > 1e38] = -1.0     # their product with this row overflows, times 0: no similarity
            assert sim[slot[r]] >= sim.max() * (1 - 1e-5), (l, h, r)


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("L,hkv,T,d,kept", SPLIT)
def test_keys_too_short_to_split(L, hkv, T, d, kept, zero):
    """The same keys times 2^-45 (the queries times 2^45, so that the same ones are conserved): below the lengths that are
    split, so with the fp32 instruction alone; the powers of two change no rounding.  With a few keys of length 0 as well,
    which are as near to every key, and to which every key is as near, as the lowest slot."""
    g = torch.Generator().manual_seed(T + 3)
    k = torch.randn(L, hkv, 1, d, generator=g) + 0.3 * torch.randn(L, hkv, T, d, generator=g)
    if zero:
        k[:, :, T // 3::T // 3] = 0.0
    runs = zip(_run(L, hkv, T, d, kept, k, 1.0), _run(L, hkv, T, d, kept, k * 2.0 ** -45, 1.0, 2.0 ** 45))
    for (l, h, sel, slot), (_, _, sel_short, slot_short) in runs:
        assert torch.equal(sel, sel_short)
        assert torch.equal(slot, slot_short), (l, h, int((slot != slot_short).sum()))
        less = torch.ones(T, dtype=torch.bool)
        less[sel] = False
        assert bool((slot[less & (k[l, h] == 0).all(1)] == 0).all())
