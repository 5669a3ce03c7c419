"""How much scratch a decoding step asks for (host arithmetic, no GPU): a step whose layers, each cut into equally many
chunks, fit the array of the entry point that allocates nothing has to fit it; a workspace for a larger budget and more
appended rows serves every smaller step; any budget is taken."""
import random

import pytest
import torch

import paper_2502_17599_amd as pkg

LIMIT = pkg.DECODE_NOALLOC_MAX_BYTES


def _bytes(L, hq, hkv, d, B, n_new, dtype=torch.bfloat16):
    return pkg.meda_decode_workspace_bytes(pkg.make_decode_params(L, hq, hkv, d, B, dtype, n_new))


def _even_split_bytes(L, hq, hkv, d, B, n_new):
    """Every layer in as many chunks as its average length holds of 128 rows per query head of the group (up to 4; 64
    chunks at most), the appended rows in chunks of 128."""
    gp = next(p for p in (1, 2, 4, 8) if hq // hkv <= p)
    rows = 128 * min(gp, 4)
    ns = min(64, max(1, -(-(B // L) // rows)))
    return (L * hq * (ns + min(64, -(-n_new // 128))) * (d + 2) * 4 + 255) // 256 * 256


def _shapes(n, seed):
    rng = random.Random(seed)
    while n:
        L = rng.choice([1, 2, rng.randint(3, 100), rng.randint(100, 3000)])
        g = rng.randint(1, 8)
        hkv = rng.choice([1, 2, 4, 8, 16, rng.randint(1, 64)])
        B = L * int(2 ** rng.uniform(0, 15)) + rng.randrange(L)
        n_new = rng.choice([0, 1, rng.randint(1, 300), rng.randint(1, 20000)])
        if L * g * hkv < 1 << 20:
            n -= 1
            yield L, g * hkv, hkv, rng.choice([64, 128]), B, n_new


@pytest.mark.parametrize("shape", [(73, 64, 16, 128, 10681, 2000), (39, 112, 16, 128, 9936, 2000), (19, 64, 8, 128, 5737, 10000),
                                   (10000, 8, 1, 128, 100000, 0)])
def test_steps_near_the_limit_of_the_built_in_scratch(shape):
    assert _even_split_bytes(*shape) <= LIMIT
    assert 0 < _bytes(*shape) <= LIMIT


def test_what_fits_in_an_even_split_fits():
    near = 0
    for shape in _shapes(30000, 1):
        even = _even_split_bytes(*shape)
        near += LIMIT * 3 // 4 < even <= LIMIT
        if even <= LIMIT:
            assert 0 < _bytes(*shape) <= LIMIT and 0 < _bytes(*shape, torch.float32) <= LIMIT, (shape, even)
    assert near > 300


def test_a_workspace_for_more_serves_less():
    for i, (L, hq, hkv, d, B, n_new) in enumerate(_shapes(400, 2)):
        dtype = (torch.bfloat16, torch.float32)[i % 2]
        last = 0
        for b in sorted({L, 2 * L, B // 2 + L, B, B + 1, *(B + i * max(1, B // 37) for i in range(60)), 200 * B}):
            now = _bytes(L, hq, hkv, d, b, n_new, dtype)
            assert now >= last, (L, hq, hkv, d, b, n_new)
            last = now
        last = 0
        for m in (0, 1, 32, 33, 127, 128, 129, 256, 257, 300, 1000, 1025, 5000, 8192, 9000, 20000, 10 ** 6):
            now = _bytes(L, hq, hkv, d, B, m, dtype)
            assert now >= last, (L, hq, hkv, d, B, m)
            last = now
    sizes = [_bytes(32, 32, 8, 128, b, 0) for b in range(20000, 40000, 16)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("B", [1 << 33, 1 << 40, 1 << 60, (1 << 63) - 1])
def test_any_budget_is_taken(B):
    for L, hq, hkv in ((1, 1, 1), (32, 32, 8), (256, 2048, 1024)):
        n = _bytes(L, hq, hkv, 128, B, 5)
        assert 0 < n <= 64 * L * hq * 130 * 4 + 256
