"""Column scores and entropies of observation windows at the edges of the scoring kernels: windows of one to three
32-row blocks with both modalities among their rows, key tiles that end inside a block, grouped and ungrouped heads,
against the fp64 oracle (the rules of parity.py)."""
import pytest

from workloads import generate, get_workload, variant

from parity import check_all, run_gpu

pytestmark = pytest.mark.gpu
TINY = get_workload("tiny")


def _layout(T, W):
    """Vision and text alternate inside the window as well as before it."""
    segs, left, i = [], T, 0
    cut = [max(1, T // 3), max(1, T // 5), 40, 9, 33, 5, 1]
    while left > 0:
        n = min(left, cut[i % len(cut)])
        segs.append(("v", n, i // 2) if i % 2 else ("t", n, -1))
        left -= n
        i += 1
    return tuple(segs)


# few column tiles: the kernels without LDS tiles
FEW_TILES = [
    (129, 31, 2, 2, 128, "bf16"), (160, 64, 1, 4, 128, "bf16"), (257, 33, 2, 7, 64, "bf16"), (300, 96, 1, 3, 128, "bf16"),
    (96, 96, 2, 2, 64, "bf16"), (383, 65, 2, 3, 64, "bf16"), (255, 32, 3, 2, 64, "f32"), (131, 50, 1, 5, 64, "f32"),
    (290, 95, 1, 2, 64, "f32"), (161, 1, 2, 2, 128, "bf16"),
    # many query heads and few key tiles
    (70, 33, 8, 7, 64, "f32"), (130, 64, 8, 8, 128, "bf16"), (200, 32, 12, 1, 64, "bf16"), (65, 16, 32, 1, 64, "f32"),
    (300, 17, 4, 1, 128, "f32"), (257, 40, 1, 32, 64, "bf16"), (33, 20, 5, 3, 128, "f32"),
]
# 33 layers of five tiles or more: the kernels over LDS tiles, pass B / pass A with so many (head, row block) pairs per wave
OVER_TILES = [
    (513, 31, 2, 2, 128, "bf16", "copies, keys in LDS", 1), (600, 1, 1, 4, 64, "bf16", "copies, keys in LDS", 1),
    (515, 31, 1, 3, 64, "f32", "copies, keys in LDS", 1), (513, 33, 1, 2, 128, "bf16", "copies, keys in LDS", 1),
    (513, 40, 1, 2, 64, "f32", "copies, keys in LDS", 1),
    (530, 50, 1, 3, 64, "bf16", "copies", 2), (513, 64, 1, 4, 128, "bf16", "copies", 2), (513, 50, 1, 4, 64, "f32", "copies", 2),
    (520, 95, 1, 2, 128, "bf16", "copies", 2), (515, 70, 2, 3, 64, "f32", "copies", 3), (513, 96, 1, 4, 128, "bf16", "copies", 3),
    (640, 50, 1, 7, 128, "bf16", "copies", 4), (513, 65, 1, 8, 64, "bf16", "copies", 4),
    (640, 40, 3, 1, 128, "bf16", "staged", 1), (577, 17, 2, 1, 64, "bf16", "staged", 1), (513, 97, 1, 2, 128, "bf16", "staged", 2),
    (513, 50, 1, 3, 128, "f32", "staged", 2), (513, 96, 1, 4, 128, "f32", "staged", 2), (520, 33, 2, 1, 128, "f32", "staged", 1),
]
# windows of more than 128 rows: pass-A workgroups of 4, 8 and 16 (head, row block) pairs.  layers, positions, rows, kv heads,
# query heads per kv head, row blocks of a workgroup, pairs per wave
LONG = [
    (2, 400, 129, 8, 4, 1, 1), (2, 300, 200, 2, 1, 4, 1), (20, 300, 160, 8, 4, 2, 2), (41, 300, 160, 8, 4, 4, 4), (41, 333, 161, 6, 5, 3, 4),
    (13, 290, 129, 1, 32, 1, 4),
]


@pytest.mark.parametrize("T,W,hkv,G,d,dtype", FEW_TILES)
def test_window_edges(T, W, hkv, G, d, dtype):
    _check(2, T, W, hkv, G, d, dtype)


@pytest.mark.parametrize("T,W,hkv,G,d,dtype,pass_b,fragments", OVER_TILES)
def test_window_edges_over_tiles(T, W, hkv, G, d, dtype, pass_b, fragments):
    _check(33, T, W, hkv, G, d, dtype, heads=[(l, (l * 5) % hkv) for l in (0, 13, 32)])


@pytest.mark.parametrize("L,T,W,hkv,G,row_blocks,fragments", LONG)
def test_long_windows(L, T, W, hkv, G, row_blocks, fragments):
    _check(L, T, W, hkv, G, 128, "bf16", heads=[(l, (l * 5) % hkv) for l in (0, L - 1)])


def _check(L, T, W, hkv, G, d, dtype, **kw):
    wl = variant(TINY, name=f"win{T}_{W}", n_layers=L, n_q_heads=hkv * G, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                 layout=_layout(T, W), window=W, total_budget=L * max(W, T // 3), seed=T + W, tau_lo=0.3, tau_hi=3.0)
    print(f"[window] L={L} T={T} W={W} Hkv={hkv} G={G} d={d} {dtype}", flush=True)
    data = generate(wl)
    _, gpu = run_gpu(wl, data)
    check_all(wl, data, gpu, verbose=L == 2, **kw)
