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


@pytest.mark.parametrize("T,W,hkv,G,d,dtype", [
    (129, 31, 2, 2, 128, "bf16"), (160, 64, 1, 4, 128, "bf16"), (257, 33, 2, 7, 64, "bf16"), (300, 96, 1, 3, 128, "bf16"),
    (96, 96, 2, 2, 64, "bf16"), (383, 65, 2, 3, 64, "bf16"), (255, 32, 3, 2, 64, "f32"), (131, 50, 1, 5, 64, "f32"),
    (290, 95, 1, 2, 64, "f32"), (161, 1, 2, 2, 128, "bf16"),
    # many query heads and few key tiles
    (70, 33, 8, 7, 64, "f32"), (130, 64, 8, 8, 128, "bf16"), (200, 32, 12, 1, 64, "bf16"), (65, 16, 32, 1, 64, "f32"),
    (300, 17, 4, 1, 128, "f32"), (257, 40, 1, 32, 64, "bf16"), (33, 20, 5, 3, 128, "f32"),
])
def test_window_edges(T, W, hkv, G, d, dtype):
    L = 2
    wl = variant(TINY, name=f"win{T}_{W}", n_layers=L, n_q_heads=hkv * G, n_kv_heads=hkv, head_dim=d, dtype=dtype,
                 layout=_layout(T, W), window=W, total_budget=L * max(W, T // 3), seed=T + W, tau_lo=0.3, tau_hi=3.0)
    print(f"[window] T={T} W={W} Hkv={hkv} G={G} d={d} {dtype}", flush=True)
    data = generate(wl)
    _, gpu = run_gpu(wl, data)
    check_all(wl, data, gpu)
