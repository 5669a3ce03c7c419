"""The shapes of the GPU tests reach the kernels that the tests are about (host arithmetic and the library's own plan, no GPU)."""
import os

import pytest
import torch

import test_gpu_full_prompt
import test_gpu_parity
import test_gpu_random_shapes
import test_gpu_score_windows as windows
import test_gpu_select_allocate as select
import test_gpu_similarity_split as split
from routes import HIPCC, routes
from workloads import get_workload

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
DTYPE = {torch.float32: "f32", torch.bfloat16: "bf16"}
FULL_PROMPT = 4


def _windows(L, cases, B=None):
    return routes([(L, hkv * G, hkv, d, T, W, L * max(W, T // 3), dtype, 0, 0) for T, W, hkv, G, d, dtype in cases])


def test_scoring_windows():
    for case, r in zip(windows.FEW_TILES, _windows(2, windows.FEW_TILES)):
        assert r.pass_b == "direct" or case[3] * ((case[1] + 31) // 32) > 32, (case, r)
    got = _windows(33, [c[:6] for c in windows.OVER_TILES])
    for case, r in zip(windows.OVER_TILES, got):
        assert (r.pass_b, r.fragments) == case[6:], (case, r)
    # every form of the kernels fed by copies, with padded and with full windows, in 16 and in 32 bits
    forms = {(r.pass_b, r.row_blocks) for r in got}
    assert {("copies, keys in LDS", 1), ("copies, keys in LDS", 2), ("copies", 2), ("copies", 3), ("staged", 1), ("staged", 2)} <= forms
    assert {r.waves > 4 for r in got if r.pass_a == "copies" and r.fragments == 4} == {False, True}
    assert any(r.waves > 4 and r.pass_a == "staged" for r in got)


def test_long_windows():
    got = routes([(L, hkv * G, hkv, 128, T, W, L * max(W, T // 3), "bf16", 0, 0) for L, T, W, hkv, G, *_ in windows.LONG])
    for case, r in zip(windows.LONG, got):
        assert (r.pass_a, r.row_blocks, r.fragments) == ("copies", *case[5:]), (case, r)


def test_full_prompts():
    cases = test_gpu_full_prompt.LARGE
    got = routes([(L, hkv * G, hkv, 128, T, 16, L * 60, "bf16", FULL_PROMPT, 0) for L, T, hkv, G, *_ in cases])
    for case, r in zip(cases, got):
        assert (r.row_blocks, r.fragments, r.groups, r.pass_b) == (*case[4:], "blocks"), (case, r)
    w = get_workload("llava7b_multi_image")
    big, = routes([(w.n_layers, w.n_q_heads, w.n_kv_heads, w.head_dim, w.seq_len, w.window, w.total_budget, w.dtype, FULL_PROMPT, 0)])
    assert got[0][:5] == big[:5]    # the first case runs the kernels of the benchmarked shape


def test_similarity():
    def sims(shapes):
        return [r.similarity for r in routes(shapes)]
    assert set(sims([(L, h, h, d, T, min(T, 16), max(L * min(T, 16), int(kept * L * T)), "f32", 0, 0)
                     for L, h, T, d, kept in split.DIRECT])) == {"direct"}
    assert set(sims([(L, h, h, d, T, min(T, 16), max(L * min(T, 16), int(kept * L * T)), "f32", 0, 0)
                     for L, h, T, d, kept in split.SPLIT])) == {"split"}
    assert set(sims([(L, h, h, d, T, 16, L * kept, "f32", 0, 0) for d, T, L, h, kept in select.MANY_FP32])) == {"split"}
    got = sims([(L, h, h, d, T, 16, L * kept, DTYPE[dt], 1, 0) for dt, d, T, L, h, kept, _ in select.TIES])
    assert got == [c[-1] for c in select.TIES]
    shapes = [(L, h, h, 128, T, 16, L * kept, "bf16", 0, 0) for T, L, h, kept in select.SETS_IN_LDS]
    assert set(sims(shapes)) == {"resident"}
    L = test_gpu_parity.RESIDENT_LAYERS
    assert sims([(L, 32, 32, 128, 2048, 32, L * 600, "bf16", 0, 0)]) == ["resident"]
    got = [(w.dtype, *sims([(w.n_layers, w.n_q_heads, w.n_kv_heads, w.head_dim, w.seq_len, w.window, w.total_budget, w.dtype, 0, 0)]))
           for w in test_gpu_random_shapes._many_pairs_configs()]
    assert ("bf16", "resident") in got and set(got) <= {("bf16", "resident"), ("bf16", "tiled"), ("f32", "split")}, got
