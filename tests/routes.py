"""Which kernels a pass takes (helper, not a test): the plan's own answer, from a small native program linked with the host
side of the library.  Tests that mean a certain kernel assert its route, so that a moved rule cannot leave them behind."""
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SIMILARITY = ("direct", "tiled", "resident", "split")

# pass_a, pass_b, similarity: kernel names; row_blocks: 32-row blocks of the window, or of a pass-A workgroup in the row-block
# mode; fragments: (head, row block) pairs a wave of pass A keeps; waves at work; groups: row blocks of pass A
Route = namedtuple("Route", "pass_a pass_b row_blocks fragments waves groups similarity")


@functools.lru_cache(maxsize=None)
def _program():
    exe = os.path.join(tempfile.mkdtemp(prefix="plan_routes_"), "plan_routes")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "plan_routes.cpp"),
                    os.path.join(ROOT, "paper_2502_17599_amd", "csrc", "meda_api.hip"), "-o", exe],
                   check=True, capture_output=True)
    return exe


def routes(shapes):
    """One Route per (L, Hq, Hkv, d, T, W, B, "f32" or "bf16", flags, n_seqs)."""
    text = "".join(" ".join(str({"f32": 0, "bf16": 1}.get(x, x)) for x in s) + "\n" for s in shapes)
    lines = subprocess.run([_program()], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(shapes)
    out = []
    for s, line in zip(shapes, lines):
        assert not line.startswith("status"), (s, line)
        direct, blocks, rb, rba, nq, waves, groups, sim = (int(x) for x in line.split())
        L, hq, hkv, d, T, W, B, dtype, flags, n = s
        row_bytes, G = d * (4 if dtype == "f32" else 2), hq // hkv
        if direct:
            a = b = "direct"
        elif blocks:
            a = "copies" if row_bytes <= 256 else "staged"
            lds = 3 * 128 * row_bytes * 17 // 16 + 2 * 2048 + 512 * hkv + 1024 + 128     # a key tile, two stages, column sums
            b = "blocks" if row_bytes <= 256 and lds <= 160 * 1024 else "staged"
        else:
            a = "copies" if row_bytes <= 256 and G >= 2 else "staged"
            b = "staged" if row_bytes > 256 or G == 1 or rb > 3 else "copies, keys in LDS" if rb == 1 or (rb == 2 and G == 2) else "copies"
        out.append(Route(a, b, rba if blocks else rb, nq, waves, groups, SIMILARITY[sim]))
    return out


def route(*shape):
    return routes([shape])[0]
