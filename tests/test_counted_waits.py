"""Kernels that wait for asynchronous copies by number (`s_waitcnt vmcnt(n)`, n > 0, behind younger loads) need those loads to
be global ones: a FLAT load counts as an LDS access too and comes back in no order.  Whether a load is FLAT depends on what
the compiler can prove about its address, so the compiled kernels are looked at (gfx950 assembly, no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2502_17599_amd.build import HIPCC_FLAGS, PKG_DIR, ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("source", ["score_accum_dma", "score_accum_blocks", "score_stats_dma"])
def test_kernels_with_counted_waits_have_no_flat_loads(tmp_path, source):
    out = tmp_path / "kernels.asm"
    res = subprocess.run([HIPCC, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), "-S", "--offload-device-only",
                          os.path.join(PKG_DIR, "csrc", source + ".hip"), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    kernels = re.findall(r"^(_ZN4meda\w+):(.*?)^\.Lfunc_end", out.read_text(), re.S | re.M)
    assert kernels
    for name, body in kernels:
        assert "global_load_lds" in body, name
        assert not re.search(r"\bflat_(load|store)", body), name
