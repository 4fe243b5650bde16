"""Pivots per work item of the hypothesis kernel, on the host (no GPU): items shrink only as far as they all run
at once, and no further than one pass over the matches needs."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "common.h"
using namespace tr;

int main()
{
    for (int slots : {64, 256, 512})
        for (int B : {1, 2, 7, 40, 100, 150, 300})
            for (int k1 : {1, 3, 16, 32, 100, 130, 250, 255, 257, 550, 1000, 2500})
                for (int k2 = 1; k2 <= 8; ++k2)
                    for (int ppw = 4; ppw <= 16; ppw += 4) {
                        const int p = hyp_item_pivots(B, k1, k2, ppw, slots);
                        auto items = [&](int q) { return (long long)B * ((k1 + q - 1) / q); };
                        const bool ok = p >= 1 && p <= ppw && (p == ppw || items(p) <= slots) &&
                                        (p == 1 || p * k2 <= 8 || items(p / 2) > slots);
                        if (!ok) {
                            std::printf("B %d k1 %d k2 %d ppw %d slots %d: %d\n", B, k1, k2, ppw, slots, p);
                            return 1;
                        }
                    }
    std::puts("ok");
    return 0;
}
"""


def test_items_run_in_one_round(tmp_path):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not found")
    src, exe = str(tmp_path / "rule.cpp"), str(tmp_path / "rule")
    with open(src, "w") as f:
        f.write(SOURCE)
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "paper_2507_01439_amd", "csrc"), "-x", "hip", src, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
