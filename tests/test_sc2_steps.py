"""The dense SC2 product's loads of C stay inside the pair's bits: the kernel's loop over steps of 256
columns, replayed on the host with the kernel's own offsets (no GPU)."""
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
    for (int64_t npad = kSc2Tile; npad <= 32768; npad += kSc2Tile) {
        const uint32_t kbs = (uint32_t)npad * 16;   // bytes of one 128-column block over all rows
        const int ns = (int)(kbs >> 12);
        const int64_t lane = (int64_t)kbs + (npad - 1) * 16;   // the last row's piece of a step's second block
        int64_t most = 0;
        auto load = [&](int s) {
            const int64_t at = sc2_step_offset(s, ns, kbs);
            if (at < 0) most = INT64_MAX / 2;
            if (at + lane + 16 > most) most = at + lane + 16;
            if (s < ns && at != (int64_t)s * 2 * kbs) most = INT64_MAX / 2;   // a step the product uses
        };
        load(0);
        load(1);
        for (int s = 0; s + 1 < ns; s += 2) {
            load(s + 2);
            load(s + 3);
        }
        if (most > npad * npad / 8) {
            std::printf("npad %lld: reads up to byte %lld of %lld\n", (long long)npad, (long long)most,
                        (long long)(npad * npad / 8));
            return 1;
        }
    }
    std::puts("ok");
    return 0;
}
"""


def test_loads_of_the_dense_product_stay_inside_c(tmp_path):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not found")
    src, exe = str(tmp_path / "steps.cpp"), str(tmp_path / "steps")
    with open(src, "w") as f:
        f.write(SOURCE)
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "paper_2507_01439_amd", "csrc"), "-x", "hip", src, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
