"""The SC2 bit-count kernel's tile edge, on the host (no GPU): lists that one round of 256 x 256 tiles holds
take the product, and every longer list gets an edge that no other beats under the rule's cost."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "common.h"
using namespace tr;

static int edge_of(const std::vector<int> &ns, int cus)
{
    int32_t t[kSpEdges] = {};
    for (int n : ns)
        for (int k = 0; k < kSpEdges; ++k) t[k] += (int32_t)stage_items(kSp, n, 0, 256 * (k + 1));
    return sparse_tile(t, cus);
}

static int fail(const char *what, int n, int B, int got)
{
    std::printf("%s: n %d B %d edge %d\n", what, n, B, got);
    return 1;
}

int main()
{
    for (int cus : {256, 64})
        for (int B : {1, 2, 4, 16, 64, 300})
            for (int n = 3; n <= 32767; n += n < 3000 ? 61 : 977) {
                const int S = edge_of(std::vector<int>(B, n), cus);
                const long long nb = (n + 255) / 256, tiles = B * (nb * (nb + 1) / 2);
                if ((S == 0) != (tiles <= cus)) return fail("short list", n, B, S);
                if (S == 0) continue;
                if (S % 256 || S < 256 || S > 1024) return fail("edge", n, B, S);
                auto cost = [&](long long e) {
                    const long long b = (n + e - 1) / e;
                    return (B * (b * (b + 1) / 2) + cus - 1) / cus * (e * e + (1 << 17));
                };
                for (int e = 256; e <= 1024; e += 256)
                    if (cost(e) < cost(S)) return fail("cost", n, B, S);
            }
    // the pairs' own sizes count: sixteen of 1000 matches are a short list, a large one beside them is not
    std::vector<int> ns(16, 1000);
    if (edge_of(ns, 256) != 0) return fail("sixteen of 1000", 1000, 16, edge_of(ns, 256));
    ns[3] = 20000;
    if (edge_of(ns, 256) < 512) return fail("one of 20000", 20000, 16, edge_of(ns, 256));
    if (stage_items(kSp, 5000, 0, 0) != 0) return fail("no tiles", 5000, 1, 0);
    std::puts("ok");
    return 0;
}
"""


def test_edges_of_short_and_long_lists(tmp_path):
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
