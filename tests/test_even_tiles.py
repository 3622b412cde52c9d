"""The host's word on launches of both experts that no routing gives lower tiles, against what the workgroups work out, for every routing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include "gemm_mfma.h"
using namespace sa;
template <int BM_S, int BM_M, int OCC>
int look(long n, int N, int cg_s, int cg_m, int *never) {
    GemmArgs s, m;
    s.N = m.N = N;
    s.share_out(128, cg_s);
    m.share_out(128, cg_m);
    const bool may = may_be_even<BM_S, BM_M, OCC>(s, m, n);
    const long fewest = least_tiles<BM_S, BM_M>(s, m, n);
    if (!may) ++*never;
    auto tiles = [](const GemmArgs &g, long rows, long bm) { return ((rows + bm - 1) / bm + (8 >> g.log_groups) - 1) / (8 >> g.log_groups) * g.cols_per_group; };
    int wrong = 0;
    for (long ns = 0; ns <= n; ++ns) {
        const long rest = tiles(m, n - ns, BM_M);
        if (!may && even_rows<BM_S, OCC>((uint32_t)ns, s, (uint32_t)rest) != ns) ++wrong;
        if (tiles(s, ns, BM_S) + rest < fewest) ++wrong;
    }
    if (wrong) printf("%ld rows, %d columns, %d and %d groups: %d\n", n, N, cg_s, cg_m, wrong);
    return wrong;
}
int main() {
    int wrong = 0, never = 0, all = 0;
    for (int N : {64, 100, 320, 384, 768, 1152, 3072})
        for (int cg_s : {1, 2, 4, 8})
            for (int cg_m : {1, 4})
                for (long n = 1; n < 30000; n = n * 5 / 4 + 3) {
                    wrong += look<128, 128, 3>(n, N, cg_s, cg_m, &never) + look<192, 128, 2>(n, N, cg_s, cg_m, &never);
                    all += 2;
                }
    printf("wrong %d never %d all %d\n", wrong, never, all);
    return wrong != 0 || never * 10 < all || never * 10 > all * 9;
}
"""


def test_launches_without_lower_tiles_never_have_them(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "driver.hip", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.check_call([hipcc, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-function",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2306_06446_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
