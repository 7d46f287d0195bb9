"""Launch shapes chosen on the host (CPU): fs_api.cpp built with the launcher stubs, its pass
configurations printed by a small program."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

MAIN = r"""
#include <cstdio>
#include "%s/paper_2609_32525_amd/csrc/fs_internal.h"
int main() {
  // samples, points, heads, width, slots, bf16
  const long long shapes[][6] = {{1024, 1024, 8, 32, 32, 0}, {64, 2048, 8, 32, 1024, 1},
                                 {768, 1024, 8, 16, 64, 1}, {1, 1 << 22, 8, 32, 64, 1},
                                 {1, 1 << 20, 8, 32, 64, 1}, {1, 4096, 8, 16, 32, 0}};
  for (auto& s : shapes) {
    fs::Geom g{};
    g.B = s[0]; g.N = s[1]; g.H = (int)s[2]; g.D = g.V = (int)s[3]; g.G = (int)s[4]; g.bf16 = s[5] != 0;
    const fs::Pass passes[] = {fs::PASS_SLICE, fs::PASS_DESLICE, fs::PASS_BWD_A, fs::PASS_BWD_B};
    for (auto p : passes) {
      const fs::PassCfg c = fs::pick_cfg(g, p);
      std::printf("%%d %%lld ", c.group ? 1 : 0, (long long)c.chunks * g.BH() * c.nblk);
    }
    std::printf("\n");
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs the GNU host compiler")
def test_grids_of_several_waves_are_grouped(tmp_path):
    """Workgroups that read the same rows are dispatched together on every grid above 4096
    workgroups, whichever pass and however it got so large, and on long capped streams of the
    deslice; grids resident in one wave keep the plain numbering."""
    main = tmp_path / "shapes.cpp"
    main.write_text(MAIN % ROOT)
    exe = str(tmp_path / "shapes")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), str(main),
                    os.path.join(ROOT, "paper_2609_32525_amd", "csrc", "fs_api.cpp"),
                    os.path.join(HERE, "asan", "abi_stubs.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    rows = [list(map(int, l.split())) for l in out.splitlines()]
    assert len(rows) == 6
    for i, row in enumerate(rows):
        for p, (group, grid) in enumerate(zip(row[::2], row[1::2])):
            capped = i == 3 and p == 1
            assert group == int(grid > 4096 or capped), (i, p, group, grid)
    assert min(rows[0][1::2]) > 4096 and min(rows[2][1::2]) > 4096
    assert rows[3][3] <= 4096 and max(rows[4][1::2] + rows[5][1::2]) <= 4096
