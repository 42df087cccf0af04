"""CPU test of the host side of the envs-per-wavefront choice: a number that the
autotuner reports as automatic (its bit of envs_per_wave[0]) follows the batch it
is used for; without the bit it is kept."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "rs_run.hpp"
#include <cstdio>
namespace rs {
int lanes_for(const rs_schedule &, int n) { return pow2_group(n); }
}
int main() {
  for (int marked = 0; marked < 2; ++marked) {
    rs_schedule s{};
    s.envs_per_wave[3] = s.envs_per_wave[8] = 1;  // as spread over idle SIMDs
    s.envs_per_wave[0] = marked << 8;
    int32_t total[17] = {}, lanes[17] = {}, epw[17] = {};
    total[3] = 16384;
    total[8] = 16384;
    for (int n = 2; n <= 16; ++n) {
      lanes[n] = rs::lanes_for(s, n);
      epw[n] = rs::scheduled_envs_per_wave(s, n);
    }
    rs::spread_envs(total, lanes, 1024, epw);
    std::printf("%d %d\n", epw[3], epw[8]);
  }
}
"""


@pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)), reason="needs hipcc")
def test_reported_automatic_choice_follows_the_batch(tmp_path):
    src, exe = tmp_path / "spread.hip", tmp_path / "spread"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2505_06771_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    assert out[0] == "1 1"  # pinned values
    assert out[1] == "1 8"  # the marked one: full wavefronts in a batch that fills the chip
