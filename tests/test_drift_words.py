"""Words of a drift record (host functions of dem_device.hpp, compiled for the
CPU): at most 64 wavefronts of a force launch raise one word, up to the words
that a record has, and no more words than that needs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include "dem_device.hpp"
using namespace demgpu;
int main() {
  for (int64_t n = 1; n <= kMaxParticles; n += 1 + n / 997) {
    const int words = drift_words_for(n), lanes = force_lanes(n);
    const int64_t waves = (n * lanes + 63) / 64;
    if (words < 1 || words > kDriftSpread || (words & (words - 1)) ||
        (words < kDriftSpread && waves > 64 * words) || (words > 1 && waves <= 32 * words)) {
      std::printf("n %ld: %d words for %ld wavefronts\n", (long)n, words, (long)waves);
      return 1;
    }
  }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_wavefronts_to_a_drift_word(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2106_09576_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
