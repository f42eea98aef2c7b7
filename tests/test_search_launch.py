"""Launch arithmetic of the contact search (host functions of dem_device.hpp,
compiled for the CPU): for every number of particles and of search blocks that
a context can have, the workgroups suffice for the blocks that are gone through
and their threads stay below the 2^32 of one launch; for every mean row, what a
workgroup keeps in LDS stays below 64 KB."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include "dem_device.hpp"
using namespace demgpu;
int main() {
  long checked = 0;
  for (int64_t n0 = 1; n0 <= kMaxParticles; n0 *= 2)
    for (int64_t dn = -1; dn <= 1; ++dn)
      for (int64_t b0 = 1; b0 <= (int64_t)1 << 30; b0 *= 2)
        for (int64_t db = -1; db <= 1; ++db)
          for (int fits = 0; fits < 2; ++fits) {
            const int64_t n = n0 + dn, nb = b0 + db;
            if (n < 1 || n > kMaxParticles || nb < 1 || nb > (int64_t)1 << 30) continue;
            const int way = search_way(n, nb, fits != 0);
            if (way == kSearchEach) continue;
            const int64_t wg = search_workgroups(n, nb, way);
            // blocks to go through: every one, or the occupied ones of a search
            // that stays with blocks
            const int64_t most = way == kSearchBlocks ? nb : (n / kBlockMin < nb ? n / kBlockMin : nb);
            if (wg < 1 || wg < most || wg * kBlock >= (int64_t)1 << 32 || wg > nb ||
                (nb + kBlock - 1) / kBlock * kBlock >= (int64_t)1 << 32) {
              std::printf("n %ld blocks %ld fits %d: %ld workgroups\n", (long)n, (long)nb, fits, (long)wg);
              return 1;
            }
            ++checked;
          }
  for (double row = 1e-3; row < 1e300; row *= 1.01) {
    // 256 lists of 2 bytes an entry beside the region's stage, rows of 4 bytes
    const int list = list_capacity(row);
    const double l = 1.5 * row, r = 1.2 * row;
    if (list < 1 || list != (l < 87.0 ? (int)l + 1 : 88) || 18 * 1024 + 512 * list > 64 * 1024) {
      std::printf("row %g: list of %d\n", row, list);
      return 1;
    }
    for (int max_nb : {1, 16, 44, 47, 48, 49, 4096}) {
      const int cap = row_capacity(row, max_nb), want = r < 46.0 ? (int)r + 2 : 48;
      if (cap != (want < max_nb ? want : max_nb) || cap < 1 || 1024 * cap > 64 * 1024) {
        std::printf("row %g, %d neighbours: row of %d\n", row, max_nb, cap);
        return 1;
      }
    }
  }
  std::printf("%ld launches\n", checked);
  return checked > 500 ? 0 : 1;
}
"""


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_search_launches_stay_in_range(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2106_09576_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
