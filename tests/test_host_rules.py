"""Rules of the host code, on the CPU: small programs compiled against the library's own
headers."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1509_08089_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def _run(tmp_path, source, *link):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                           "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe), *link])
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


def test_tiles_of_claims(tmp_path):
    """A block's claims of a list of tiles run on from the grid's size, every tile once, and
    the failed ones (one a block, up to `tiles`) are all past the list, also where the list
    ends within a grid of 2^32."""
    out = _run(tmp_path, """
#include <cstdio>
#include "kernels.h"
int main() {
  const uint32_t grids[] = {1, 255, 1536, 16384};
  const uint32_t lists[] = {1u << 20, 0xFFFFFFFEu, 0xFFFFFFFFu - 1536, 0xFFFFFFFFu - 16384};
  for (uint32_t g : grids)
    for (uint32_t tiles : lists) {
      for (uint32_t i = 0; i < 40000; ++i) {  // the first and the last claims that get a tile
        if (moss::next_tile(i, g, tiles) != g + i) return 1;
        const uint32_t c = tiles - g - 1 - i;
        if (moss::next_tile(c, g, tiles) != tiles - 1 - i) return 2;
      }
      for (uint32_t i = 0; i < g; ++i)
        if (moss::next_tile(tiles - g + i, g, tiles) < tiles) return 3;
    }
  std::puts("ok");
}
""")
    assert out == "ok\n"
