"""Rules of the host code, on the CPU: small programs compiled against the library's own
headers and, where they call it, linked with a stand-in for the HIP runtime (fake_hip.c)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1509_08089_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
LIB = os.path.join(ROOT, "paper_1509_08089_amd", "libmoss.so")


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    """Folder of the stand-in, under the runtime's name."""
    where = tmp_path_factory.mktemp("hip")
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-w", "-Wl,-soname,libamdhip64.so.7",
                           os.path.join(ROOT, "tests", "fake_hip.c"), "-o", str(where / "libamdhip64.so.7")])
    return str(where)


def _run(tmp_path, source, hip=None):
    """The output of a program, linked with the library on the stand-in in folder `hip`."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    link = [LIB, os.path.join(hip, "libamdhip64.so.7"), "-Wl,-rpath," + os.path.dirname(LIB),
            "-Wl,--unresolved-symbols=ignore-in-shared-libs"] if hip else []  # the stand-in's symbols have no version
    src.write_text(source)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                           "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe), *link])
    env = {**os.environ, "LD_LIBRARY_PATH": hip} if hip else None
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, env=env).stdout


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


@pytest.mark.parametrize("words", [22, 2**32 - 1, 2**32 + 5, 22 * (2**32 - 1)])
def test_histogram_words_of_a_batch(tmp_path, fake_hip, words):
    """A batch has 22 words a slot and as many slots as memory holds: the kernels that clear
    and collect them count beyond 32 bits."""
    out = _run(tmp_path, """
#include "kernels.h"
int main() {
  const uint64_t words = %dull;
  if (moss::launch_batch_stage(nullptr, nullptr, 64, nullptr, words, nullptr, nullptr) != hipSuccess) return 1;
  if (moss::launch_batch_collect(nullptr, words, nullptr, nullptr, 1, nullptr) != hipSuccess) return 2;
}
""" % words, fake_hip)
    assert [x for x in out.splitlines() if x.startswith("words")] == ["words %d" % words] * 2
