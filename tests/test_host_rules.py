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


PATH_GRAPH = """
#include <sys/wait.h>
#include <unistd.h>
#include <vector>
#include "hip/hip_runtime.h"
#include "moss.h"
// a path of m edges, made on a device; kernels don't run here, so checked graphs end refused
static moss_status make(int device, int m, uint32_t flags, moss_graph** g) {
  std::vector<int32_t> rp(m + 2), col;
  for (int v = 0; v <= m; ++v) {
    if (v > 0) col.push_back(v - 1);
    if (v < m) col.push_back(v + 1);
    rp[v + 1] = (int32_t)col.size();
  }
  hipSetDevice(device);
  return moss_graph_create(m + 1, (int64_t)col.size(), rp.data(), col.data(), flags, nullptr, g);
}
"""


def test_pinned_words_of_two_devices(tmp_path, fake_hip):
    """The pinned words that a graph's kernels store into belong to its device or to all,
    also where a graph of another device had them before."""
    out = _run(tmp_path, PATH_GRAPH + """
int main() {
  for (int device : {0, 1}) {
    moss_graph* g = nullptr;
    if (make(device, 100, MOSS_TRUST_CSR, &g) != MOSS_OK || moss_graph_destroy(g) != MOSS_OK) return 1;
  }
}
""", fake_hip)
    blocks, used = [], set()
    for f in map(str.split, out.splitlines()):
        if f[:2] == ["host", "block"]:
            at = int(f[4], 16)
            blocks.append((at, at + int(f[5]), int(f[2]), int(f[3])))
        elif f[0] == "copy" and f[2] == "2":  # to the host
            device, to = int(f[1]), int(f[3], 16)
            (owner, flags), = [b[2:] for b in blocks if b[0] <= to < b[1]]
            used.add(device)
            assert owner == device or flags & 1, (owner, device, flags)  # 1: hipHostMallocPortable
    assert used == {0, 1}


def test_memory_of_a_graph(tmp_path, fake_hip):
    """The hub filters' bytes are held where a graph may have them: a checked one of more
    than 2^19 edges.  The bucketed creation's list grows with its buckets."""
    out = _run(tmp_path, PATH_GRAPH + """
int main() {
  for (uint32_t flags : {0u, MOSS_TRUST_CSR})
    for (int m : {(1 << 15) - 8, 1 << 15, 1 << 19, (1 << 19) + 8}) {
      if (fork() == 0) {  // a process each: the library keeps released blocks for the next graph
        moss_graph* g = nullptr;
        (void)make(0, m, flags, &g);
        return 0;
      }
      wait(nullptr);
    }
}
""", fake_hip)
    size = [int(x.split()[3]) for x in out.splitlines() if x.startswith("device block")]
    per_graph = size[1::2]  # a graph's CSR, then its own block
    assert len(size) == 16
    checked, trusted = per_graph[:4], per_graph[4:]
    grain = 2 << 20  # of blocks past 8 MB (64 KB below)
    assert checked[:3] == trusted[:3]
    assert checked[3] - trusted[3] >= 2 * (1 << 19) - grain and checked[3] > trusted[3]
    assert trusted[3] - trusted[2] <= (1 << 19) + grain  # the filter doubles there: half a MB
    assert checked[1] - checked[0] <= 2 * (64 << 10)
