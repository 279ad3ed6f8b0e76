"""Hub filters of long rows, which many blocks fill together: classes are the oracle's on rows
at the largest size that one block puts together (16,384 entries) and past it, beginning and
ending inside spans, one after another; and a row of 2^20 entries takes the table build no
more than a few times as long as without filters."""
import time

import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import ORACLE_SAMPLER
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu

HUBS = (16_384, 16_449, 16_500, 70_001, 300)  # rows 0 to 4: they follow one another in the CSR


@pytest.fixture(scope="module")
def graph():
    rng = np.random.Generator(np.random.PCG64(12))
    n, core = 90_000, 10 + np.arange(250)  # every hub has the whole core
    e = [np.stack([np.full(d, h), np.concatenate([core, 300 + rng.choice(n - 300, d - 250, replace=False)])], 1)
         for h, d in enumerate(HUBS)]
    a, b = np.triu_indices(250, 1)
    e.append(np.stack([core[a], core[b]], 1)[rng.random(len(a)) < 0.7])
    e.append(300 + rng.integers(0, n - 300, (440_000, 2)))
    e = np.concatenate(e)
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], 1), axis=0)
    g = gg.from_edges(n, e, "long hubs")
    assert g.nnz // 2 > 1 << 19 and tuple(np.diff(g.row_ptr)[:5]) == HUBS
    return g


@pytest.mark.parametrize("sampler", [moss.MOSS_SAMPLER_MOSS4, moss.MOSS_SAMPLER_MOSS4MIN, moss.MOSS_SAMPLER_T5,
                                     moss.MOSS_SAMPLER_PATH5])
def test_long_rows_classes(graph, sampler):
    G, og = moss.Graph(graph), oracle.Graph(graph)
    n = 20_011
    cls = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    hits = G.sample_range(sampler, 3, 0, n, cls)
    osid = ORACLE_SAMPLER[sampler]
    want = np.array([og.sample(osid, 3, k)[0] for k in range(n)], dtype=np.uint8)
    np.testing.assert_array_equal(cls.cpu().numpy(), want)
    np.testing.assert_array_equal(hits, og.run(osid, 3, 0, n, 8))
    assert len(np.unique(want)) > 3


def test_build_time_of_the_longest_row():
    """One pass over the row's entries is less than the other passes take together, so a
    factor of 3 is generous; a pass for every 16,384 entries is some hundred times it."""
    d = 1 << 20
    n = d + 1
    rng = np.random.Generator(np.random.PCG64(13))
    e = np.stack([np.zeros(d, np.int64), 1 + np.arange(d)], 1)
    rest = 1 + rng.integers(0, d, (200_000, 2))
    e = np.unique(np.sort(np.concatenate([e, rest[rest[:, 0] != rest[:, 1]]]), 1), axis=0)
    csr = gg.from_edges(n, e, "star")
    t = [torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda() for x in (csr.row_ptr, csr.col)]

    def best(flags):
        times = []
        for _ in range(5):
            G = moss.Graph.from_device(*t, flags=flags)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            G.build_tables(moss.MOSS_TABLES_K4)
            times.append(time.perf_counter() - t0)
            G.close()
        return min(times)

    without, with_filters = best(moss.MOSS_TRUST_CSR), best(0)
    print(f"without {1e6 * without:.0f} us, with {1e6 * with_filters:.0f} us")
    assert with_filters < 3 * without
