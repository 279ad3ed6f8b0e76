"""Hub filters: on graphs of more than 2^19 edges, rows of at least 256 entries answer their
probes from a filter of their own.  Samples on a graph with rows just below, at and above
that size, and one that takes several passes to build, have the oracle's classes."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import ORACLE_SAMPLER
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    """One hub of 40,000 entries, rows of 255, 256 and 257 entries beside it, a dense
    core whose rows link to all of them, and a sparse rest: 2^19 + 2^13 edges."""
    rng = np.random.Generator(np.random.PCG64(8))
    n, m = 60_000, (1 << 19) + (1 << 13)
    e = [np.stack([np.zeros(40_000, np.int64), 1 + np.arange(40_000)], 1)]
    for v, d in ((50_001, 254), (50_002, 255), (50_003, 256)):  # + the link to node 50_000
        e.append(np.stack([np.full(d, v), 1 + rng.choice(40_000, d, replace=False)], 1))
        e.append(np.array([[v, 50_000]]))
    core = 41_000 + np.arange(700)
    a, b = np.triu_indices(700, 1)
    e.append(np.stack([core[a], core[b]], 1)[rng.random(len(a)) < 0.8])
    e = np.concatenate(e)
    low = 1 + rng.integers(0, 45_000, (2 * m, 2))
    low = low[low[:, 0] < low[:, 1]]
    every = np.unique(np.sort(np.concatenate([e, low]), 1), axis=0)
    keep = np.isin(every[:, 0] * n + every[:, 1], np.sort(e, 1)[:, 0] * n + np.sort(e, 1)[:, 1])
    rest = rng.permutation(np.flatnonzero(~keep))[: m - int(keep.sum())]
    g = gg.from_edges(n, every[np.sort(np.concatenate([np.flatnonzero(keep), rest]))], "hubs")
    d = np.diff(g.row_ptr)
    assert g.nnz // 2 > 1 << 19 and list(d[50_001:50_004]) == [255, 256, 257] and d[0] == 40_000
    return g


@pytest.mark.parametrize("sampler", [moss.MOSS_SAMPLER_MOSS4, moss.MOSS_SAMPLER_MOSS4MIN, moss.MOSS_SAMPLER_T5,
                                     moss.MOSS_SAMPLER_PATH5])
def test_hub_rows_classes(graph, sampler):
    G, og = moss.Graph(graph), oracle.Graph(graph)
    n = 30_011
    cls = torch.full((n,), 255, dtype=torch.uint8, device="cuda")
    hits = G.sample_range(sampler, 3, 0, n, cls)
    osid = ORACLE_SAMPLER[sampler]
    want = np.array([og.sample(osid, 3, k)[0] for k in range(n)], dtype=np.uint8)
    np.testing.assert_array_equal(cls.cpu().numpy(), want)
    np.testing.assert_array_equal(hits, og.run(osid, 3, 0, n, 8))
    assert len(np.unique(want)) > 3
