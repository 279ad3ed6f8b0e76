"""Node guides where a thread takes 1, 2, 4 and 8 buckets in a row: tables of 2^18 to 2^22
buckets, over nodes of which long runs carry no weight (also at both ends) and a few own
thousands of buckets.  Samples have the oracle's classes."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import ORACLE_SAMPLER
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


def _sparse(n):
    """Three hubs, a dense patch of consecutive nodes and 20,000 random edges between
    every 11th node of the middle; the first and the last 1,000 nodes have no edge."""
    rng = np.random.Generator(np.random.PCG64(n))
    mid = np.arange(1_000, n - 1_000)
    e = [np.stack([np.full(800, h), rng.choice(mid, 800, replace=False)], 1) for h in (1_000, n // 2, n - 1_001)]
    patch = n // 3 + np.arange(60)
    a, b = np.triu_indices(60, 1)
    e.append(np.stack([patch[a], patch[b]], 1))
    e.append(rng.choice(mid[::11], (20_000, 2)))
    e = np.sort(np.concatenate(e), 1)
    return gg.from_edges(n, np.unique(e[e[:, 0] < e[:, 1]], axis=0), "n%d" % n)


@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, (1 << 18) + 1, (1 << 19) + 1, (1 << 20) + 3])
def test_node_draws(n):
    g = _sparse(n)
    G, og = moss.Graph(g), oracle.Graph(g)
    k = 8_009
    for sampler in (moss.MOSS_SAMPLER_MOSS4, moss.MOSS_SAMPLER_MOSS4MIN, moss.MOSS_SAMPLER_T5,
                    moss.MOSS_SAMPLER_PATH5):
        cls = torch.full((k,), 255, dtype=torch.uint8, device="cuda")
        G.sample_range(sampler, 5, 0, k, cls)
        osid = ORACLE_SAMPLER[sampler]
        want = np.array([og.sample(osid, 5, i)[0] for i in range(k)], dtype=np.uint8)
        np.testing.assert_array_equal(cls.cpu().numpy(), want)
        assert len(np.unique(want)) > 1  # T-5 and Path-5 draw mostly around the hubs
