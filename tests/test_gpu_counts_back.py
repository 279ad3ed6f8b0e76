"""A launch's blocks add into rows of partial counts and its last block hands the sums to the
host and clears the rows: the counts must be whole for any number of blocks (around the
number of rows), for one sampler and for two side by side, call after call."""
import time

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graphs():
    g = gg.chung_lu(2000, 10000, 2.5, 200, 1)
    return moss.Graph(g), oracle.Graph(g)


@pytest.mark.parametrize("n", [2, 256 * 31, 256 * 32, 256 * 33 + 1, 256 * 64, 256 * 3000 + 7])
@pytest.mark.parametrize("k,flags", [(4, 0), (4, moss.MOSS_K4_MIN), (5, 0)])
def test_counts_are_whole(graphs, n, k, flags):
    G, og = graphs
    want = og.estimate4min(n, 3, threads=8) if flags else og.estimate(k, n, 3, threads=8)
    for _ in range(3):
        t = time.perf_counter()
        r = G.estimate(k, n, 3, flags)
        wall_ms = 1e3 * (time.perf_counter() - t)
        np.testing.assert_array_equal(r.hits_np, want.hits)
        assert 0.0 < r.device_ms < wall_ms


def test_calls_of_both_schedules_in_turn(graphs):
    """Both schedules leave the rows clear for the other."""
    G, og = graphs
    want = og.estimate(5, 40_000, 5, threads=8).hits
    try:
        for sch in (moss.MOSS_SCHEDULE_XCD, moss.MOSS_SCHEDULE_PLAIN) * 2:
            moss.moss_set_tuning(schedule=sch)
            np.testing.assert_array_equal(G.estimate(5, 40_000, 5).hits_np, want)
    finally:
        moss.moss_set_tuning()


def test_a_sampler_that_draws_nothing():
    """A star has no 4-paths: Path-5 draws nothing and its counts stay 0 beside T-5's."""
    g = gg.star(8)
    G, og = moss.Graph(g), oracle.Graph(g)
    for k in (4, 5):
        np.testing.assert_array_equal(G.estimate(k, 10_001, 2).hits_np, og.estimate(k, 10_001, 2, threads=2).hits)


@pytest.mark.parametrize("requests,budget", [(1, 1), (1, 5_000_000), (3, 257), (65, 300), (700, 600)])
def test_batch_items_and_tiles(graphs, requests, budget):
    """One item to more than a thousand, fewer tiles than blocks and more, batch after batch
    with fewer slots than the one before: each request as alone."""
    G, og = graphs
    for count in (requests, max(1, requests // 2)):
        reqs = [(G.h, 4 + i % 2, budget + i + 1, 40 + i, 0) for i in range(count)]
        out = moss.moss_estimate_batch(reqs)
        for i in sorted({0, count // 3, count - 1}):
            _, k, n, seed, _ = reqs[i]
            np.testing.assert_array_equal(out[i].hits_np, G.estimate(k, n, seed).hits_np)
            assert out[i].hits_np.sum() == n and out[i].device_ms > 0
