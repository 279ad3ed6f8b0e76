"""Creation by buckets (graphs of at least 2^15 edges): every defect is reported as by the
general way, a set whose keys crowd into one bucket is built the general way, and probes
against either set give the oracle's classes."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from gpu_util import ORACLE_SAMPLER
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


def _edges(n, m, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    e = rng.integers(0, n, (int(1.3 * m), 2))
    e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], 1), axis=0)
    return e[np.sort(rng.permutation(len(e))[:m])]


@pytest.fixture(scope="module")
def graph():
    return gg.from_edges(30_000, _edges(30_000, (1 << 18) + 77, 5), "gnm")


def _create(rp, col, flags=0):
    t = [torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda() for x in (rp, col)]
    return moss.Graph.from_device(*t, flags=flags)


def test_sound_graph(graph):
    g = _create(graph.row_ptr, graph.col)
    og = oracle.Graph(graph)
    for s in (moss.MOSS_SAMPLER_MOSS4, moss.MOSS_SAMPLER_PATH5):
        np.testing.assert_array_equal(g.sample_range(s, 3, 0, 50_000), og.run(ORACLE_SAMPLER[s], 3, 0, 50_000, 8))


@pytest.mark.parametrize("at", [0, 255, 256, 16_383, 16_384, 300_001, -1])
def test_defects(graph, at):
    """One entry spoiled, at the edges of spans and of blocks' shares and at either end."""
    rp, col = graph.row_ptr.astype(np.int64), graph.col
    e = at % len(col)
    v = int(np.searchsorted(rp, e, side="right")) - 1
    lo, hi = rp[v], rp[v + 1]

    def status(new, flags=0):
        c = col.copy()
        c[e] = new
        with pytest.raises(moss.MossError) as x:
            _create(rp, c, flags)
        return x.value.status

    assert status(graph.n) == moss.MOSS_E_ARG and status(-1) == moss.MOSS_E_ARG
    assert status(graph.n, moss.MOSS_TRUST_CSR) == moss.MOSS_E_ARG
    if e > lo:
        assert status(col[e - 1]) == moss.MOSS_E_DUPLICATE
    # another neighbour in its place, in order: the old one's mirror and the new one's are missing
    below, above = (col[e - 1] if e > lo else -1), (col[e + 1] if e + 1 < hi else graph.n)
    free = [x for x in range(below + 1, above) if x not in (v, col[e])]
    assert free and status(free[0]) == moss.MOSS_E_ASYMMETRIC and status(free[-1]) == moss.MOSS_E_ASYMMETRIC


def test_dropped_mirror(graph):
    rp, col = graph.row_ptr.astype(np.int64), graph.col
    e = len(col) // 2
    v = int(np.searchsorted(rp, e, side="right")) - 1
    rp2 = rp.copy()
    rp2[v + 1:] -= 1
    with pytest.raises(moss.MossError) as x:
        _create(rp2, np.delete(col, e))
    assert x.value.status == moss.MOSS_E_ASYMMETRIC


def test_keys_in_one_bucket():
    """5,000 edges of one bucket of 8,192 slots (an upper and a lower key each)."""
    n, m = 30_000, (1 << 18) + 5
    e = _edges(n, 900_000, 9)
    key = (e[:, 0].astype(np.uint64) << np.uint64(32)) | e[:, 1].astype(np.uint64)
    bucket = (key * np.uint64(0x9E3779B97F4A7C15)) >> np.uint64(64 - 7)  # 2^20 slots: 128 buckets
    one = np.flatnonzero(bucket == 77)[:5_000]
    assert len(one) == 5_000
    rest = np.flatnonzero(bucket != 77)[: m - 5_000]
    csr = gg.from_edges(n, e[np.sort(np.concatenate([one, rest]))], "crowded")
    g, og = _create(csr.row_ptr, csr.col), oracle.Graph(csr)
    s = moss.MOSS_SAMPLER_T5
    np.testing.assert_array_equal(g.sample_range(s, 4, 0, 50_000), og.run(ORACLE_SAMPLER[s], 4, 0, 50_000, 8))
    c = csr.col.copy()
    c[0] = (set(range(1, int(c[1]))) - {int(c[0])}).pop()
    with pytest.raises(moss.MossError) as x:
        _create(csr.row_ptr, c)
    assert x.value.status == moss.MOSS_E_ASYMMETRIC


@pytest.mark.parametrize("m", [(1 << 15) - 1, 1 << 15, (1 << 15) + 1, 50_003])
def test_around_the_smallest(m):
    """From 2^15 edges on the set is built by buckets (16 of them there)."""
    csr = gg.from_edges(9_000, _edges(9_000, m, m), "gnm")
    g, og = _create(csr.row_ptr, csr.col), oracle.Graph(csr)
    for s in (moss.MOSS_SAMPLER_MOSS4, moss.MOSS_SAMPLER_T5):
        np.testing.assert_array_equal(g.sample_range(s, 3, 0, 20_000), og.run(ORACLE_SAMPLER[s], 3, 0, 20_000, 8))
    c = csr.col.copy()
    c[0] = (set(range(1, int(c[1]))) - {int(c[0])}).pop()
    with pytest.raises(moss.MossError) as x:
        _create(csr.row_ptr, c)
    assert x.value.status == moss.MOSS_E_ASYMMETRIC
