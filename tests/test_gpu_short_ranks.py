"""Ranks of rows of one span's length and less, where many neighbours have the same degree:
circulant rows of 2 to 258 entries (all degrees equal) and the same with chords that spread
the degrees, with and without the creation's checks, equal the oracle's."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, moss.MOSS_TRUST_CSR])
@pytest.mark.parametrize("half,chords", [(1, 0), (1, 700), (15, 0), (16, 0), (16, 300), (17, 0), (32, 900), (33, 0),
                                         (64, 50), (127, 0), (128, 0), (129, 0)])
def test_circulant_rows(half, chords, flags):
    n = 1_003
    rng = np.random.Generator(np.random.PCG64(half))
    at = np.arange(n)
    e = [np.stack([at, (at + k) % n], 1) for k in range(1, half + 1)] + [rng.integers(0, n, (chords, 2))]
    e = np.sort(np.concatenate(e), 1)
    g = gg.from_edges(n, np.unique(e[e[:, 0] != e[:, 1]], axis=0), "circulant")
    G, og = moss.Graph(g, flags=flags), oracle.Graph(g)
    G.build_tables(moss.MOSS_TABLES_K4MIN)
    rank = G.table(moss.MOSS_TAB_RANK)
    np.testing.assert_array_equal(rank[:, 0], og.table(oracle.TAB_RANK))
    np.testing.assert_array_equal(rank[:, 1], og.table(oracle.TAB_RANK_MIRROR))
    np.testing.assert_array_equal(G.table(moss.MOSS_TAB_COL_RANK), og.table(oracle.TAB_COL_RANK))
    np.testing.assert_array_equal(G.table(moss.MOSS_TAB_ACC_CHECK), og.table(oracle.TAB_ACC_CHECK))
