"""The sorted kernel's windows are put in lane order by bits that travel with the sorted
entries: every sample of a window must be drawn once, with the outcome the plain launch
gives it, at windows and blocks of any size and at the edges of windows and spans."""
import numpy as np
import pytest
import torch

import graphgen as gg
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    return moss.Graph(gg.chung_lu(20000, 150000, 2.1, 2000, 34))


@pytest.mark.parametrize("window,threads", [(64, 64), (64, 256), (192, 128), (448, 192), (512, 64), (0, 0)])
@pytest.mark.parametrize("count", [1, 63, 513, 8192, 8193, 200_003])
def test_windows_draw_every_sample_once(graph, window, threads, count):
    out = []
    try:
        for sch in (moss.MOSS_SCHEDULE_PLAIN, moss.MOSS_SCHEDULE_XCD):
            moss.moss_set_tuning(threads_per_block=threads, schedule=sch, sort_window=window)
            cls = torch.full((count,), 255, dtype=torch.uint8, device="cuda")
            hits = graph.sample_range(moss.MOSS_SAMPLER_PATH5, 6, 1 << 33, (1 << 33) + count, cls)
            out.append((hits, cls.cpu().numpy()))
    finally:
        moss.moss_set_tuning()
    (ha, ca), (hb, cb) = out
    np.testing.assert_array_equal(ca, cb)
    np.testing.assert_array_equal(ha, hb)
    np.testing.assert_array_equal(ha, np.bincount(ca, minlength=22))


@pytest.mark.parametrize("k,flags", [(4, moss.MOSS_K4_MIN), (5, 0)])
@pytest.mark.parametrize("n", [2, 3, 16_385, 300 * 16_384 + 1])
def test_two_samplers_grouped_together(graph, k, flags, n):
    """An estimate's two samplers share the grouping launches; the first may have a block (and
    with 300 blocks a row more to a row-lane of the scan) more than the second."""
    try:
        moss.moss_set_tuning(schedule=moss.MOSS_SCHEDULE_PLAIN)
        a = graph.estimate(k, n, 12, flags)
        moss.moss_set_tuning(schedule=moss.MOSS_SCHEDULE_XCD)
        b = graph.estimate(k, n, 12, flags)
    finally:
        moss.moss_set_tuning()
    np.testing.assert_array_equal(a.hits_np, b.hits_np)
    assert b.hits_np[:, :7 if k == 4 else 22].sum() == n
