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
