"""Creation by buckets, keys past a bucket's end: edges whose home slots are the last of one
bucket, inner or the last of all, go on into the first slots of the next one, which hold keys
of their own, and past the 64 that a bucket may list the set is built the general way.  Two
hubs share all ends of those edges, so that T-5 samples probe every one of them."""
import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
from paper_1509_08089_amd import moss

pytestmark = pytest.mark.gpu

BITS, BUCKET = 17, 8192  # slots of 40,000 edges, slots of a bucket
BUCKETS = (1 << BITS) // BUCKET
M, N, ENDS = 40_000, 200_000, 60_000


def _home(e):
    e = np.sort(e, 1).astype(np.uint64)
    return (((e[:, 0] << np.uint64(32)) | e[:, 1]) * np.uint64(0x9E3779B97F4A7C15)) >> np.uint64(64 - BITS)


def _past_the_end(home, bucket):
    """Keys that linear probing pushes out of a bucket (their number: the order is immaterial)."""
    at, out = 0, 0
    for h in np.sort(home[home // BUCKET == bucket].astype(np.int64) % BUCKET):
        at = max(at, int(h))
        out += at >= BUCKET
        at += 1
    return out


def _graph(bucket, spills):
    """Edges (their ends in [2, ENDS)) by home slot, hubs 0 and 1 over their ends, and as
    many single edges beside them as M takes."""
    rng = np.random.Generator(np.random.PCG64(17))
    pairs = rng.integers(2, ENDS, (6_000_000, 2))
    home = _home(pairs)
    last, first = (bucket + 1) * BUCKET - 6, (bucket + 1) % BUCKETS * BUCKET

    def with_home(slot):  # in the order drawn; pairs of one end or drawn twice are not in it
        e = np.sort(pairs[(home >= slot) & (home < slot + 6)], 1)
        e = e[np.sort(np.unique(e[:, 0] * N + e[:, 1], return_index=True)[1])]
        return e[e[:, 0] != e[:, 1]]

    tail, head = with_home(last), with_home(first)[:40]
    single = np.stack([ENDS + 2 * np.arange(M), ENDS + 1 + 2 * np.arange(M)], 1)
    lo, hi = spills, len(tail)  # more of the tail push out more keys
    while lo <= hi:
        k = (lo + hi) // 2
        special = np.concatenate([tail[:k], head])
        ends = np.unique(special)
        e = np.concatenate([special] + [np.stack([np.full(len(ends), h), ends], 1) for h in (0, 1)])
        e = np.concatenate([e, single[: M - len(e)]])
        got = _past_the_end(_home(e), bucket)
        if got == spills:
            break
        lo, hi = (k + 1, hi) if got < spills else (lo, k - 1)
    assert got == spills and len(e) == M
    return gg.from_edges(N, e, "spill"), special


@pytest.mark.parametrize("flags", [0, moss.MOSS_TRUST_CSR])
@pytest.mark.parametrize("spills", [7, 64, 65, 130])
@pytest.mark.parametrize("bucket", [5, BUCKETS - 1])
def test_spilled_keys_are_found(bucket, spills, flags):
    csr, special = _graph(bucket, spills)
    t = [torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda() for x in (csr.row_ptr, csr.col)]
    g, og = moss.Graph.from_device(*t, flags=flags), oracle.Graph(csr)
    n = 2_000_000
    np.testing.assert_array_equal(g.sample_range(moss.MOSS_SAMPLER_T5, 3, 0, n), og.run(oracle.T5, 3, 0, n, 8))
    # every one of those edges was probed: u~w, u~r or w~r of a sample
    _, u, w, r, last = g.sample_nodes(moss.MOSS_SAMPLER_T5, 3, np.arange(n))[0].astype(np.int64).T
    keep = (last != w) & (last != r)
    probed = np.concatenate([np.sort(np.stack([a[keep], b[keep]], 1), 1) for a, b in ((u, w), (u, r), (w, r))])
    assert np.isin(special[:, 0] * N + special[:, 1], probed[:, 0] * N + probed[:, 1]).all()
