"""The routed lookup gradient where its lists overflow and its slots are shared out: entries beyond a full list, chunks
that reach into the next bucket (which a fixed-point call lists twice), parts of a bucket, chunk lengths of every lane
layout.  Whole numbers, so that every order of the sums gives the oracle's bits."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def check(roast, h, D, Z, m_size, rows, rng, offsets=None):
    N = len(rows)
    tables = np.zeros(N, dtype=np.uint32)
    d = roast.embed_desc(D, Z, m_size, 1.0, h)
    dOut = rng.integers(-3, 4, (N, D)).astype(np.float32)
    ref = oracle.embed_bwd(h, D, Z, m_size, 1.0, rows, tables, dOut)
    dev = to_dev(rows), to_dev(tables), to_dev(dOut)
    for mode in (roast.ROAST_REDUCE_ATOMIC, roast.ROAST_REDUCE_DETERMINISTIC):
        ws = torch.empty(roast.roast_embed_bwd_workspace(d, N, mode), dtype=torch.uint8, device="cuda").fill_(0xa5)
        dM = torch.ones(m_size, device="cuda")
        roast.roast_embed_bwd(d, *dev, dM, mode, ws)
        assert np.array_equal(to_host_f64(dM), ref + 1.0), mode


def rows_at(h, m_size, Z, want, count=1 << 17):
    """The first row of table 0 whose chunk starts at an offset that `want` takes."""
    off = (h["a1"] * np.arange(count, dtype=object) + h["a3"]) % h["P"] % (m_size - Z + 1)
    return int(np.nonzero(want(off.astype(np.int64)))[0][0])


@pytest.mark.parametrize("m_size,N,hot", [
    (1_000_000, 70_000, (0.8, 0.0)),     # 56 000 entries for a list of some 8500: the rest is spilled
    (1_000_000, 70_000, (0.45, 0.45)),   # two neighbouring lists overflow, one by chunks that belong to both
    (1_280_000, 70_000, (0.1, 0.8)),     # the next list alone: what reaches into it is spilled for it alone
    (50_021, 200_000, (0.9, 0.0)),       # more than can be spilled
])
def test_lists_that_overflow(roast, m_size, N, hot):
    Z = 32
    rng = np.random.default_rng(N)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    R = 5120 if m_size == 1_280_000 else 4096
    across = rows_at(h, m_size, Z, lambda o: (o % R > R - Z) & (o > 2 * R))
    b = int((h["a1"] * across + h["a3"]) % h["P"] % (m_size - Z + 1)) // R
    inside = rows_at(h, m_size, Z, lambda o: (o // R == b + 1) & (o % R < R - Z))
    u = rng.random(N)
    rows = np.where(u < hot[0], across, np.where(u < sum(hot), inside, rng.integers(0, 1 << 33, N))).astype(np.int64)
    check(roast, h, Z, Z, m_size, rows, rng)


@pytest.mark.parametrize("m_size,N,D,Z", [
    (300_007, 70_000, 4, 4), (300_007, 40_000, 24, 12), (300_007, 33_000, 32, 16), (300_007, 70_000, 64, 64), (300_007, 33_000, 192, 96),
    (40_000, 66_000, 300, 300), (100_003, 33_000, 2048, 1024),
    (4_097, 70_000, 32, 32),             # one bucket and a slot
    (1_048_577, 70_000, 32, 32),         # buckets of more than 4096 slots begin
    (16_777_216, 70_000, 32, 32),        # the longest, sixteen parts
])
def test_lane_layouts_and_parts(roast, m_size, N, D, Z):
    rng = np.random.default_rng(m_size + Z)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    rows = np.where(rng.random(N) < 0.3, rng.integers(0, 50, N), rng.integers(0, 1 << 33, N)).astype(np.int64)
    check(roast, h, D, Z, m_size, rows, rng)


@pytest.mark.parametrize("B", [70_000, 280_000, 280_001])
def test_more_bags_than_lookups(roast, B):
    """The largest magnitude of dOut, that of an empty bag here, is found by a launch of its own where most bags are empty."""
    N, Z, m_size = 70_000, 32, 300_007
    rng = np.random.default_rng(B)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    rows, tables = rng.integers(0, 1 << 33, N), np.zeros(N, dtype=np.uint32)
    offsets = np.concatenate([[0, 0], np.sort(rng.integers(0, N + 1, B - 2)), [N]]).astype(np.int64)
    dOut = rng.integers(-3, 4, (B, Z)).astype(np.float32)
    dOut[0] = 1000.0
    d = roast.embed_desc(Z, Z, m_size, 1.0, h)
    ref = oracle.embed_bag_bwd(h, Z, Z, m_size, 1.0, rows, tables, offsets, dOut)
    ws = torch.empty(roast.roast_embed_bag_bwd_workspace(d, N, B, roast.ROAST_REDUCE_DETERMINISTIC), dtype=torch.uint8, device="cuda").fill_(0xa5)
    dM = torch.ones(m_size, device="cuda")
    roast.roast_embed_bag_bwd(d, to_dev(rows), to_dev(tables), to_dev(offsets), to_dev(dOut), dM, roast.ROAST_REDUCE_DETERMINISTIC, ws)
    assert np.array_equal(to_host_f64(dM), ref + 1.0)
