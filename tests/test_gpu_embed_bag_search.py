"""The bag of a lookup is found where bags of equal sizes have it, or by a bisection of what is left beside two places near that: bags of any sizes, few to
many, both gradient kernels (few chunks: direct adds; many: routed).  Whole numbers: exact."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def offsets_of(kind, B, N, rng):
    if kind == "equal":
        cut = np.arange(B) * N // B
    elif kind == "first empty":            # all lookups in the last bag
        cut = np.zeros(B, dtype=np.int64)
    elif kind == "last empty":             # all in the first
        cut = np.full(B, N); cut[0] = 0
    elif kind == "any":
        cut = np.sort(rng.integers(0, N + 1, B)); cut[0] = 0
    else:                                  # nearly all in one bag in the middle, single ones beside it
        cut = np.minimum(np.arange(B), N)
        cut[B // 2 + 1:] = np.maximum(N - np.arange(B - B // 2 - 1)[::-1], cut[B // 2])
        cut[0] = 0
    return np.concatenate([cut, [N]]).astype(np.int64)


@pytest.mark.parametrize("B", [1, 2, 3, 7, 8, 9, 63, 64, 65, 513, 4097])
@pytest.mark.parametrize("kind", ["equal", "first empty", "last empty", "any", "one long"])
@pytest.mark.parametrize("N,D,Z", [(1500, 32, 16), (33_000, 64, 32)])
def test_every_lookup_finds_its_bag(roast, B, kind, N, D, Z):
    rng = np.random.default_rng(B * 31 + N)
    m = 50_021
    offsets = offsets_of(kind, B, N, rng)
    assert offsets[0] == 0 and np.all(np.diff(offsets) >= 0)
    rows, tables = rng.integers(0, 1 << 33, N), np.zeros(N, dtype=np.uint32)
    dOut = rng.integers(-4, 5, (B, D)).astype(np.float32)
    h = wl.draw_hash(rng)
    d = roast.embed_desc(D, Z, m, 1.0, h)
    ws = torch.empty(max(roast.roast_embed_bag_bwd_workspace(d, N, B), 1), dtype=torch.uint8, device="cuda")
    dM = torch.zeros(m, device="cuda")
    roast.roast_embed_bag_bwd(d, to_dev(rows), to_dev(tables), to_dev(offsets), to_dev(dOut), dM, ws=ws)
    assert np.array_equal(to_host_f64(dM), oracle.embed_bag_bwd(h, D, Z, m, 1.0, rows, tables, offsets, dOut))


@pytest.mark.parametrize("B", [5, 64, 700, 4097])
@pytest.mark.parametrize("off", [-1, 0, 1, 2, 300])
@pytest.mark.parametrize("at_end", [False, True])
@pytest.mark.parametrize("N,D,Z", [(1500, 32, 16), (33_000, 64, 32)])
def test_bags_that_lie_beside_the_guess(roast, B, off, at_end, N, D, Z):
    """Empty bags before (or behind) bags of equal sizes: the guess is wrong by their number at one end of the lookups and right at the other; as many of them as
    there are places to the one asked for beside the guess, one fewer, one and more beyond it."""
    empty = max((B >> 6) + 4 + off, 1)
    full = np.arange(B + 1) * N // B
    offsets = (np.concatenate([full, np.full(empty, N)]) if at_end else np.concatenate([np.zeros(empty), full])).astype(np.int64)
    B = len(offsets) - 1
    rng = np.random.default_rng(B + N)
    m = 50_021
    rows, tables = rng.integers(0, 1 << 33, N), np.zeros(N, dtype=np.uint32)
    dOut = rng.integers(-4, 5, (B, D)).astype(np.float32)
    h = wl.draw_hash(rng)
    d = roast.embed_desc(D, Z, m, 1.0, h)
    ws = torch.empty(max(roast.roast_embed_bag_bwd_workspace(d, N, B), 1), dtype=torch.uint8, device="cuda")
    dM = torch.zeros(m, device="cuda")
    roast.roast_embed_bag_bwd(d, to_dev(rows), to_dev(tables), to_dev(offsets), to_dev(dOut), dM, ws=ws)
    assert np.array_equal(to_host_f64(dM), oracle.embed_bag_bwd(h, D, Z, m, 1.0, rows, tables, offsets, dOut))
