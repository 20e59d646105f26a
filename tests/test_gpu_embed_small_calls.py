"""Lookup calls whose launch shape depends on their size: lookups per wave (1 ... 64), direct adds against
the routed gradient, chunks per route workgroup.  Forward exact, gradients (per lookup and pooled) at the
fp32 bar, both sides of every line."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import F32_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,D,Z", [
    (1, 128, 32), (65, 128, 32), (8191, 128, 32), (16385, 64, 32), (19_533, 128, 32),
    (300, 128, 16), (8193, 128, 16), (777, 96, 40), (40_000, 64, 16), (131_073, 128, 32), (262_200, 32, 16),
])
def test_small_calls_match_oracle(roast, N, D, Z):
    m_size = 50_021
    rng = np.random.default_rng(N + D + Z)
    h = wl.draw_hash(rng)
    lam = np.float32(0.8)
    rows = np.where(rng.random(N) < 0.3, rng.integers(0, 40, N), rng.integers(0, 1 << 33, N)).astype(np.int64)
    tables = rng.integers(0, 26, N).astype(np.uint32)
    M = rng.standard_normal(m_size).astype(np.float32)
    d = roast.embed_desc(D, Z, m_size, lam, h)
    rd, td = to_dev(rows), to_dev(tables)
    out = roast.roast_embed_fwd(d, rd, td, to_dev(M))
    assert np.array_equal(out.cpu().numpy(), oracle.embed_fwd(h, D, Z, float(lam), rows, tables, M).astype(np.float32))
    dOut = rng.standard_normal((N, D)).astype(np.float32)
    ref = oracle.embed_bwd(h, D, Z, m_size, float(lam), rows, tables, dOut)
    for mode in (roast.ROAST_REDUCE_ATOMIC, roast.ROAST_REDUCE_DETERMINISTIC):
        ws = torch.empty(max(roast.roast_embed_bwd_workspace(d, N, mode), 16), dtype=torch.uint8, device="cuda")
        dM = torch.zeros(m_size, device="cuda")
        roast.roast_embed_bwd(d, rd, td, to_dev(dOut), dM, mode, ws)
        assert rel_err(to_host_f64(dM), ref) <= F32_TOL, mode
    # pooled, bags of 0 .. 9 lookups
    cuts = np.unique(np.concatenate([[0, N], rng.integers(0, N + 1, N // 5)])).astype(np.int64)
    offsets = np.sort(np.concatenate([cuts, rng.choice(cuts, 3)]))
    offsets[0], offsets[-1] = 0, N
    B = len(offsets) - 1
    g = rng.standard_normal((B, D)).astype(np.float32)
    ws = torch.empty(max(roast.roast_embed_bag_bwd_workspace(d, N, B), 16), dtype=torch.uint8, device="cuda")
    dM = torch.zeros(m_size, device="cuda")
    roast.roast_embed_bag_bwd(d, rd, td, to_dev(offsets), to_dev(g), dM, ws=ws)
    ref = oracle.embed_bwd(h, D, Z, m_size, float(lam), rows, tables, np.repeat(g, np.diff(offsets), axis=0))
    assert rel_err(to_host_f64(dM), ref) <= F32_TOL
