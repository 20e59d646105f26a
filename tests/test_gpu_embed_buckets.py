"""Bucketed lookup gradient (route by destination, accumulate in on-chip memory) over large arrays:
buckets grow with M beyond 1 Mi slots, and the workgroups of a bucket share out its slots.  Both
reduce modes against the oracle's explicit scatter-add (gradient equation of Section 4.3), repeated
ids included so that slots collect many addends."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import F32_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m_size,N,D,Z", [
    (10_000_019, 32_768, 128, 32),   # 512 buckets, parts of 4096 slots and fewer
    (16_777_216, 20_000, 128, 64),   # the largest array the bucket path takes; wider chunks
    (8_388_609, 70_001, 64, 16),     # ragged lookup count
    (3_000_000, 40_000, 128, 32),    # 256 buckets
])
def test_bucketed_gradient_matches_oracle_in_both_modes(roast, m_size, N, D, Z):
    rng = np.random.default_rng(m_size % 9973 + N)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    lam = np.float32(0.8)
    # a third of the lookups repeat a few hundred hot rows, so some slots collect hundreds of addends
    rows = rng.integers(0, 1 << 33, N).astype(np.int64)
    hot = rng.integers(0, 300, N).astype(np.int64)
    rows = np.where(rng.random(N) < 0.33, hot, rows)
    tables = rng.integers(0, 26, N).astype(np.uint32)
    dOut = rng.standard_normal((N, D)).astype(np.float32)
    d = roast.embed_desc(D, Z, m_size, lam, h)
    ref = oracle.embed_bwd(h, D, Z, m_size, float(lam), rows, tables, dOut)
    rd, td, gd = to_dev(rows), to_dev(tables), to_dev(dOut)
    for mode in (roast.ROAST_REDUCE_ATOMIC, roast.ROAST_REDUCE_DETERMINISTIC):
        nbytes = roast.roast_embed_bwd_workspace(d, N, mode)
        assert nbytes > 0
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        dM = torch.zeros(m_size, dtype=torch.float32, device="cuda")
        roast.roast_embed_bwd(d, rd, td, gd, dM, mode, ws)
        torch.cuda.synchronize()
        assert rel_err(to_host_f64(dM), ref) <= F32_TOL, mode
        if mode == roast.ROAST_REDUCE_DETERMINISTIC:
            again = torch.zeros(m_size, dtype=torch.float32, device="cuda")
            roast.roast_embed_bwd(d, rd, td, gd, again, mode, ws)
            assert torch.equal(dM, again)
