"""Reproducible gradient of M: slots summed in windows of 64 and 256 by 4 and 16 waves.  Sizes of M at the edges of the windows and of the
choice between them, M of one tile (every tile at one place), ragged last tiles, tiles of odd sides, one sign per element."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import F32_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,O,Z1,Z2,m,sign", [
    (256, 384, 64, 64, 4096, True),            # all tiles at one place
    (256, 384, 64, 64, 4097, True),
    (256, 384, 64, 64, 64 * 65 + 1, True),     # 23 products to a slot: 4 waves
    (512, 1024, 32, 32, 5000, True),           # 105: 16 waves
    (200, 136, 32, 64, 2111, False),           # ragged in both
    (96, 90, 7, 5, 3000, True),                # 252 tiles of 35
    (96, 90, 7, 5, 3000, 2),
    (40, 24, 1, 1, 500, True),
    (256, 128, 128, 32, (256 << 10) - 1, True),
    (256, 128, 128, 32, 256 << 10, True),      # windows of 256
    (1000, 520, 32, 32, (256 << 10) + 255, True),
    (256, 256, 4, 4, 300, True),               # 4096 tiles at 285 places, and more than 4096 and 16384 (ranks of 1, 2, 4 tiles to a lane)
    (258, 260, 4, 4, 5000, True),
    (512, 516, 4, 4, 16, True),                # 16512 tiles at one place
    (520, 520, 4, 4, 90_000, True),
])
@pytest.mark.parametrize("I", [3, 700])
def test_gradient_is_the_oracles(roast, H, O, Z1, Z2, m, sign, I):
    rng = np.random.default_rng(H + m + I)
    h = wl.draw_hash(rng, use_sign=sign)
    lam = 0.37
    X, dY = (rng.standard_normal((I, n)).astype(np.float32) for n in (H, O))
    start = rng.standard_normal(m).astype(np.float32)
    d = roast.mm_desc(H, O, Z1, Z2, m, 3, lam, h)
    det = roast.ROAST_REDUCE_DETERMINISTIC
    runs = []
    for _ in range(2):
        ws = torch.randint(0, 256, (roast.roast_mm_bwd_dM_workspace(d, I, det),), dtype=torch.uint8, device="cuda")
        dM = to_dev(start.copy())
        roast.roast_mm_bwd_dM(d, to_dev(X), to_dev(dY), dM, det, ws)
        runs.append(dM)
    assert torch.equal(runs[0].view(torch.int32), runs[1].view(torch.int32))
    ref = oracle.mm_bwd_dm(h, 3, Z1, Z2, m, lam, X.astype(np.float64), dY.astype(np.float64))
    got = to_host_f64(runs[0])
    assert np.array_equal(got[ref == 0], start[ref == 0].astype(np.float64))
    # (the sum with what was there before is rounded too)
    assert rel_err(got - start, ref) <= F32_TOL + 2.0 ** -24 * np.abs(start).max() / np.sqrt(np.mean(ref ** 2))
