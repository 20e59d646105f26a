"""Gradient of M of few bf16 tokens by windows of slots: numbers of tokens around a step, rows and columns that end inside a unit or a tile, every
tile width, an M of one window, of whole ones and of a piece more, tiles over two windows, one tile for each of many workgroups and
lists of tiles that fill up; dM at any multiple of four bytes, and added to.  Whole numbers: exact in any order."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (tokens, H, O, Z1, Z2, |M|)
SHAPES = [
    (1, 1024, 2048, 64, 64, 8192),         # one window
    (16, 1088, 2048, 64, 64, 8193),        # a second one of one slot
    (31, 2048, 2048, 32, 32, 4096),        # a small one
    (33, 1032, 2056, 64, 64, 30011),       # ragged units
    (64, 1000, 2504, 96, 96, 20011),       # tiles that are no power of two, ragged
    (61, 1640, 3208, 128, 128, 65537),
    (40, 2048, 1536, 32, 64, 16385),
    (100, 2048, 1536, 64, 32, 16385),
    (60, 2432, 2816, 64, 128, 40000),
    (384, 640, 6784, 32, 32, 12050),
    (20, 8192, 4096, 32, 32, 150001),      # 32768 tiles: several searches to a workgroup
    (40, 1152, 4096, 32, 128, 12345),
    (17, 4096, 4096, 64, 64, 2200000),     # more windows than CUs
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("at", [0, 3])
def test_windows_match_oracle(roast, shape, at):
    I, H, O, Z1, Z2, m = shape
    rng = np.random.default_rng(I + H + O)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.mm_desc(H, O, Z1, Z2, m, 1, np.float32(0.5), h)
    assert roast.roast_mm_wide_blocks(d, torch.bfloat16, I, 2) is None
    X, dY = (rng.integers(-2, 3, (I, n)).astype(np.float32) for n in (H, O))
    Xd, dYd = (torch.full((I, n + 8), 9.0, dtype=torch.bfloat16, device="cuda")[:, :n].copy_(to_dev(t)) for n, t in ((H, X), (O, dY)))
    flat = torch.ones(m + at + 1, device="cuda")
    roast.roast_mm_bwd_dM(d, Xd, dYd, flat[at:at + m])
    ref = oracle.mm_bwd_dm(h, 1, Z1, Z2, m, 0.5, X.astype(np.float64), dY.astype(np.float64))
    assert np.abs(ref).max() < 2 ** 23     # sums of halves stay exact
    assert np.array_equal(to_host_f64(flat[at:at + m]), ref + 1.0)
    assert torch.all(flat[:at] == 1.0) and flat[-1] == 1.0


def test_an_infinity_in_the_last_token_stays_an_infinity(roast):
    """What fills the last step repeats the last token: its infinity meets no zero.  One tile for all, no signs, dY > 0."""
    I, H, O = 35, 1024, 2048
    h = wl.draw_hash(np.random.default_rng(I), use_sign=False, align=1)
    d = roast.mm_desc(H, O, 64, 64, 64 * 64, 0, 1.0, h)
    assert roast.roast_mm_wide_blocks(d, torch.bfloat16, I, 2) is None
    X = torch.randn((I, H), device="cuda").bfloat16()
    X[I - 1, 5] = float("inf")
    dM = torch.zeros(64 * 64, device="cuda")
    roast.roast_mm_bwd_dM(d, X, torch.rand((I, O), device="cuda").add_(0.5).bfloat16(), dM)
    dM = dM.view(64, 64)
    assert torch.all(dM[5] == float("inf"))
    assert torch.all(torch.isfinite(dM[torch.arange(64) != 5]))
