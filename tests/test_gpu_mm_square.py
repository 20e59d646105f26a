"""Forward and dX in 128 x 128 blocks: ragged rows, columns and steps, both ways to apply the signs, parts of the contraction that
begin inside a tile; bit for bit the sums that a call without a copy of M gives."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import BF16_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FWD, DX = 0, 1
# product, rows, contraction, columns, Z1, Z2, |M|, parts
CASES = [
    (FWD, 1290, 320, 1344, 64, 64, 16384, 1),
    (FWD, 1290, 328, 1352, 32, 128, 16385, 1),         # eight indices in the last step, eight columns in the last block
    (DX, 1301, 328, 1096, 64, 32, 30011, 1),
    (DX, 3823, 896, 448, 128, 128, 65537, 1),
    (FWD, 2200, 832, 520, 128, 64, 4300001, 1),        # signs by XOR
    (DX, 2201, 840, 1032, 32, 32, 4300001, 1),
    (DX, 878, 4160, 640, 32, 64, 64571, 6),
    (FWD, 2537, 2624, 256, 64, 64, 65536, 6),
    (FWD, 2079, 2696, 264, 64, 32, 4300001, 5),
    (DX, 2065, 2696, 264, 32, 64, 4300001, 5),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("pad", [0, 8])
def test_square_blocks_match_oracle(roast, case, pad):
    which, I, K, N, Z1, Z2, m, parts = case
    H, O = (N, K) if which else (K, N)
    rng = np.random.default_rng(I + K + N)
    lam = np.float32(0.37)
    M, A, h = wl.draw_m(rng, m, ("normal", 0.05)), wl.draw_act(rng, I, K, "bf16"), wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.mm_desc(H, O, Z1, Z2, m, 2, lam, h)
    BF = torch.bfloat16
    need = (roast.roast_mm_bwd_dx_workspace if which else roast.roast_mm_fwd_workspace)(d, BF, I)
    assert roast.roast_mm_wide_blocks(d, BF, I, which, parts > 1) == (128, 128, 1, parts)
    Md = to_dev(M)
    Mb = roast.roast_m_shadow_bf16(Md)
    Ad = torch.full((I, K + pad), 9.0, dtype=BF, device="cuda")[:, :K]
    Ad.copy_(to_dev(A))
    rows = np.unique(np.concatenate([np.arange(0, I, 29), np.arange(I - 20, I)]))
    W = oracle.materialize_w(h, 2, H, O, Z1, Z2, float(lam), M)
    ref = (oracle.mm_bwd_dx if which else oracle.mm_fwd)(wl.act_as_f64(A)[rows], W)
    got = []
    for copy in (Mb, None):
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda") if parts > 1 else None
        out = torch.full((I, N + pad), 7.0, dtype=BF, device="cuda")
        (roast.roast_mm_bwd_dx if which else roast.roast_mm_fwd)(d, Ad, Md, out[:, :N], M_bf16=copy, ws=ws)
        assert torch.all(out[:, N:] == 7.0)
        got.append(out[:, :N])
    assert torch.equal(*got)
    assert rel_err(to_host_f64(got[0])[rows], ref) <= BF16_TOL


@pytest.mark.parametrize("which,I,K,N", [(FWD, 1290, 328, 1352), (DX, 1301, 328, 1096)])
def test_an_infinity_stays_in_its_row(roast, which, I, K, N):
    """A step beyond the end of the contraction loads the start of the row, rows beyond the last one repeat it."""
    H, O = (N, K) if which else (K, N)
    d = roast.mm_desc(H, O, 64, 64, 4097, 0, 1.0, wl.draw_hash(np.random.default_rng(K), use_sign=False, align=1))
    assert roast.roast_mm_wide_blocks(d, torch.bfloat16, I, which, False) == (128, 128, 1, 1)
    M = torch.rand(4097, device="cuda") + 0.5
    A = torch.randn((I, K), device="cuda").bfloat16()
    A[3, 5] = A[I - 1, K - 1] = float("inf")
    R = (roast.roast_mm_bwd_dx if which else roast.roast_mm_fwd)(d, A, M, M_bf16=roast.roast_m_shadow_bf16(M))
    assert torch.all(R[[3, I - 1]] == float("inf"))
    R[[3, I - 1]] = 0
    assert torch.all(torch.isfinite(R))
