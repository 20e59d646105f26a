"""Forward and dX of mid-sized bf16 calls on 64 x 64 blocks whose operands go through LDS, in one launch and in parts of the contraction with a
workspace: rows around the block edge, shares of the contraction that begin and end inside a pair of units (or have none), tile sides
below, at and above the block's, odd and even bases, an M whose copy is not negated, strided rows; the same bits without a copy of M."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import BF16_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FWD, DX = 0, 1
# (which product, rows, contraction, columns, Z1, Z2, |M|, parts)
CASES = [
    (FWD, 512, 2048, 2048, 64, 64, 1 << 20, 1),
    (FWD, 513, 1088, 1024, 32, 128, 65537, 1),         # a row too many; 34 units for eight waves: shares of four and five
    (FWD, 1871, 1856, 320, 32, 32, 289873, 1),
    (FWD, 700, 1152, 1024, 96, 96, 30011, 1),          # tiles that are no power of two: a unit in each third
    (FWD, 524, 1984, 1536, 64, 64, 4300001, 1),        # signs by XOR
    (DX, 1, 4416, 640, 64, 32, 19073, 9),
    (DX, 220, 1024, 3904, 64, 64, 133183, 1),
    (DX, 600, 1344, 1536, 96, 96, 4300001, 1),
    (FWD, 17, 4288, 576, 32, 32, 13533, 8),            # parts of eight and nine pairs
    (FWD, 45, 3200, 1344, 96, 96, 4300001, 5),         # parts that begin inside a tile; signs by XOR
    (FWD, 97, 11072, 384, 128, 128, 117271, 12),
    (FWD, 363, 10240, 256, 128, 32, 65537, 8),
    (DX, 18, 4416, 640, 64, 64, 19073, 8),
    (DX, 42, 14208, 384, 128, 128, 4300001, 15),
    (DX, 62, 6656, 1920, 128, 64, 131629, 8),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("pad", [0, 8])
def test_blocks_through_lds_match_oracle(roast, case, pad):
    which, I, K, N, Z1, Z2, m, parts = case
    H, O = (N, K) if which else (K, N)
    rng = np.random.default_rng(I + K + N)
    lam = np.float32(0.37)
    M, A, h = wl.draw_m(rng, m, ("normal", 0.05)), wl.draw_act(rng, I, K, "bf16"), wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.mm_desc(H, O, Z1, Z2, m, 2, lam, h)
    BF = torch.bfloat16
    need = (roast.roast_mm_bwd_dx_workspace if which else roast.roast_mm_fwd_workspace)(d, BF, I)
    blocks = roast.roast_mm_direct_blocks(d, BF, I, which, True)
    assert blocks == (64, 64, 1, parts) and need >= (4 * parts * I * N if parts > 1 else 0)
    Md = to_dev(M)
    Mb = roast.roast_m_shadow_bf16(Md)
    Ad = torch.full((I, K + pad), 9.0, dtype=BF, device="cuda")[:, :K]
    Ad.copy_(to_dev(A))
    W = oracle.materialize_w(h, 2, H, O, Z1, Z2, float(lam), M)
    ref = (oracle.mm_bwd_dx if which else oracle.mm_fwd)(wl.act_as_f64(A), W)
    call = roast.roast_mm_bwd_dx if which else roast.roast_mm_fwd
    for room in (need, 0):
        got = []
        for copy in (Mb, None):
            ws = torch.full((room,), 0xFF, dtype=torch.uint8, device="cuda") if room else None
            out = torch.full((I, N + pad), 7.0, dtype=BF, device="cuda")
            call(d, Ad, Md, out[:, :N], M_bf16=copy, ws=ws)
            assert torch.all(out[:, N:] == 7.0)
            got.append(out[:, :N])
        assert torch.equal(*got)               # the copy holds the roundings that are made without it
        assert rel_err(to_host_f64(got[0]), ref) <= BF16_TOL


@pytest.mark.parametrize("which,I,K,N", [(FWD, 67, 4288, 576), (DX, 67, 4416, 640), (FWD, 513, 1088, 1024), (DX, 220, 1024, 3904)])
def test_an_infinity_stays_in_its_row(roast, which, I, K, N):
    """Rows beyond the last one repeat it, pairs of units are loaded by two waves: neither puts a row's infinity anywhere else."""
    h = wl.draw_hash(np.random.default_rng(K), use_sign=False, align=1)
    H, O = (N, K) if which else (K, N)
    m = 64 * 64 + 1
    d = roast.mm_desc(H, O, 64, 64, m, 0, 1.0, h)
    M = torch.rand(m, device="cuda") + 0.5
    A = torch.randn((I, K), device="cuda").bfloat16()
    A[3, 5] = A[I - 1, K - 1] = float("inf")
    need = (roast.roast_mm_bwd_dx_workspace if which else roast.roast_mm_fwd_workspace)(d, torch.bfloat16, I)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    R = (roast.roast_mm_bwd_dx if which else roast.roast_mm_fwd)(d, A, M, M_bf16=roast.roast_m_shadow_bf16(M), ws=ws)
    assert torch.all(R[[3, I - 1]] == float("inf"))
    R[[3, I - 1]] = 0
    assert torch.all(torch.isfinite(R))


@pytest.mark.parametrize("case", [
    (FWD, 524, 1984, 1408, 64, 64, 1 << 20, 1),        # without a copy: rows of blocks one after the other
    (FWD, 524, 1984, 1408, 64, 64, (1 << 20) + 1, 1),  # by eighths: 198 blocks, the last eighth two short
    (FWD, 65, 4288, 576, 32, 32, (1 << 20) + 1, 7),    # 126
    (FWD, 130, 3200, 704, 96, 96, (1 << 20) + 1, 5),   # 165
    (DX, 129, 6656, 448, 64, 64, (1 << 20) + 1, 9),
])
def test_blocks_by_eighths(roast, case):
    """A call without a copy of an M beyond the L2 deals its blocks to the XCDs as one with a copy does."""
    test_blocks_through_lds_match_oracle(roast, case, 0)
