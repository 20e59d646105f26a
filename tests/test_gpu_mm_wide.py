"""GPU parity of the wide matrix-core kernels (tiles that are multiples of 32; a bf16 shadow of M, or fp32 planes) where
their blocks, strips, splits and steps end: rows, columns and contraction lengths around the block edges,
one contraction step, ragged last steps, every tile extent, odd and even tile bases."""
import numpy as np
import pytest

import oracle
from paper_2207_10702_amd import workloads as wl
from tests.util import BF16_TOL, F32_TOL, rel_err, to_dev, to_host_f64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (I, H, O, Z1, Z2, |M|)
SHAPES = [
    (1, 8, 8, 32, 32, 1025),               # one row, one 16-byte piece
    (127, 64, 192, 32, 64, 5001),          # one step; a row and a column block just missed / just full
    (129, 72, 200, 64, 32, 9000),          # ragged step, one row and one column piece too many
    (257, 136, 264, 96, 96, 20011),
    (2057, 1096, 1160, 96, 96, 20011),     # tiles that are no power of two
    (255, 128, 128, 128, 128, 16384),      # |M| == one tile: every tile at base 0
    (300, 1096, 520, 32, 96, 30000),
    (300, 6152, 2056, 32, 96, 30000),      # contraction split (with a workspace), ragged last part
    (301, 2056, 6152, 96, 32, 30000),
    (8200, 520, 776, 64, 64, 47185),       # many rows: uneven dM parts
    (2100, 192, 6144, 64, 64, 33333),      # 256 x 256 blocks, ragged rows
    (2100, 6144, 192, 64, 64, 33333),
    (5000, 1024, 4096, 128, 64, 100003),   # 256 x 192 blocks
    (509, 1344, 5632, 128, 64, 100003),    # dM: 256 x 256 blocks
    (516, 1664, 4672, 128, 128, 100003),   # fp32 dM: 256 x 192
    (3747, 128, 4608, 128, 64, 100003),    # strips, ragged rows
    (3747, 4608, 128, 64, 128, 100003),
    (1585, 128, 14592, 64, 64, 100003),
    (6958, 128, 3456, 32, 64, 100003),
    (5855, 5760, 128, 64, 128, 100003),
    # |M| beyond 4 Mi: the shadow has no negated copies
    (129, 72, 200, 64, 32, 5000001),
    (300, 6152, 2056, 32, 96, 4300000),
    (2100, 192, 6144, 64, 64, 4300001),
    (5000, 1024, 4096, 128, 64, 4300001),
    (3747, 128, 4608, 128, 64, 4300001),
    (1585, 14592, 128, 64, 64, 4300001),
    (6958, 3456, 128, 64, 32, 4300001),
    (5855, 128, 5760, 128, 64, 4300001),
    (2047, 1000, 1024, 64, 32, 4300001),   # dX on the 256 x 96 blocks; ragged rows and columns
    (6144, 768, 640, 64, 64, 4300001),     # ... the most of them that it takes
]

FWD, DX, DM = 0, 1, 2
BF16, F32 = torch.bfloat16, torch.float32
# What some of them are there for: (I, H, O) -> (which product, type, workspace given, (rows, columns, strip, parts); None: the 128-column kernels and their
# narrower blocks).  The smallest shapes run on the kernels of small calls in the products that are not listed.
BLOCKS = {
    (1, 8, 8): [(FWD, BF16, False, (256, 128, 1, 1))],
    (127, 64, 192): [(FWD, BF16, False, (256, 128, 1, 1))],
    (129, 72, 200): [(FWD, BF16, False, (256, 128, 1, 1))],
    (2057, 1096, 1160): [(FWD, BF16, False, (128, 192, 1, 1)), (DX, BF16, False, (128, 192, 1, 1)), (FWD, F32, True, (128, 192, 1, 2)), (DX, F32, True, (256, 128, 1, 3))],
    (300, 6152, 2056): [(FWD, BF16, True, (128, 192, 1, 7)), (FWD, F32, True, (128, 192, 1, 7)), (DX, F32, True, (256, 256, 1, 5))],
    (301, 2056, 6152): [(DX, BF16, True, (128, 192, 1, 7)), (DX, F32, True, (128, 192, 1, 7))],
    (8200, 520, 776): [(DM, BF16, False, (128, 192, 1, 7))],
    (2100, 192, 6144): [(FWD, BF16, False, (256, 256, 1, 1)), (FWD, F32, True, (256, 256, 1, 1)), (DM, F32, True, (256, 128, 1, 5))],
    (2100, 6144, 192): [(DX, BF16, False, (256, 256, 1, 1)), (DX, F32, True, (256, 256, 1, 1)), (FWD, BF16, True, (128, 192, 1, 12))],
    (5000, 1024, 4096): [(FWD, BF16, False, (256, 192, 1, 1)), (DM, BF16, False, (256, 128, 1, 2))],
    (509, 1344, 5632): [(DM, BF16, False, (256, 256, 1, 1)), (DM, F32, True, (256, 256, 1, 1))],
    (516, 1664, 4672): [(DM, F32, True, (256, 192, 1, 1))],
    (3747, 128, 4608): [(FWD, BF16, False, (128, 192, 3, 1))],
    (3747, 4608, 128): [(DX, BF16, False, (128, 192, 3, 1))],
    (1585, 128, 14592): [(FWD, BF16, True, (128, 192, 4, 1))],
    (1585, 14592, 128): [(DX, BF16, True, (128, 192, 4, 1))],
    (6958, 128, 3456): [(FWD, BF16, False, (256, 192, 2, 1))],
    (6958, 3456, 128): [(DX, BF16, False, (256, 192, 2, 1)), (FWD, BF16, True, (256, 128, 1, 6))],
    (5855, 128, 5760): [(FWD, BF16, False, (256, 192, 3, 1))],
    (5855, 5760, 128): [(DX, BF16, False, (256, 192, 3, 1))],
    (2047, 1000, 1024): [(DX, BF16, False, None)],
    (6144, 768, 640): [(DX, BF16, False, None)],
}


def check_blocks(roast, shape, d):
    """The shape still runs on the blocks that it is listed for."""
    for which, dtype, workspace, blocks in BLOCKS.get(shape[:3], []):
        assert roast.roast_mm_wide_blocks(d, dtype, shape[0], which, workspace) == blocks, (shape, which, dtype)
        assert roast.roast_mm_direct_blocks(d, dtype, shape[0], which, workspace) is None if which != DM else True


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pad", [0, 8])
def test_wide_kernels_match_oracle(roast, shape, pad):
    I, H, O, Z1, Z2, m = shape
    rng = np.random.default_rng(I + 7 * H + O)
    M = wl.draw_m(rng, m, ("normal", 0.05))
    X = wl.draw_act(rng, I, H, "bf16")
    dY = wl.draw_act(rng, I, O, "bf16")
    h = wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.mm_desc(H, O, Z1, Z2, m, 2, np.float32(0.43), h)
    check_blocks(roast, shape, d)
    Md = to_dev(M)
    Mb = roast.roast_m_shadow_bf16(Md)

    def padded(x, n, fill):
        t = torch.full((I, n + pad), fill, dtype=torch.bfloat16, device="cuda")
        if x is not None:
            t[:, :n] = to_dev(x)
        return t[:, :n]

    Xd, dYd = padded(X, H, 9.0), padded(dY, O, 9.0)
    W = oracle.materialize_w(h, 2, H, O, Z1, Z2, float(np.float32(0.43)), M)
    Xo, dYo = wl.act_as_f64(X), wl.act_as_f64(dY)
    Yr, dXr = oracle.mm_fwd(Xo, W), oracle.mm_bwd_dx(dYo, W)
    need = max(roast.roast_mm_fwd_workspace(d, torch.bfloat16, I), roast.roast_mm_bwd_dx_workspace(d, torch.bfloat16, I), 16)
    for ws in (None, torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")):
        Y, dX = padded(None, O, 7.0), padded(None, H, 7.0)
        roast.roast_mm_fwd(d, Xd, Md, Y, M_bf16=Mb, ws=ws)
        roast.roast_mm_bwd_dx(d, dYd, Md, dX, M_bf16=Mb, ws=ws)
        torch.cuda.synchronize()
        if pad:                                             # nothing is written between the rows
            assert torch.all(Y._base[:, O:] == 7.0) and torch.all(dX._base[:, H:] == 7.0)
        assert rel_err(to_host_f64(Y), Yr) <= BF16_TOL
        assert rel_err(to_host_f64(dX), dXr) <= BF16_TOL
    dM = torch.zeros(m, device="cuda")
    roast.roast_mm_bwd_dM(d, Xd, dYd, dM)
    torch.cuda.synchronize()
    ref = oracle.mm_bwd_dm(h, 2, Z1, Z2, m, float(np.float32(0.43)), Xo, dYo)
    assert rel_err(to_host_f64(dM), ref) <= 1e-4


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[5] < 1 << 22])
def test_wide_plane_products_match_oracle(roast, shape):
    I, H, O, Z1, Z2, m = shape
    rng = np.random.default_rng(2 * I + 7 * H + O)
    M = wl.draw_m(rng, m, ("normal", 0.05))
    X = rng.standard_normal((I, H)).astype(np.float32)
    dY = rng.standard_normal((I, O)).astype(np.float32)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    lam = np.float32(0.43)
    d = roast.mm_desc(H, O, Z1, Z2, m, 2, lam, h)
    check_blocks(roast, shape, d)
    Md, Xd, dYd = to_dev(M), to_dev(X), to_dev(dY)
    ws = lambda n: torch.full((max(n, 16),), 0xFF, dtype=torch.uint8, device="cuda")  # noqa: E731
    Y, dX, dM = torch.empty((I, O), device="cuda"), torch.empty((I, H), device="cuda"), torch.zeros(m, device="cuda")
    roast.roast_mm_fwd(d, Xd, Md, Y, ws=ws(roast.roast_mm_fwd_workspace(d, torch.float32, I)))
    roast.roast_mm_bwd_dx(d, dYd, Md, dX, ws=ws(roast.roast_mm_bwd_dx_workspace(d, torch.float32, I)))
    roast.roast_mm_bwd_dM(d, Xd, dYd, dM, roast.ROAST_REDUCE_ATOMIC, ws(roast.roast_mm_bwd_dM_workspace_f32(d, I)))
    torch.cuda.synchronize()
    W = oracle.materialize_w(h, 2, H, O, Z1, Z2, float(lam), M)
    Xo, dYo = X.astype(np.float64), dY.astype(np.float64)
    assert rel_err(to_host_f64(Y), oracle.mm_fwd(Xo, W)) <= F32_TOL
    assert rel_err(to_host_f64(dX), oracle.mm_bwd_dx(dYo, W)) <= F32_TOL
    assert rel_err(to_host_f64(dM), oracle.mm_bwd_dm(h, 2, Z1, Z2, m, float(lam), Xo, dYo)) <= F32_TOL


@pytest.mark.parametrize("I", [9001, 8705, 32769])             # 18 parts; 18, the last of one token; 64, seven of them empty
def test_deterministic_gradient_of_many_parts(roast, I):
    """The reproducible gradient of M takes up to 64 parts of the tokens, whatever number the wide blocks would take."""
    H, O, Z1, Z2, m = 136, 264, 96, 96, 20011
    rng = np.random.default_rng(I)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    lam = np.float32(0.43)
    d = roast.mm_desc(H, O, Z1, Z2, m, 2, lam, h)
    X, dY = wl.draw_act(rng, I, H, "bf16"), wl.draw_act(rng, I, O, "bf16")
    Xd, dYd = to_dev(X), to_dev(dY)
    need = roast.roast_mm_bwd_dM_workspace(d, I, roast.ROAST_REDUCE_DETERMINISTIC)
    assert need >= 4 * H * O * min(-(-I // 512), 64)
    got = []
    for fill in (0xFF, 0x00):
        dM = torch.zeros(m, device="cuda")
        roast.roast_mm_bwd_dM(d, Xd, dYd, dM, roast.ROAST_REDUCE_DETERMINISTIC, torch.full((need,), fill, dtype=torch.uint8, device="cuda"))
        got.append(dM)
    assert torch.equal(got[0], got[1])
    ref = oracle.mm_bwd_dm(h, 2, Z1, Z2, m, float(lam), wl.act_as_f64(X), wl.act_as_f64(dY))
    assert rel_err(to_host_f64(got[0]), ref) <= F32_TOL


@pytest.mark.parametrize("shape", [(67, 128, 128), (1027, 768, 1536), (4099, 4096, 4096)])
def test_infinity_in_the_last_token_stays_an_infinity(roast, shape):
    """A ragged number of tokens: what fills the last step meets no infinity of the last token.  One tile
    for all (|M| = Z1 * Z2), no signs, dY > 0: the row of that infinity is +inf, the rest is finite."""
    I, H, O = shape
    h = wl.draw_hash(np.random.default_rng(I), use_sign=False, align=1)
    d = roast.mm_desc(H, O, 128, 128, 128 * 128, 0, 1.0, h)
    g = torch.Generator(device="cuda").manual_seed(I)
    X = torch.randn((I, H), generator=g, device="cuda", dtype=torch.bfloat16)
    dY = torch.rand((I, O), generator=g, device="cuda").add_(0.5).bfloat16()
    X[I - 1, 5] = float("inf")
    dM = torch.zeros(128 * 128, device="cuda")
    roast.roast_mm_bwd_dM(d, X, dY, dM)
    dM = dM.view(128, 128).cpu()
    assert torch.all(dM[5] == float("inf"))
    assert torch.all(torch.isfinite(dM[torch.arange(128) != 5]))


@pytest.mark.parametrize("I,H,O,Z1,Z2,wide", [
    (300, 72, 200, 32, 32, [(FWD, False, True)]), (300, 200, 72, 128, 32, [(DX, False, True)]),              # wide blocks with a copy of M
    (300, 6152, 2056, 64, 64, [(FWD, True, True)]), (300, 2056, 6152, 64, 64, [(DX, True, True)]),           # (a contraction of several parts, with a workspace)
    (3000, 1096, 1544, 8, 8, [(FWD, False, False), (DX, False, False)]),                                     # blocks of 128 columns, with and without a copy
    (300, 72, 200, 5, 3, [(FWD, False, False), (DX, False, False)])])                                        # element by element
def test_infinity_in_a_row_stays_an_infinity(roast, I, H, O, Z1, Z2, wide):
    """A ragged contraction: what fills the last step of forward / dX meets no infinity of the row.  No signs and
    M > 0: the row of that infinity is +inf, the others are finite.  wide: (product, workspace given, on wide blocks) of
    what a case is there for."""
    m = Z1 * Z2 + 1
    h = wl.draw_hash(np.random.default_rng(H), use_sign=False, align=1)
    d = roast.mm_desc(H, O, Z1, Z2, m, 0, 1.0, h)
    for which, workspace, on in wide:
        blocks = roast.roast_mm_wide_blocks(d, BF16, I, which, workspace)
        assert (blocks is not None) == on and (not workspace or blocks[3] > 1)
        assert roast.roast_mm_direct_blocks(d, BF16, I, which, workspace) is None
    g = torch.Generator(device="cuda").manual_seed(H)
    M = torch.rand(m, generator=g, device="cuda") + 0.5
    Mb = roast.roast_m_shadow_bf16(M)
    for n, call, want in ((H, roast.roast_mm_fwd, roast.roast_mm_fwd_workspace), (O, roast.roast_mm_bwd_dx, roast.roast_mm_bwd_dx_workspace)):
        A = torch.randn((I, n), generator=g, device="cuda").bfloat16()
        A[3, 5] = float("inf")                                                      # in the row's first piece
        A[I - 1, n - 1] = float("inf")                                              # in its last
        for copy in (None, Mb):
            for ws in (None, torch.empty(max(want(d, torch.bfloat16, I), 16), dtype=torch.uint8, device="cuda")):
                R = call(d, A, M, M_bf16=copy, ws=ws).cpu()
                assert torch.all(R[[3, I - 1]] == float("inf"))
                assert torch.all(torch.isfinite(R[[r for r in range(I) if r not in (3, I - 1)]]))
