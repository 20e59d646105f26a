"""Which kernels a call is planned for, where a rule of a plan says more than that it is the fastest by its model (asked of the host side alone)."""
import numpy as np
import pytest

from paper_2207_10702_amd import workloads as wl

torch = pytest.importorskip("torch")

FWD = 0


@pytest.mark.parametrize("I,K,N,Z1,Z2,m", [
    (750, 10432, 2752, 32, 96, 502_916),       # 516 blocks
    (1451, 11520, 1472, 96, 96, 3_344_413),    # 529
    (154, 10240, 11712, 256, 96, 1_705_638),   # 549
    (133, 9920, 11712, 128, 96, 13_077_085),
])
@pytest.mark.parametrize("workspace", [0, 1])
def test_blocks_through_lds_come_in_two_rounds_at_most(roast, I, K, N, Z1, Z2, m, workspace):
    """64 x 64 blocks of mid-sized bf16 calls: a third round of 256 workgroups is no faster than larger blocks."""
    d = roast.mm_desc(K, N, Z1, Z2, m, 2, 1.0, wl.draw_hash(np.random.default_rng(0)))
    blocks = roast.roast_mm_direct_blocks(d, torch.bfloat16, I, FWD, bool(workspace))
    assert not blocks or blocks[:2] != (64, 64) or -(-I // 64) * (N // 64) * blocks[3] <= 512


def test_two_rounds_are_taken(roast):
    d = roast.mm_desc(2048, 2048, 64, 64, 1 << 20, 2, 1.0, wl.draw_hash(np.random.default_rng(0)))
    assert roast.roast_mm_direct_blocks(d, torch.bfloat16, 1024, FWD, False) == (64, 64, 1, 1)
