"""Reproducible lookup gradient: the fixed-point scales of its workgroups, bit for bit those that numbers give which no order of
execution changes -- the sample of dOut, the chunks that touch a bucket, the largest of a part's chunks -- also where neighbouring lists
overflow and a chunk that both hold is spilled once or twice, as the order has it.  Values of 2^30 make every scale's rounding visible."""
import numpy as np
import pytest

from paper_2207_10702_amd import workloads as wl
from tests.util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

R = 4096                                  # slots of a bucket (M up to 1 Mi)
LINE = 32                                 # floats that eight threads of a route workgroup sample


def sample(dOut, C):
    """Largest magnitude of what the route workgroups sample: 64 lines each."""
    N, D = dOut.shape
    items = 8192
    while items > 2048 and N * C // items < 256:
        items //= 2
    rows, top = items // C, np.float32(0)
    for n0 in range(0, N, rows):
        own = np.abs(dOut[n0:n0 + rows].reshape(-1))
        share = len(own) // 4 // 64               # of a line, in 16 bytes
        for line in range(64):
            first = 4 * (share * line + (line % (share // 8) * 8 if share >= 8 else 0))
            top = max(top, own[min(first, len(own) - 4):first + LINE].max())
    return top


def exponent(x):
    return int(np.frexp(np.float32(x))[1])


def expected(off, sgn, D, Z, m, dOut):
    """dM by the rule of the header, from the chunks' places (lambda 1)."""
    C = D // Z
    N = len(dOut)
    off, sgn = off.reshape(-1).astype(np.int64), sgn.reshape(-1)
    chunks = dOut.reshape(N * C, Z)
    first, last = off // R, (off + Z - 1) // R
    touching = np.bincount(first, minlength=m // R + 2) + np.bincount(last[last != first], minlength=m // R + 2)
    call_bits = 62 - (N * C).bit_length()
    bits = np.array([min(50, 63 - int(max(c, 1)).bit_length()) for c in touching])       # of a bucket's largest addend
    parts = 1                             # of a bucket, a workgroup each: for most of 512 places
    while parts * -(-m // R) < 400:
        parts *= 2
    S = R // parts
    top = np.zeros(m // S + 2, dtype=np.float32)
    for p in (off // S, (off + Z - 1) // S):
        np.maximum.at(top, p, np.abs(chunks).max(1))
    seen = sample(dOut, C)
    part_bits = bits[np.arange(len(top)) * S // R]
    spare = np.minimum(part_bits - call_bits, 6)
    again = top > np.ldexp(seen, spare)
    shift = np.where(again, part_bits - np.array([exponent(t) for t in top]), part_bits - spare - exponent(seen))
    acc = np.zeros(m, dtype=np.int64)
    for o in range(Z):
        slot = off + o
        np.add.at(acc, slot, np.rint(np.ldexp(chunks[:, o].astype(np.float64) * sgn, shift[slot // S])).astype(np.int64))
    return np.ldexp(acc.astype(np.float64), -shift[np.arange(m) // S]).astype(np.float32), touching, again


def popular(roast, d, h, m, Z, C, want, count=1 << 16):
    """A row of table 0 one of whose chunks starts at an offset that `want` takes."""
    rows = np.arange(count, dtype=np.int64)
    off, _ = roast.roast_chunk_index_device(d, to_dev(rows), to_dev(np.zeros(count, dtype=np.uint32)))
    hit = want(off.cpu().numpy().reshape(count, C)).any(1)
    return int(rows[np.nonzero(hit)[0][0]])


@pytest.mark.parametrize("N,D,Z,m,hot", [
    (70_000, 32, 32, 1_000_000, (0.45, 0.45)),    # two neighbouring lists overflow, one by chunks that belong to both
    (70_000, 32, 32, 1_000_000, (0.45, 0.0)),
    (100_000, 128, 32, 1_000_003, (0.3, 0.0)),    # four popular chunks, one of them across a bucket's end
    (40_000, 128, 64, 500_009, (0.0, 0.0)),
])
@pytest.mark.parametrize("where", ["sampled", "not sampled", "nowhere"])
def test_scales_are_those_of_the_rule(roast, N, D, Z, m, hot, where):
    C = D // Z
    rng = np.random.default_rng(N + Z)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.embed_desc(D, Z, m, 1.0, h)
    across = popular(roast, d, h, m, Z, C, lambda o: (o % R > R - Z) & (o > 2 * R) & (o < m - 2 * R))
    off, _ = roast.roast_chunk_index_device(d, to_dev(np.array([across])), to_dev(np.zeros(1, dtype=np.uint32)))
    off = off.cpu().numpy()
    b = int(off[off % R > R - Z][0]) // R
    inside = popular(roast, d, h, m, Z, C, lambda o: (o // R == b + 1) & (o % R < R - Z))
    u = rng.random(N)
    rows = np.where(u < hot[0], across, np.where(u < sum(hot), inside, rng.integers(0, 1 << 33, N))).astype(np.int64)
    rows[[1, 3]] = across, rows[N // 2]
    tables = np.zeros(N, dtype=np.uint32)
    dOut = rng.standard_normal((N, D)).astype(np.float32)
    if where == "sampled":
        dOut[0, 3] = 1.3 * 2.0 ** 30
    elif where == "not sampled":          # in a popular row, and in any
        dOut[1] *= np.float32(2.0 ** 30)
        dOut[3] *= np.float32(2.0 ** 29)
    off, sgn = roast.roast_chunk_index_device(d, to_dev(rows), to_dev(tables))
    ref, touching, again = expected(off.cpu().numpy(), sgn.cpu().numpy(), D, Z, m, dOut)
    assert again.any() == (where == "not sampled")
    if hot[0]:                            # (a list has room for the mean load and all that the workspace has beyond two of them)
        assert touching[b] > 1.2 * (N * C / (m // R) + 8192)
    args = to_dev(rows), to_dev(tables), to_dev(dOut)
    mode = roast.ROAST_REDUCE_DETERMINISTIC
    for _ in range(3):
        ws = torch.randint(0, 256, (roast.roast_embed_bwd_workspace(d, N, mode),), dtype=torch.uint8, device="cuda")
        dM = torch.zeros(m, device="cuda")
        roast.roast_embed_bwd(d, *args, dM, mode, ws)
        assert np.array_equal(dM.cpu().numpy().view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("N,D,Z,m", [(32_768, 128, 32, 1_000_003), (32_768, 256, 64, 500_009), (69_632, 64, 32, 1_000_003), (16_385, 128, 16, 300_007)])
@pytest.mark.parametrize("part", ["columns", "rows"])
def test_the_sample_is_of_all_columns_and_rows(roast, N, D, Z, m, part):
    """Whole rows to a line's share, and only the first columns, or every second row, small: no workgroup has to start over."""
    rng = np.random.default_rng(N + D)
    h = wl.draw_hash(rng, use_sign=True, align=1)
    d = roast.embed_desc(D, Z, m, 1.0, h)
    rows, tables = rng.integers(0, 1 << 33, N), np.zeros(N, dtype=np.uint32)
    dOut = rng.standard_normal((N, D)).astype(np.float32)
    if part == "columns":
        dOut[:, LINE:] *= np.float32(2.0 ** 30)
    else:
        dOut[1::2] *= np.float32(2.0 ** 30)
    off, sgn = roast.roast_chunk_index_device(d, to_dev(rows), to_dev(tables))
    ref, _, again = expected(off.cpu().numpy(), sgn.cpu().numpy(), D, Z, m, dOut)
    assert not again.any()
    mode = roast.ROAST_REDUCE_DETERMINISTIC
    ws = torch.randint(0, 256, (roast.roast_embed_bwd_workspace(d, N, mode),), dtype=torch.uint8, device="cuda")
    dM = torch.zeros(m, device="cuda")
    roast.roast_embed_bwd(d, to_dev(rows), to_dev(tables), to_dev(dOut), dM, mode, ws)
    assert np.array_equal(dM.cpu().numpy().view(np.uint32), ref.view(np.uint32))
