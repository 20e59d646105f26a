"""The compiled form of the Python layer's calls: the results of the Python form (which a call with an explicit stream takes), the same
errors, and anything but a plain tensor left to the Python form."""
import ctypes as C

import numpy as np
import pytest

from paper_2207_10702_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H, O, Z, MS, I = 64, 128, 32, 5000, 48


@pytest.fixture(scope="module")
def case(roast):
    h = wl.draw_hash(np.random.default_rng(3))
    g = torch.Generator(device="cuda").manual_seed(1)
    t = dict(M=torch.randn(MS, generator=g, device="cuda"), X=torch.randn((I, H), generator=g, device="cuda"), dY=torch.randn((I, O), generator=g, device="cuda"),
             rows=torch.arange(I, device="cuda"), tables=torch.arange(I, device="cuda", dtype=torch.int32), g=torch.randn((I, 2 * Z), generator=g, device="cuda"),
             off=torch.arange(0, I + 1, 6, device="cuda"), gb=torch.randn((I // 6, 2 * Z), generator=g, device="cuda"))
    return roast.mm_desc(H, O, Z, Z, MS, 1, 1.0, h), roast.embed_desc(2 * Z, Z, MS, 1.0, h), t


def calls(roast, case, **kw):
    d, e, t = case
    new = lambda *s, dtype=torch.float32: torch.zeros(s, dtype=dtype, device="cuda")  # noqa: E731
    M, S1, S2 = t["M"].clone(), new(MS), new(MS)
    out = [roast.roast_mm_fwd(d, t["X"], t["M"], new(I, O), **kw), roast.roast_mm_bwd_dx(d, t["dY"], t["M"], new(I, H), **kw),
           roast.roast_embed_fwd(e, t["rows"], t["tables"], t["M"], new(I, 2 * Z), **kw),
           roast.roast_embed_bag_fwd(e, t["rows"], t["tables"], t["off"], t["M"], new(I // 6, 2 * Z), **kw),
           roast.roast_m_shadow_bf16(t["M"], new(roast.roast_m_shadow_bytes(MS) // 2, dtype=torch.bfloat16), **kw),
           roast.roast_m_planes_bf16(t["M"], new(roast.roast_m_planes_bytes(MS) // 2, dtype=torch.bfloat16), **kw)]
    det = roast.ROAST_REDUCE_DETERMINISTIC
    ws = lambda n: torch.zeros(n, dtype=torch.uint8, device="cuda")  # noqa: E731
    out.append(roast.roast_mm_bwd_dM(d, t["X"], t["dY"], new(MS), det, ws(roast.roast_mm_bwd_dM_workspace(d, I, det)), **kw))
    out.append(roast.roast_embed_bwd(e, t["rows"], t["tables"], t["g"], new(MS), det, ws(roast.roast_embed_bwd_workspace(e, I, det)), **kw))
    out.append(roast.roast_embed_bag_bwd(e, t["rows"], t["tables"], t["off"], t["gb"], new(MS), det, ws(roast.roast_embed_bag_bwd_workspace(e, I, I // 6, det)), **kw))
    out.append(roast.roast_optim_step(roast.optim_desc(roast.ROAST_OPT_ADAM, 0.1, step=2), M, torch.ones(MS, device="cuda"), S1, S2, **kw))
    return out + [S1, S2]


def test_both_forms_give_the_same(roast, case):
    assert roast._call is not None
    compiled = calls(roast, case)
    for a, b in zip(compiled, calls(roast, case, stream=torch.cuda.current_stream())):
        assert torch.equal(a, b)
    other = torch.cuda.Stream()                                   # the caller's stream
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        again = calls(roast, case)
    torch.cuda.current_stream().wait_stream(other)
    for a, b in zip(compiled, again):
        assert torch.equal(a, b)


def test_what_the_compiled_form_leaves_to_python(roast, case):
    d, e, t = case
    Y = torch.zeros((I, O), device="cuda")
    ok = lambda *a: roast._call.mm_fwd(*a)  # noqa: E731
    assert ok(d, t["X"], t["M"], Y, None, None) == 0
    class Sub(torch.Tensor):
        pass
    for a in ((d, t["X"].as_subclass(Sub), t["M"], Y, None, None), (d, t["X"].cpu(), t["M"], Y, None, None), (d, t["X"].t(), t["M"], Y, None, None),
              (d, t["X"].double(), t["M"], Y, None, None), (d, t["X"], t["M"][::2], Y, None, None), (d, t["X"], t["M"], Y[:-1], None, None),
              (d, t["X"], t["M"], Y.bfloat16(), None, None), (e, t["X"], t["M"], Y, None, None), (d, t["X"], t["M"], Y, Y, None), (d, t["X"], t["M"], Y, None, 3),
              (d, t["X"], None, Y, None, None), (d, t["X"], t["M"], Y, None)):
        assert ok(*a) is None


def test_the_same_errors(roast, case):
    d, e, t = case
    Y = torch.zeros((I, O), device="cuda")
    with pytest.raises(ValueError, match="X must be I x H"):
        roast.roast_mm_fwd(d, t["dY"], t["M"], Y)
    with pytest.raises(ValueError, match="Y must be I x O"):
        roast.roast_mm_fwd(d, t["X"], t["M"], Y[1:])
    with pytest.raises(ValueError, match="X must be a 2-D device tensor"):
        roast.roast_mm_fwd(d, t["X"].cpu(), t["M"], Y)
    with pytest.raises(TypeError):
        roast.roast_mm_fwd(d, t["X"].half(), t["M"], Y.half())
    with pytest.raises(ValueError, match="M_bf16"):
        roast.roast_mm_fwd(d, t["X"], t["M"], Y, M_bf16=t["M"].bfloat16())
    with pytest.raises(ValueError, match="dM must have m_size"):
        roast.roast_mm_bwd_dM(d, t["X"], t["dY"], t["M"][1:])
    with pytest.raises(roast.RoastError) as err:
        roast.roast_mm_bwd_dM(d, t["X"], t["dY"], t["M"].clone(), roast.ROAST_REDUCE_DETERMINISTIC)
    assert err.value.status == roast.ROAST_ERR_WORKSPACE and "roast_mm_bwd_dM" in str(err.value)
    with pytest.raises(ValueError, match="bag_offsets"):
        roast.roast_embed_bag_fwd(e, t["rows"], t["tables"], t["off"].int(), t["M"], torch.zeros((I // 6, 2 * Z), device="cuda"))


class Recorded:
    """torch._C as far as the compiled form asks it, every question noted."""
    def __init__(self):
        self.asked = []

    def _cuda_getDevice(self):
        self.asked.append("device")
        return torch._C._cuda_getDevice()

    def _cuda_getCurrentRawStream(self, device):
        self.asked.append("stream")
        return torch._C._cuda_getCurrentRawStream(device)


@pytest.mark.parametrize("mode", [2 ** 31, -2 ** 31 - 1, 2 ** 40, 2 ** 63, 2 ** 70, -2 ** 70])
def test_a_mode_beyond_an_int_ends_the_checks(roast, case, monkeypatch, mode):
    """Nothing after it is called, least of all with the interpreter's error pending; the Python form then takes it as ctypes does."""
    d, e, t = case
    recorded = Recorded()
    monkeypatch.setattr(roast, "_call", roast._connect(roast.load(), recorded))
    dM = torch.zeros(MS, device="cuda")
    try:
        assert roast._call.mm_bwd_dM(d, t["X"], t["dY"], dM, 0, None) == 0 and recorded.asked == ["device", "stream"]
        assert roast._call.mm_bwd_dM(d, t["X"], t["dY"], dM, mode, None) is None
        assert roast._call.embed_bwd(e, t["rows"], t["tables"], t["g"], dM, mode, None) is None
        assert recorded.asked == ["device", "stream"]
    finally:
        roast._connect(roast.load())


def test_a_descriptor_is_its_own_structure(roast, case):
    """A buffer of its length is none, nor a structure of another name with the same fields; one derived from it is, as for ctypes."""
    d, e, t = case
    o = roast.optim_desc(roast.ROAST_OPT_SGD, 0.1)
    Y, out, dM = torch.zeros((I, O), device="cuda"), torch.zeros((I, 2 * Z), device="cuda"), torch.zeros(MS, device="cuda")
    forms = [(d, lambda x: roast._call.mm_fwd(x, t["X"], t["M"], Y, None, None)), (e, lambda x: roast._call.embed_fwd(x, t["rows"], t["tables"], t["M"], out)),
             (o, lambda x: roast._call.optim_step(x, t["M"].clone(), dM, None, None, None))]
    for desc, call in forms:
        assert call(desc) == 0
        lookalike = type("Lookalike", (C.Structure,), {"_fields_": type(desc)._fields_})
        derived = type("Derived", (type(desc),), {"_fields_": [("note", C.c_int64)]})
        for no in (bytes(desc), bytearray(desc), np.frombuffer(bytes(desc), dtype=np.uint8), lookalike.from_buffer_copy(desc), None, C.byref(desc)):
            assert call(no) is None
        assert call(derived.from_buffer_copy(bytes(desc) + bytes(8))) == 0
        for other, _ in forms:
            assert other is desc or call(other) is None
    with pytest.raises(AttributeError):                           # as without the compiled form
        roast.roast_mm_fwd(bytes(d), t["X"], t["M"], Y)
