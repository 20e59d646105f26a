"""Loading the compiled form of the Python layer's calls: without a usable file, and without what it takes to build one, the library
loads all the same and its calls go through ctypes; a file of other sources is built anew; no process sees half a file; the file has no thread-local data."""
import os
import struct
import subprocess
import warnings

import numpy as np
import pytest

from paper_2207_10702_amd import binding, build, workloads as wl

torch = pytest.importorskip("torch")
if not hasattr(torch._C, "_cuda_getCurrentRawStream"):
    pytest.skip("this torch has no device streams to ask for", allow_module_level=True)


@pytest.fixture
def call_path(tmp_path, monkeypatch):
    binding.load()                             # (with its own file, before the path is another)
    path = str(tmp_path / "_roast_call.so")
    monkeypatch.setattr(binding, "CALL_PATH", path)
    return path


def no_compiler(*args, **kw):
    raise FileNotFoundError("g++")


def failing_compiler(*args, **kw):
    raise subprocess.CalledProcessError(1, "g++")


def host_call():
    """The library answers through ctypes."""
    h = wl.draw_hash(np.random.default_rng(0))
    off, sgn = binding.roast_tile_index(binding.mm_desc(64, 64, 32, 32, 5000, 0, 1.0, h))
    assert len(off) == len(sgn) == 4 and binding.roast_mm_fwd_workspace(binding.mm_desc(64, 64, 32, 32, 5000, 0, 1.0, h), torch.float32, 64) >= 0


@pytest.mark.parametrize("compiler", [no_compiler, failing_compiler])
@pytest.mark.parametrize("there", ["nothing", "no library", "part of one", "another's"])
def test_a_file_that_cannot_be_had_is_done_without(call_path, monkeypatch, compiler, there):
    if there != "nothing":
        with open(os.path.join(os.path.dirname(binding.__file__), "_roast_call.so"), "rb") as f:
            whole = f.read()
        stamp = build.call_stamp().encode()
        assert stamp in whole
        with open(call_path, "wb") as f:
            # (the first with the right mark, so that it is loaded: an ImportError)
            f.write({"no library": b"not an object " + stamp, "part of one": whole[:len(whole) // 3].replace(stamp, b""), "another's": whole.replace(stamp, b"x" * len(stamp))}[there])
    monkeypatch.setattr(build.subprocess, "run", compiler)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_call", None)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        binding.load()
    assert binding._call is None
    host_call()
    assert os.listdir(os.path.dirname(call_path)) == ([] if there == "nothing" else ["_roast_call.so"])      # (nothing left behind)


def test_a_stale_file_is_built_anew_beside_its_place(call_path, monkeypatch):
    with open(call_path, "wb") as f:
        f.write(b"roast_call for other sources")
    real, seen = subprocess.run, []

    def run(cmd, **kw):
        seen.append(cmd[cmd.index("-o") + 1])
        assert seen[-1] != call_path and os.path.dirname(seen[-1]) == os.path.dirname(call_path)
        with open(call_path, "rb") as f:
            assert f.read() == b"roast_call for other sources"
        return real(cmd, **kw)

    monkeypatch.setattr(build.subprocess, "run", run)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        module = binding._connect(binding.load())
    assert module is not None and len(seen) == 1 and build.call_is_current(call_path)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert binding._connect(binding.load()) is not None
    assert len(seen) == 1 and os.listdir(os.path.dirname(call_path)) == ["_roast_call.so"]


def test_the_file_has_no_thread_local_data():
    """With some that no thread uses, every use of another library's thread-local data takes longer as long as the file is loaded."""
    binding.load()
    with open(binding.CALL_PATH, "rb") as f:
        elf = f.read()
    assert elf[:6] == b"\x7fELF\x02\x01"                        # 64 bits, little-endian
    at, = struct.unpack_from("<Q", elf, 32)                      # program headers: where,
    size, count = struct.unpack_from("<HH", elf, 54)             # and how many
    kinds = [struct.unpack_from("<I", elf, at + i * size)[0] for i in range(count)]
    assert 1 in kinds and 7 not in kinds                         # (PT_LOAD, PT_TLS)
