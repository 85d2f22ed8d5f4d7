"""The library is built from the sources that are there."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2111_14255_amd import binding, build


def test_host_sources_compile():
    """A library of an older source may be what the tests load, so that the sources compile is shown for itself."""
    def check(src):
        return subprocess.run([build._hipcc(), "-fsyntax-only", os.path.join(build.CSRC, src)] + build.COMMON + build.HOST_FLAGS, capture_output=True, text=True)
    with ThreadPoolExecutor(max_workers=len(build.HOST_SOURCES)) as ex:
        for src, r in zip(build.HOST_SOURCES, ex.map(check, build.HOST_SOURCES)):
            assert r.returncode == 0, "%s\n%s" % (src, r.stderr)


def test_a_build_that_fails_leaves_no_library(tmp_path, monkeypatch):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"an older one")
    (tmp_path / "broken.cpp").write_text("int f( {")
    for name, value in (("CSRC", str(tmp_path)), ("OBJ", str(tmp_path / "obj")), ("LIB", str(lib)), ("DEVICE_SOURCES", []), ("HOST_SOURCES", ["broken.cpp"])):
        monkeypatch.setattr(build, name, value)
    with pytest.raises(RuntimeError, match="compile failed"):
        build.build()
    assert not lib.exists()


def test_a_library_of_other_sources_is_refused(tmp_path, monkeypatch):
    monkeypatch.delenv("MTSCHED_LIB", raising=False)
    binding.load()
    other = tmp_path / "csrc"
    shutil.copytree(build.CSRC, other)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(build, "CSRC", str(other))
    binding.load()                                           # the same contents
    with open(other / "lanes.h", "a") as f:
        f.write(" ")
    monkeypatch.setattr(binding, "_lib", None)
    with pytest.raises(RuntimeError, match="other sources"):
        binding.load()


def test_a_process_tries_to_build_once(tmp_path, monkeypatch):
    monkeypatch.delenv("MTSCHED_LIB", raising=False)
    tries = []

    def fails():
        tries.append(1)
        raise RuntimeError("compile failed")
    for owner, name, value in ((build, "LIB", str(tmp_path / "none.so")), (build, "build", fails), (binding, "_lib", None), (binding, "_unbuilt", None)):
        monkeypatch.setattr(owner, name, value, raising=False)
    for _ in range(2):
        with pytest.raises(RuntimeError, match="compile failed"):
            binding.load()
    assert len(tries) == 1
