"""The library is built from the sources that are there."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2111_14255_amd import build


def test_host_sources_compile():
    """A library of an older source may be what the tests load, so that the sources compile is shown for itself."""
    def check(src):
        return subprocess.run([build._hipcc(), "-fsyntax-only", os.path.join(build.CSRC, src)] + build.COMMON + build.HOST_FLAGS, capture_output=True, text=True)
    with ThreadPoolExecutor(max_workers=len(build.HOST_SOURCES)) as ex:
        for src, r in zip(build.HOST_SOURCES, ex.map(check, build.HOST_SOURCES)):
            assert r.returncode == 0, "%s\n%s" % (src, r.stderr)
