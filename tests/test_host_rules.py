"""Rules of the kernels' launches and index ranges, checked on the host by a
small program built from the kernel headers (tests/host/rules.hip).  CPU only."""
import os
import re
import subprocess

import pytest

from paper_2305_17875_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(build.HERE, "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared", "-O3")]
    subprocess.check_call([build.HIPCC, *flags, "-O1", "-I", os.path.join(build.ROOT, "include"),
                           "-I", CSRC, "-o", exe, os.path.join(HERE, "host", "rules.hip")])

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout
    return run


def test_batched_coarse_correction(rules):
    """Every batched way up takes the coarse correction from the buffer where
    the coarse level's own way up left it: x, the tile path's second buffer or,
    on a marching level, r -- also below a finest level that is too large to
    march (2^28 cells and more)."""
    rules("coarse_correction")
    # the choice is made in one place
    for name in ("kernels.hpp", "tile.hpp", "march.hpp"):
        text = open(os.path.join(CSRC, name)).read()
        assert len(re.findall(r"\.tile \?", text)) == (1 if name == "kernels.hpp" else 0), name


def test_elimination_reads_within_its_block(rules):
    """In the chunked r-line elimination a wavefront reads only the values of
    its own line's wavefronts, and one that holds no line (a batched block of 16
    wavefronts whose lines need 3, 5, 6, ...) reads none, for every line length."""
    rules("elimination_slots")
