"""The row kernels as the compiler emits them (no GPU needed: hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2501_08071_amd import build as B

SRC = "rowops_gfx950.hip"


@pytest.fixture(scope="module")
def isa(tmp_path_factory):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("isa") / "rowops.s")
    cmd = [B.HIPCC, *[f for f in B.FLAGS if f != "-fPIC"], "--cuda-device-only", "-S", "-x", "hip", os.path.join(B.CSRC, SRC), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return open(out).read()


def test_results_stay_in_the_caches_for_whoever_reads_them_next(isa):
    """Every store is an ordinary one (a non-temporal store carries the modifier nt)."""
    stores = re.findall(r"^\s*(global_store\w*[^\n]*)", isa, flags=re.M)
    assert len([s for s in stores if s.startswith("global_store_dwordx4")]) >= 100
    assert not [s for s in stores if re.search(r"\bnt\b", s)]


def test_rows_stay_in_registers(isa):
    """No instance keeps any part of a row in scratch memory."""
    sizes = re.findall(r"\.name:\s+(\S*rowop\S*)\n.*?\.private_segment_fixed_size:\s+(\d+)", isa, flags=re.S)
    assert len(sizes) >= 100
    assert not [s for s in sizes if s[1] != "0"]
