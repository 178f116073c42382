"""The streaming attention kernel as the compiler emits it (no GPU needed: hipcc cross-compiles): nothing spills, and the debug build
fills every place in LDS with NaN patterns right before the load that writes it."""
import os
import re
import subprocess

import pytest

from isa_lint import parse
from paper_2501_08071_amd import build as B

SRC = "attn_fwd_stream_gfx950.hip"


@pytest.fixture(scope="module")
def isa(tmp_path_factory):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")

    def emit(*flags):
        out = str(tmp_path_factory.mktemp("isa") / "stream.s")
        res = subprocess.run([B.HIPCC, *[f for f in B.FLAGS if f != "-fPIC"], *flags, "--cuda-device-only", "-S", "-x", "hip", os.path.join(B.CSRC, SRC),
                              "-o", out], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        return open(out).read()

    return {"shipped": emit(), "poison": emit("-DATTN_DEBUG_POISON=1")}


def test_no_spills(isa):
    kernels = parse(isa["shipped"], "attn_fwd_halves_stream_kernel")
    assert len(kernels) == 24                    # two element types, three head dimensions, the mask, one and two row groups
    for name, (ins, _) in kernels.items():
        assert not any(op.startswith("scratch_") for op, _ in ins), name
    assert all(int(n) == 0 for n in re.findall(r"\.vgpr_spill_count:\s+(\d+)", isa["shipped"]))


def test_the_debug_build_poisons_before_every_load(isa):
    kernels = parse(isa["poison"], "attn_fwd_halves_stream_kernel")
    assert len(kernels) == 24
    for name, (ins, _) in kernels.items():
        loads, poisoned = 0, False
        for op, args in ins:
            if op == "ds_write_b128":
                poisoned = True
            elif op.startswith("global_load_lds"):
                assert poisoned, name
                loads, poisoned = loads + 1, False
        # and it takes the same paths: the loads of a whole block, which skip the clamp at the end of the sequence, are there too
        shipped = sum(op.startswith("global_load_lds") for op, _ in parse(isa["shipped"], "attn_fwd_halves_stream_kernel")[name][0])
        assert loads == shipped > 0, (name, loads, shipped)
