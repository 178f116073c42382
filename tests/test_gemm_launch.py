"""The host-side rules of the GEMM launch: tile counts up to the largest sizes the entry point accepts."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
TOP = 2 ** 31 - 1     # the largest M, N or K


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    out = str(tmp_path_factory.mktemp("gemm_launch") / "gemm_launch_host.so")
    res = subprocess.run([gxx, "-std=c++20", "-O1", "-fwrapv", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                          os.path.join(HERE, "csrc", "gemm_launch_host.cpp"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return ctypes.CDLL(out)


@pytest.mark.parametrize("t", [32, 64, 128, 256])
def test_pieces_up_to_the_largest_size(L, t):
    for x in (0, 1, t - 1, t, t + 1, TOP - 256, TOP - 31, TOP - 30, TOP - 1, TOP):
        assert L.pieces(x, t) == -(-x // t), x


def test_tile_choice_at_the_largest_sizes(L):
    """Sums of 2^31 - 1 terms, a single row or column of 2^31 - 1 elements: no overflow on the way to a choice."""
    for shape in ((1, 1, 1, TOP), (1, TOP, 1, 1), (1, 1, TOP, 1), (65535, TOP, 1, 1)):
        assert L.tile_of(*shape) in (1, 2, 3, 5)
