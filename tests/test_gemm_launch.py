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
    lib = ctypes.CDLL(out)
    lib.position64.argtypes = [ctypes.c_longlong] * 3
    lib.position64.restype = ctypes.c_longlong
    return lib


@pytest.mark.parametrize("t", [32, 64, 128, 256])
def test_pieces_up_to_the_largest_size(L, t):
    for x in (0, 1, t - 1, t, t + 1, TOP - 256, TOP - 31, TOP - 30, TOP - 1, TOP):
        assert L.pieces(x, t) == -(-x // t), x


def test_tile_choice_at_the_largest_sizes(L):
    """Sums of 2^31 - 1 terms, a single row or column of 2^31 - 1 elements: no overflow on the way to a choice."""
    for shape in ((1, 1, 1, TOP), (1, TOP, 1, 1), (1, 1, TOP, 1), (65535, TOP, 1, 1)):
        assert L.tile_of(*shape) in (1, 2, 3, 5)


def grid_of(L, *args):
    out = (ctypes.c_longlong * 5)()
    L.grid_of(*args, out)
    return list(out)


@pytest.mark.parametrize("batch,M,N,t", [(1, 1, 1, 64), (3, 70, 130, 64), (65535, 1, 64 * 65, 64), (16, 2 ** 28, 8, 256), (1, TOP, 1, 32),
                                         (65535, 4, 1 << 20, 256), (4, 32, 32 << 20, 32)])
def test_grid_holds_every_tile(L, batch, M, N, t):
    """No dimension of 2^32 threads or more, and no more than one surplus row of workgroups."""
    tm, tn, total, x, y = grid_of(L, batch, M, N, t, t)
    assert (tm, tn) == (-(-M // t), -(-N // t)) and total == tm * tn * batch
    assert x * 256 < 2 ** 32 and y <= 65535 and x * y >= total > x * (y - 1)
    assert y == 1 or x % 8 == 0        # a workgroup's number modulo 8 is its XCD also in the second dimension


@pytest.mark.parametrize("group", [0, 1, 4, 64, 100, 128, 129, 1000])
@pytest.mark.parametrize("total", [1, 7, 8, 9, 31, 32, 100, 257, 512, 513, 514, 1024, 1025, 4099])
def test_list_positions_are_a_permutation(L, total, group):
    """Every XCD (number modulo 8) a run of its own, every position once."""
    pos = [L.position32(b, total, group) for b in range(total)]
    assert [L.position64(b, total, group) for b in range(total)] == pos
    end = 0
    for x in range(min(8, total)):
        run = sorted(pos[x::8])
        assert run == list(range(end, end + len(run)))
        end += len(run)
    assert end == total


def test_list_positions_above_2_to_the_31(L):
    total = 2 ** 33 + 5                    # runs of 2^30 + 1 for XCD 0 to 4, of 2^30 for the others
    start = [x * 2 ** 30 + min(x, 5) for x in range(9)]
    for b in (0, 1, 7, 8, 12, total - 8, total - 1):
        x = b % 8
        run = start[x + 1] - start[x]
        assert L.position64(b, total, 0) == start[x] + b // 8
        for group in (2 ** 10, 2 ** 32):     # whole groups, parts of a group
            assert L.position64(b, total, group) == start[x] + (b // 8 + x * run // 8) % run
        assert L.position64(b, total, 1000) == start[x] + b // 8


@pytest.mark.parametrize("tiles_m,tiles_n", [(32, 32), (32, 33), (32, 95), (64, 32), (16, 64)])
def test_many_rounds_do_not_march_in_step(L, tiles_m, tiles_n):
    """Large matrices in tiles of 256: no more than two XCDs in the same column of tiles."""
    total = tiles_m * tiles_n
    for b in range(0, total // 8, 8):
        cols = [L.tile_in_list(L.position32(b + x, total, 4 * tiles_n), tiles_m, tiles_n, 0) % tiles_n for x in range(8)]
        assert max(cols.count(c) for c in cols) <= 2


@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (3, 7), (4, 5), (5, 64), (7, 9), (8, 8), (9, 40), (11, 3), (16, 16), (1, 300), (300, 1)])
def test_every_tile_once_in_compact_blocks(L, tiles_m, tiles_n):
    apart = [L.tile_in_list(t, tiles_m, tiles_n, 0) for t in range(tiles_m * tiles_n)]
    assert sorted(apart) == list(range(tiles_m * tiles_n))      # 256 x 256 tiles: the last rows may be a group of their own
    assert {i // tiles_n for i in apart[:4 * tiles_n]} == set(range(min(4, tiles_m)))
    order = [L.tile_in_list(t, tiles_m, tiles_n, 1) for t in range(tiles_m * tiles_n)]
    assert sorted(order) == list(range(tiles_m * tiles_n))
    # 32 neighbours in the list (what an XCD runs together) touch few rows and columns: never a run along one row
    # of tiles where there are more rows to choose from
    for s in range(0, len(order) - 31, 32):
        rows = {i // tiles_n for i in order[s:s + 32]}
        cols = {i % tiles_n for i in order[s:s + 32]}
        assert tiles_m < 4 or tiles_n == 1 or len(rows) + len(cols) <= 20, (s, len(rows), len(cols))


@pytest.mark.parametrize("shape,tile", [((1024, 8, 64, 64), 3), ((4096, 64, 1024, 64), 3), ((4096, 65, 1024, 64), 2), ((4096, 128, 1024, 64), 2),
                                        ((4096, 129, 1024, 64), 1), ((4096, 129, 128, 64), 2), ((1, 1 << 20, 8, 32), 3), ((1, 1 << 20, 72, 32), 2),
                                        ((1, 1 << 20, 136, 32), 1), ((1, 3584, 3584, 32), 1),
                                        ((4, 64, 8192, 736), 3), ((4, 64, 8192, 768), 2), ((4, 8192, 64, 4096), 3)])
def test_tiles_are_not_more_than_half_empty(L, shape, tile):
    assert L.tile_of(*shape) == tile


def test_deep_pipelines_are_for_long_sums(L):
    for shape, want in (((1024, 64, 64, 64), 0), ((1, 1000, 1000, 128), 0), ((1, 32768, 64, 384), 0), ((1, 700, 480, 448), 0), ((1, 300, 1400, 639), 0),
                        ((1, 64, 9000, 287), 0), ((1, 64, 9000, 288), 1), ((1, 1000, 1000, 640), 1), ((4, 512, 512, 2048), 1)):
        assert L.deep(*shape) == want, shape


def test_one_round_of_larger_tiles(L):
    """Tiles between the square ones, on either side of each condition."""
    for shape, want in (((1, 1536, 1536, 4096), 2), ((1, 1536, 1536, 640), 2), ((1, 1536, 1536, 632), 3), ((1, 1664, 1536, 384), 2), ((1, 1664, 1536, 376), 3),
                        ((8, 556, 448, 1536), 3), ((1, 1536, 1280, 4096), 3), ((2, 777, 1000, 1000), 3)):
        assert L.tile_of(*shape) == want, shape
    # (the first five and the last but one were 4 to 13 % slower with 128 x 128: one round of 64 x 64 tiles, two to a compute unit)
    for shape, want in (((1, 5952, 320, 1024), 3), ((2, 2176, 448, 1024), 3), ((2, 1728, 576, 2048), 3), ((2, 1408, 704, 704), 3), ((2, 2784, 288, 1440), 3), ((4, 1600, 320, 1024), 3),
                        ((1, 6395, 264, 2048), 2), ((1, 6395, 264, 1192), 3), ((1, 4736, 448, 1024), 2), ((1, 4864, 448, 512), 2), ((4, 704, 704, 3368), 2),
                        ((2, 2200, 448, 2992), 3), ((1, 5984, 296, 488), 3)):
        assert L.tile_of(*shape) == want, shape
    for shape, want in (((1, 3072, 1536, 3072), 1), ((1, 3072, 1536, 376), 0), ((1, 2048, 2048, 2048), 0), ((1, 2176, 4096, 1000), 0), ((20, 1792, 128, 1024), 0)):
        assert L.tiles_128x256(*shape) == want, shape
    for shape, want in (((1, 1536, 1536, 1280), 1), ((1, 1536, 1536, 1272), 0), ((1, 1536, 1536, 1288), 1), ((1, 1536, 1536, 1312), 0), ((1, 2176, 2048, 2048), 0)):
        assert L.two_parts(*shape) == want, shape
    for shape, want in (((2, 777, 1000, 1000), 1), ((2, 777, 1000, 592), 0), ((2, 777, 1000, 600), 1), ((2, 777, 1000, 608), 0), ((20, 1792, 128, 1024), 0), ((1, 1000, 1000, 1000), 0), ((1, 1536, 1536, 1024), 0), ((1, 20000, 64, 1024), 0),
                        ((8, 64, 4096, 760), 0), ((5, 64, 4096, 768), 1), ((1, 4071, 320, 704), 0), ((1, 4071, 320, 2560), 1)):
        assert L.tiles_64x128(*shape) == want, shape
    for shape, want in (((4, 512, 512, 2048), 1), ((4, 512, 512, 2056), 0), ((4, 512, 512, 576), 0), ((1, 1024, 1088, 1024), 0)):
        assert L.long_blocks(*shape) == want, shape


def test_the_shapes_of_the_gpu_tests_take_the_tiles_they_are_for(L):
    """test_gemm_gpu.py's shapes between the square tiles, and of rows that are not aligned, by the tile and the block of K they take."""
    from test_gemm_gpu import BETWEEN

    def route(batch, M, N, K):
        s = (batch, M, N, K)
        if L.per_element(*s) and (K % 32 or N % 8):
            return "element"
        if K % 8 or N % 8:
            return ("any 64, %d" % (64 if L.unaligned_blocks_64(*s) else 32)) if L.unaligned_64(*s) else "any 32"
        tile = L.tile_of(*s)
        if tile == 2:
            return "128 x 256" if L.tiles_128x256(*s) else "two parts" if L.two_parts(*s) else "128"
        if tile == 3:
            return "64 x 128" if L.tiles_64x128(*s) else "64, long" if L.long_blocks(*s) else "64"
        return str(tile)

    want = ["64 x 128"] * 4 + ["two parts"] * 3 + ["128 x 256"] * 3 + ["64, long"] * 2
    assert [route(*s) for s in BETWEEN[:12]] == want
    rest = [route(*s) for s in BETWEEN[12:]]
    assert set(rest) == {"any 64, 32", "any 64, 64"} and rest.count("any 64, 32") >= 5 and rest.count("any 64, 64") >= 5


def test_unaligned_rows(L):
    """64 x 64 tiles from more than 512 (640) tiles of 32 x 32 on, in blocks of 64 for a long K or a middling one with few tiles."""
    for shape, want in (((2, 512, 511, 100), 0), ((2, 513, 511, 100), 1), ((2, 640, 511, 1201), 0), ((2, 641, 511, 1201), 1), ((1, 1 << 20, 7, 100), 0), ((1, 1 << 20, 8, 100), 1),
                        ((1, 20000, 9, (1 << 22) + 1), 0), ((65535, 1, TOP, 1), 0)):
        assert L.unaligned_64(*shape) == want, shape
    for shape, want in (((1, 1500, 1501, 256), 0), ((1, 1500, 1501, 257), 1), ((1, 1600, 1601, 257), 0), ((1, 1600, 1601, 701), 1)):
        assert L.unaligned_blocks_64(*shape) == want, shape
    assert L.per_element(2, 2318, 2350, 86) == 0 and L.per_element(1, 660, 3283, 33) == 0


def test_few_products_take_one_thread_per_element(L):
    """Sizes that fit no tile, on either side by a factor in the time measured."""
    for shape in ((4000, 1, 9, 3), (4000, 1, 35, 17), (1, 1, 65537, 7), (1, 33, 33, 1), (1, 1500, 1500, 8), (16384, 8, 64, 8), (1, 1 << 20, 8, 8),
                  (1, 5, 7, 0), (1, TOP, 1, 1), (1, 1, TOP, 1)):
        assert L.per_element(*shape) == 1, shape
    for shape in ((1, 1003, 1003, 129), (1, 65536, 64, 40), (2, 777, 1000, 1000), (1, 777, 1001, 1003), (1, 1000, 8, 1000), (16384, 33, 64, 40),
                  (1, 3000, 1500, 3008), (1, 1, 1, TOP)):
        assert L.per_element(*shape) == 0, shape


def test_tall_and_short_products(L):
    """A single column of tiles goes through memory in order unless the product is long; two wavefronts per SIMD for two blocks
    of K where the tiles are few or in one column, up to four or eight of them with fewer tiles still, and for a long K in one column."""
    for args, want in (((200, 64, 200), 1), ((256, 128, 256), 1), ((129, 128, 257), 0), ((256, 160, 200), 0), ((256, 64, 4096), 1), ((256, 32, 4096), 0),
                       ((248, 64, 513), 0), ((257, 64, 200), 0), ((256, 40, 200), 1), ((256, 56, 257), 0)):
        assert L.in_order(*args) == want, args
    for args, want in (((1, 3584, 3584, 64), 1), ((1, 3584, 3584, 65), 1), ((1, 3584, 3584, 128), 1), ((1, 3584, 3584, 136), 0),
                       ((1, 4096, 4096, 64), 0), ((1, 4096, 3840, 32), 1), ((1, 1 << 20, 256, 64), 1),
                       ((1, 1 << 20, 264, 64), 0), ((1, 1 << 20, 256, 72), 0), ((1, 1 << 20, 256, 32), 0), ((1, 1 << 20, 256, 56), 0), ((448, 256, 256, 32), 1), ((449, 256, 256, 32), 0),
                       ((200, 256, 512, 24), 0), ((100, 256, 512, 24), 1), ((200, 256, 256, 32), 1), ((200, 256, 256, 8), 0), ((1, 50000, 256, 64), 1),
                       ((1, 50000, 512, 64), 0), ((1, 3500, 3584, 64), 0), ((1, 3584, 3496, 64), 0),
                       ((1, 256, 53248, 256), 1), ((1, 256, 53504, 256), 0), ((1, 256, 53248, 264), 0), ((1, 3840, 4096, 96), 0), ((208, 256, 256, 72), 1),
                       ((1, 49152, 136, 1536), 1), ((1, 49152, 256, 1504), 0), ((1, 49152, 256, 2056), 0), ((1, 49100, 256, 2048), 0), ((200, 256, 256, 2048), 0),
                       ((1, 1 << 17, 200, TOP - 31), 1), ((1, 1 << 18, 200, 2048), 0), ((1, 24576, 512, 8192), 0)):
        assert L.eight_waves(*args) == want, args
    # in runs, in runs that start apart, one after the other
    for args, want in (((1, 4096, 4096, 64), 0), ((1, 8192, 8192, 64), 1), ((1, 7203, 16848, 1280), 0), ((200, 256, 256, 64), 2), ((1, 1 << 20, 256, 64), 2),
                       ((1 << 23, 256, 256, 64), 1)):
        assert L.order_of(*args) == want, args
