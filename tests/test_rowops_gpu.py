"""Parity of the HIP row kernels (softmax, rmsnorm; include/rowops.h) against the float64 oracle.

Tolerance.  Both kernels compute in fp32 and round once, to nearest even, into the 16-bit output type.  The
fp32 part is within 3e-5 relative of the exact value (the exponent's argument (x - m) log2(e) is rounded to
fp32 at magnitudes up to a few hundred: 2^-24 * 300 * ln 2 = 1.3e-5; sums of up to 16384 fp32 terms of
one sign; one-ulp exp2, sqrt and division), the final rounding adds half an ulp of the output: 2^-11
relative for binary16, 2^-8 for bfloat16; below the smallest normal binary16 value the spacing is the
absolute 2^-24.  So |y - ref| <= (2^-p + 3e-5) |ref| + floor, p = 11 / 8, floor = 2^-25 (binary16: half a
subnormal step) or 1e-37 (bfloat16: its smallest normal values; fp32 flushes nothing above that).
"""
import numpy as np
import pytest
import torch

from oracle import rowops as R
from paper_2501_08071_amd import inputs as I

pytestmark = pytest.mark.gpu

REL = {I.F16: 2.0 ** -11 + 3e-5, I.BF16: 2.0 ** -8 + 3e-5}
FLOOR = {I.F16: 2.0 ** -25, I.BF16: 1e-37}
TDT = {I.F16: torch.float16, I.BF16: torch.bfloat16}


@pytest.fixture(scope="module")
def P():
    import paper_2501_08071_amd as pkg
    assert torch.cuda.is_available()
    pkg.lib
    return pkg


def dev(bits, dtype):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(TDT[dtype])


def host_bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def check(y_bits, ref, dtype, what):
    got = R.widen(y_bits, dtype).reshape(ref.shape)
    assert np.all(np.isfinite(got)), what
    err = np.abs(got - ref)
    tol = REL[dtype] * np.abs(ref) + FLOOR[dtype]
    worst = np.unravel_index(np.argmax(err - tol), err.shape)
    assert np.all(err <= tol), f"{what}: |{got[worst]} - {ref[worst]}| = {err[worst]:.3e} > {tol[worst]:.3e} at {worst}"


# row lengths: 8 .. 64 lanes per row, a workgroup per row with 1, 2, 4 chunks per thread, lengths that leave lanes and chunks idle,
# lengths that are no multiple of 8, or longer than 16384 (what rowops_path calls 2), and, below 8, the general path
LENGTHS = [8, 16, 24, 64, 72, 128, 200, 256, 264, 512, 520, 1000, 2048, 2056, 4096, 4104, 8192, 8200, 16384,
           1, 2, 7, 9, 63, 1001, 4095, 16392, 20001]


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("n", LENGTHS)
def test_softmax_small(P, n, dtype):
    n_rows = 37 if n <= 4104 else 5          # several workgroups and a ragged last one
    xb = I.gen_rows(n_rows, n, dtype, mul=3.0)
    assert P.rowops_path(0, n, dtype) == (1 if n % 8 == 0 and n <= 16384 else 2)
    y = P.softmax_rows_fwd(dev(xb, dtype))
    torch.cuda.synchronize()
    check(host_bits(y), R.softmax_rows(xb, dtype), dtype, f"softmax n={n}")


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("n", LENGTHS)
def test_rmsnorm_small(P, n, dtype):
    n_rows = 37 if n <= 4104 else 5
    xb = I.gen_rows(n_rows, n, dtype, tensor_id=0)
    wb = I.gen_rows(1, n, dtype, tensor_id=1)[0]
    y = P.rmsnorm_fwd(dev(xb, dtype), dev(wb, dtype), 1e-6)
    torch.cuda.synchronize()
    check(host_bits(y), R.rmsnorm_rows(xb, wb, 1e-6, dtype), dtype, f"rmsnorm d={n}")


def test_softmax_paper_shape_every_element(P):
    """Table 2: softmax over n_rows x n_cols = 512 x 4096, float16."""
    _, n_rows, n, dt = I.ROWOP_SHAPES["softmax_512x4096_f16"]
    xb = I.gen_rows(n_rows, n, dt)
    y = P.softmax_rows_fwd(dev(xb, dt))
    torch.cuda.synchronize()
    check(host_bits(y), R.softmax_rows(xb, dt), dt, "softmax 512x4096")


def test_rmsnorm_paper_shape_every_element(P):
    """Table 2: rmsnorm over B, n_head, seq_len, d_head = 1, 32, 4096, 64, float16 (131072 rows of 64)."""
    _, n_rows, n, dt = I.ROWOP_SHAPES["rmsnorm_1x32x4096x64_f16"]
    xb = I.gen_rows(n_rows, n, dt, tensor_id=0)
    wb = I.gen_rows(1, n, dt, tensor_id=1)[0]
    x = dev(xb, dt).view(1, 32, 4096, 64)
    y = P.rmsnorm_fwd(x, dev(wb, dt), 1e-6)
    torch.cuda.synchronize()
    assert y.shape == x.shape
    check(host_bits(y).reshape(n_rows, n), R.rmsnorm_rows(xb, wb, 1e-6, dt), dt, "rmsnorm 1x32x4096x64")


def test_many_rows_stride_over_the_grid(P):
    """More row groups than the grid has workgroups: the kernels stride."""
    dt = I.F16
    xb = I.gen_rows(8192 * 32 + 77, 8, dt)             # 8 lanes per row, 32 rows per workgroup, > 8192 groups
    wb = I.gen_rows(1, 8, dt, tensor_id=1)[0]
    check(host_bits(P.rmsnorm_fwd(dev(xb, dt), dev(wb, dt), 1e-5)), R.rmsnorm_rows(xb, wb, 1e-5, dt), dt, "rmsnorm many rows")
    check(host_bits(P.softmax_rows_fwd(dev(xb, dt))), R.softmax_rows(xb, dt), dt, "softmax many rows")
    xb = I.gen_rows(8192 + 5, 9, dt)                   # unaligned rows of one chunk and one element
    check(host_bits(P.softmax_rows_fwd(dev(xb, dt))), R.softmax_rows(xb, dt), dt, "softmax many rows of 9")


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
def test_degenerate_rows(P, dtype):
    # constant rows -> 1/n; one dominant entry -> (1, 0, ...); the largest finite inputs; a row of zeros for rmsnorm
    big = 65504.0 if dtype == I.F16 else 3.0e38
    rows = np.zeros((6, 64), np.float32)
    rows[0, :] = 2.5
    rows[1, 3] = 40.0
    rows[2, :] = -big
    rows[2, 5] = big
    rows[3, :] = big
    rows[4, ::2] = -1.0
    xb = I.to_bits(rows, dtype)
    y = P.softmax_rows_fwd(dev(xb, dtype))
    check(host_bits(y), R.softmax_rows(xb, dtype), dtype, "softmax degenerate")
    got = R.widen(host_bits(y), dtype)
    assert np.all(got[0] == R.widen(I.to_bits(np.float32([1 / 64]), dtype), dtype)[0])
    assert got[2, 5] == 1.0 and got[2].sum() == 1.0
    x2 = rows.copy()
    x2[2, :] = 0.0
    x2[3, :] = 100.0
    xb2 = I.to_bits(x2, dtype)
    wb = I.to_bits(np.linspace(-2, 2, 64, dtype=np.float32), dtype)
    for eps in (0.0, 1e-6, 1.0):
        if eps == 0.0:
            xb_e = np.delete(xb2, [2, 5], axis=0)     # 0/0 is left out: inputs are assumed to make sense
        else:
            xb_e = xb2
        y = P.rmsnorm_fwd(dev(xb_e, dtype), dev(wb, dtype), eps)
        check(host_bits(y), R.rmsnorm_rows(xb_e, wb, eps, dtype), dtype, f"rmsnorm degenerate eps={eps}")


def test_in_place_and_preallocated(P):
    dt = I.BF16
    for n in (64, 4096, 1001):
        xb = I.gen_rows(19, n, dt, mul=2.0)
        x = dev(xb, dt)
        ref = R.softmax_rows(xb, dt)
        out = torch.full_like(x, 7.0)
        assert P.softmax_rows_fwd(x, y=out) is out
        check(host_bits(out), ref, dt, "softmax preallocated")
        P.softmax_rows_fwd(x, y=x)
        check(host_bits(x), ref, dt, "softmax in place")
        wb = I.gen_rows(1, n, dt, tensor_id=1)[0]
        x = dev(xb, dt)
        P.rmsnorm_fwd(x, dev(wb, dt), 1e-6, y=x)
        check(host_bits(x), R.rmsnorm_rows(xb, wb, 1e-6, dt), dt, "rmsnorm in place")


def test_empty_input_and_errors(P):
    x = torch.empty((0, 64), dtype=torch.float16, device="cuda")
    assert P.softmax_rows_fwd(x).shape == (0, 64)
    assert P.rmsnorm_fwd(x, torch.ones(64, dtype=torch.float16, device="cuda"), 1e-6).shape == (0, 64)
    x = torch.ones((4, 64), dtype=torch.float16, device="cuda")
    with pytest.raises(P.RowopsError) as e:
        P.rmsnorm_fwd(x, torch.ones(64, dtype=torch.float16, device="cuda"), -1.0)
    assert e.value.status == -4
    with pytest.raises(TypeError):
        P.softmax_rows_fwd(x.float())
    with pytest.raises(ValueError):
        P.rmsnorm_fwd(x, torch.ones(32, dtype=torch.float16, device="cuda"), 1e-6)
    with pytest.raises(ValueError):
        P.softmax_rows_fwd(x.t())


def test_side_stream_and_repeatability(P):
    dt = I.F16
    xb = I.gen_rows(512, 4096, dt)
    x = dev(xb, dt)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a = P.softmax_rows_fwd(x, stream=s)
    s.synchronize()
    b = P.softmax_rows_fwd(x)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    check(host_bits(a), R.softmax_rows(xb, dt), dt, "softmax side stream")


# (rows, length): the last chunk of a row moved back over 1 .. 7 elements, a row of one or two chunks; every choice of
# threads per row, on either side of the number of rows that decides (1024 workgroups of four steps, 4096, 8192, 2048
# rows) with a ragged last step; the longest row kept in registers and the first one that is not
@pytest.mark.parametrize("op", ["softmax", "rmsnorm"])
@pytest.mark.parametrize("n_rows,n", [(37, 8 + i) for i in range(1, 8)] + [
    (131072 + 5, 33), (131071, 33), (32768 + 3, 257), (16384 + 1, 511), (16384 + 3, 1023), (37, 1025), (4096 + 1, 1027),
    (4095, 1030), (8192 + 1, 2050), (8191, 2051), (2048 + 1, 4100), (2047, 4097), (2048 + 1, 8196), (2047, 8193), (3, 16391),
    (300, 32767), (3, 65535), (3, 65529), (2, 65536), (2, 65537)])
def test_row_kernel_choices(P, op, n_rows, n):
    check_choice(P, op, n_rows, n)


# the lines between 256, 512 and 1024 threads for rows of 4097 to 16384 elements, aligned and not, with full and partly idle threads
@pytest.mark.parametrize("op", ["softmax", "rmsnorm"])
@pytest.mark.parametrize("n_rows,n", [(8191, 5120), (8192, 5120), (8192, 5128), (2047, 8192), (2049, 8192), (2048, 5121), (399, 8201), (400, 8201), (401, 12288),
                                      (401, 12285), (401, 12296), (401, 12289), (2047, 16384), (37, 16383)])
def test_choices_for_long_rows(P, op, n_rows, n):
    check_choice(P, op, n_rows, n)


def check_choice(P, op, n_rows, n):
    dt = I.BF16 if (n_rows + n) % 2 else I.F16
    g = torch.Generator().manual_seed(n_rows * 131 + n)
    x = (torch.randn(n_rows, n, generator=g) * 2).to(TDT[dt])
    w = torch.randn(n, generator=g).to(TDT[dt])
    # a guard row after the tensor and a guard value before it: nothing outside may be written
    buf = torch.full(((n_rows + 1) * n + 8,), 7.0, dtype=TDT[dt], device="cuda")
    y = buf[8:8 + n_rows * n].view(n_rows, n)
    xd, wd = x.cuda(), w.cuda()
    P.softmax_rows_fwd(xd, y=y) if op == "softmax" else P.rmsnorm_fwd(xd, wd, 1e-6, y=y)
    torch.cuda.synchronize()
    x64 = x.cuda().double()
    ref = torch.softmax(x64, 1) if op == "softmax" else x64 / (x64.square().mean(1, keepdim=True) + 1e-6).sqrt() * wd.double()
    err = (y.double() - ref).abs() - (REL[dt] * ref.abs() + FLOOR[dt])
    assert err.max().item() <= 0, (op, n_rows, n, err.max().item())
    assert torch.equal(buf[:8].cpu(), torch.full((8,), 7.0, dtype=TDT[dt]))
    assert (buf[8 + n_rows * n:] == 7.0).all()


# rows that several wavefronts share, with a last chunk that reads and stores elements of the one before it
@pytest.mark.parametrize("n_rows,n", [(19, 2049), (19, 4095), (3000, 4100), (19, 8193), (5, 12289), (5, 32767), (3, 65535), (19, 8192), (5, 16384)])
def test_long_rows_in_place(P, n_rows, n):
    dt = I.BF16
    xb = I.gen_rows(n_rows, n, dt, mul=2.0)
    wb = I.gen_rows(1, n, dt, tensor_id=1)[0]
    for x in (dev(xb, dt), dev(xb, dt)):
        want = P.softmax_rows_fwd(x)
        P.softmax_rows_fwd(x, y=x)
        assert torch.equal(x.view(torch.int16), want.view(torch.int16))
        x = dev(xb, dt)
        want = P.rmsnorm_fwd(x, dev(wb, dt), 1e-6)
        P.rmsnorm_fwd(x, dev(wb, dt), 1e-6, y=x)
        assert torch.equal(x.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("n", [5, 8, 9, 64, 100, 515, 1000, 2051, 4096, 8193, 16385, 40000])
def test_softmax_of_masked_rows(P, n, dtype):
    """Minus infinity is a mask: zeros there, the others as if it were not (a whole chunk, the first element, the last eight);
    a row with a NaN is NaN, a row of nothing but minus infinity too, and neither touches its neighbours."""
    g = torch.Generator().manual_seed(n)
    x = (torch.randn(9, n, generator=g) * 2).to(TDT[dtype])
    ninf = float("-inf")
    x[0, : n // 2] = ninf
    x[1, n - 1] = ninf
    x[2, max(0, n - 8):] = ninf if n > 8 else x[2, max(0, n - 8):]
    x[3, :-1] = ninf
    x[4, 0] = ninf
    x[5] = ninf
    x[6, n // 3] = float("nan")
    x[7, n - 1] = float("nan")
    y = P.softmax_rows_fwd(x.cuda()).double().cpu()
    torch.cuda.synchronize()
    ref = torch.softmax(x.double(), 1)
    assert torch.isnan(ref[5:8]).all() and torch.isnan(y[5:8]).all()
    ok = [0, 1, 2, 3, 4, 8]
    assert ((y[ok] - ref[ok]).abs() <= REL[dtype] * ref[ok].abs() + FLOOR[dtype]).all()
    assert (y[0, : n // 2] == 0).all() and y[3, n - 1] == 1.0


@pytest.mark.parametrize("n_rows,n", [(8192 + 5, 7), (8192 + 5, 1), (2, 65537), (1, 100001)])
def test_general_path(P, n_rows, n):
    """Rows shorter than 8 or longer than 65536 elements, one workgroup per row; more rows than a grid has workgroups."""
    dt = I.F16
    xb = I.gen_rows(n_rows, n, dt)
    wb = I.gen_rows(1, n, dt, tensor_id=1)[0]
    check(host_bits(P.softmax_rows_fwd(dev(xb, dt))), R.softmax_rows(xb, dt), dt, f"softmax {n_rows} x {n}")
    check(host_bits(P.rmsnorm_fwd(dev(xb, dt), dev(wb, dt), 1e-5)), R.rmsnorm_rows(xb, wb, 1e-5, dt), dt, f"rmsnorm {n_rows} x {n}")
