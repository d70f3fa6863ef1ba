"""Device arithmetic compiled for the host and checked against double precision.

- gfc::sincospi_poly (sin/cos of pi r, a Taylor polynomial on |f| <= 1/4
  after reduction by half turns): absolute error below 1.5e-7 over a dense
  sweep of |r| <= 512 (the phases the kernels form) and a random sample,
  exact values at integer and half-integer r, and odd/even symmetry bit for
  bit (the kernels take the omega = -1/2 phase as the conjugate of the
  omega = +1/2 one).
- gfc::fft<N, SIGN>, the in-register FFTs of every kernel."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_sincospi_poly_accuracy(tmp_path):
    exe = tmp_path / "sincospi_check"
    cmd = ["hipcc", "-O2", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "paper_2012_15797_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "native", "sincospi_check.hip"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout.split()
    err_s, err_c, bad_exact, bad_sym = float(out[0]), float(out[1]), int(out[2]), int(out[3])
    assert err_s < 1.5e-7 and err_c < 1.5e-7, (err_s, err_c)
    assert bad_exact == 0
    assert bad_sym == 0


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_register_fft_accuracy(tmp_path):
    """The kernels' in-register FFTs (gfc::fft<N, SIGN>: decimation-in-time
    stages whose twiddles are written as a real scale times (1 + i tan) or
    (cot + i) and folded into FMA butterflies), compiled for the host and
    compared with a double-precision direct DFT of the same inputs at every
    power-of-two length 1..256 and both signs: error relative to the largest
    output below 4e-7 (a few float32 roundings per stage), and exact results
    for a unit impulse and a constant."""
    exe = tmp_path / "fft_check"
    cmd = ["hipcc", "-O2", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "paper_2012_15797_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "native", "fft_check.hip"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout.splitlines()
    seen = set()
    for line in lines:
        n, sign, err, bad = line.split()
        seen.add((int(n), int(sign)))
        assert float(err) < 4e-7, line
        assert int(bad) == 0, line
    assert seen == {(1 << e, s) for e in range(9) for s in (1, -1)}


def _shift_phase_cmd():
    return ["hipcc", "-std=c++17", "-O3", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
            "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2012_15797_amd", "csrc"), "-I",
            os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "shift_phase_check.hip")]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_shift_phase_accuracy(tmp_path):
    """The phase of a whole shift at every stamp size.  Its argument hi + lo / pi:
    lo / pi is the sum of two roundings of at most 2^-24 half turns each, itself
    rounded three times and scaled by a float32 pi, so the argument is within
    2^-46.  The phase: sincospi_poly's 1.5e-7 and one rounding, 2^-25."""
    exe = tmp_path / "shift_phase_check"
    subprocess.run([*_shift_phase_cmd(), "-o", str(exe)], check=True, capture_output=True, timeout=300)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout.splitlines()
    assert [int(line.split()[0]) for line in lines] == [16, 32, 64, 128, 256]
    for line in lines:
        _, arg, phase = line.split()
        assert float(arg) < 2.0 ** -46, line
        assert float(phase) < 1.5e-7 + 2.0 ** -25, line


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_shift_argument_is_not_contracted(tmp_path):
    """On the device the sums and products of the argument are the ones that are
    written: none may be fused with another (fused, p - (hi - bb) takes the
    unrounded product and pe is counted twice, an error of up to 1.9e-7)."""
    ir = tmp_path / "shift_arg.ll"
    subprocess.run([*_shift_phase_cmd(), "--offload-device-only", "-S", "-emit-llvm", "-o", str(ir)], check=True,
                   capture_output=True, timeout=300)
    body = ir.read_text().split("shift_arg_kernel", 1)[1].split("\n}", 1)[0].splitlines()
    ops = [line.split("=", 1)[1].split() for line in body if re.search(r"= f(add|sub|mul) ", line)]
    assert len(ops) >= 10  # three products, seven sums
    assert all(set(op).isdisjoint({"contract", "fast", "reassoc"}) for op in ops), ops


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_flat_polynomial(tmp_path):
    """The polynomial for 2^x on [-1, 0] that the flat components share: its
    coefficients leave a relative error of 2.08e-9, without a bias that would
    add up over bins (mean below a tenth of that)."""
    exe = tmp_path / "flat_check"
    cmd = [*_shift_phase_cmd()[:-1], os.path.join(ROOT, "tests", "native", "flat_check.hip"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout.split()
    worst, mean = (float(v) for v in out)
    assert worst < 2.2e-9, worst
    assert abs(mean) < 2.1e-10, mean


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_column_split_phase(tmp_path):
    """The column phases of the adjoint from 64 up.  An error that a column's
    rows have in common moves the galaxy along x: it is that of the phase
    itself, 1.1e-8 rms at the low columns, that of tw (a float32 rounding,
    1.7e-8 rms) on the half of the sum that it multiplies, and the 64 rows' own
    roundings of 3e-8 averaged, 0.4e-8: together 1.4e-8.  Column 0, packed with
    column W / 2: four roundings."""
    exe = tmp_path / "column_split_check"
    cmd = [*_shift_phase_cmd()[:-1], os.path.join(ROOT, "tests", "native", "column_split_check.hip"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=300).stdout.splitlines()
    assert [int(line.split()[0]) for line in lines] == [64, 128, 256]
    for line in lines:
        _, rms, worst0 = line.split()
        assert float(rms) < 1.6e-8, line
        assert float(worst0) < 4 * 2.0 ** -24, line
