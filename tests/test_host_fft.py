"""The transforms of csrc/fft.hpp compiled for the CPU: lanes in lockstep from
fence to fence, so that what the result owes to the hardware's order of issue
shows as a wrong value."""
import shutil
import subprocess
from pathlib import Path

import pytest

HERE = Path(__file__).resolve().parent
CSRC = HERE.parent / "paper_2304_03306_amd" / "csrc"


def _run(tmp_path, name, flags=("-ffp-contract=off",)):
    cxx = shutil.which("g++")
    assert cxx, "g++ is needed"
    exe = tmp_path / name
    r = subprocess.run([cxx, "-std=c++17", "-O2", *flags, "-w", f"-I{HERE / 'host'}", f"-I{CSRC}",
                        str(HERE / "host" / f"{name}.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return [line.split() for line in r.stdout.splitlines()]


def test_every_exchange_is_fenced(tmp_path):
    """1 to 3 transforms per thread, one-wavefront and larger workgroups, both
    lane orders: FP64 results within 1e-14 of the largest output (64 to 1024
    terms of unit size, about 10 roundings each)."""
    lines = _run(tmp_path, "fft_order")
    assert len(lines) == 10 * 10
    bad = [" ".join(f) for f in lines if not float(f[-1]) < 1e-14]
    assert not bad, "\n".join(bad)


def test_error_is_no_larger_than_the_textbook_stages(tmp_path):
    """RMS error against long double of every length, both directions and types,
    against stages of products (with factors rounded once) followed by the
    untwiddled DFT (about 4.5 against 4.75 roundings of the output's size squared
    per radix-8 stage); contracted to fused multiply-adds as on the GPU where
    this CPU has them."""
    fused = ("-mfma", "-ffp-contract=fast") if " fma " in Path("/proc/cpuinfo").read_text() else ()
    lines = _run(tmp_path, "fft_error", fused)
    assert len(lines) == 36
    bad = [" ".join(f) for f in lines if not 0.0 < float(f[4]) <= float(f[5])]
    assert not bad, "\n".join(bad)
