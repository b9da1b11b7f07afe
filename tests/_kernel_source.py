"""Builds pieces of the kernel source as host programs: device functions and
types are copied out of csrc/lsm_kernels.hip at build time and compiled with
g++ against the small stand-ins of tests/host_kernels/, so a test on the CPU
runs the kernels' own code under a sanitizer."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1707_05354_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "host_kernels")


def excerpt(patterns) -> str:
    """The definitions whose first lines match, in the order given: one line,
    or up to the closing brace in the first column; with the template line
    before it."""
    lines = open(os.path.join(CSRC, "lsm_kernels.hip")).read().splitlines()
    out = []
    for pat in patterns:
        hits = [i for i, l in enumerate(lines) if re.match(pat, l)]
        assert len(hits) == 1, "kernel source: %r matched %d lines" % (pat, len(hits))
        i = j = hits[0]
        if lines[i - 1].startswith("template <"):
            i -= 1
        if not lines[j].startswith("constexpr"):
            while lines[j] not in ("}", "};"):
                j += 1
        out.extend(lines[i:j + 1])
    return "\n".join(out) + "\n"


def run(tmp_path, program, patterns, sanitize):
    """Builds and runs tests/host_kernels/<program> with the excerpt."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    (tmp_path / "kernel_gen.inc").write_text(excerpt(patterns))
    exe = str(tmp_path / "program")
    build = subprocess.run(
        ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=" + sanitize,
         "-fno-sanitize-recover=all", "-Wno-unknown-pragmas", "-I", str(tmp_path), "-I", HERE,
         "-I", os.path.join(ROOT, "tests", "host_sanitize"), "-I", CSRC,
         os.path.join(HERE, program), "-o", exe], capture_output=True, text=True, timeout=600)
    if build.returncode != 0 and "sanitize" in build.stderr and "cannot find" in build.stderr:
        pytest.skip("sanitizer runtime not installed: " + build.stderr.strip()[:200])
    assert build.returncode == 0, build.stderr[-4000:]
    return subprocess.run([exe], capture_output=True, text=True, timeout=600,
                          env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))


def run_host_code(tmp_path, program, wrap=()):
    """Builds and runs a program over the library's host code (csrc/lsm_api.hip)
    and the stand-in runtime and launchers of tests/host_sanitize/.  wrap: the
    functions whose calls go to the program's __wrap_ functions."""
    from test_host_sanitize import extract_layout
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    san = os.path.join(ROOT, "tests", "host_sanitize")
    src = open(os.path.join(CSRC, "lsm_kernels.hip")).read()
    (tmp_path / "layout_gen.inc").write_text(extract_layout(src))
    exe = str(tmp_path / "program")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", san, "-I", str(tmp_path), "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), "-x", "c++", os.path.join(CSRC, "lsm_api.hip"),
           "-x", "none", os.path.join(san, "stand_in.cpp"), program, "-o", exe]
    build = subprocess.run(cmd + ["-Wl,--wrap=" + w for w in wrap], capture_output=True, text=True, timeout=600)
    if build.returncode != 0 and "sanitize" in build.stderr and "cannot find" in build.stderr:
        pytest.skip("sanitizer runtime not installed: " + build.stderr.strip()[:200])
    assert build.returncode == 0, build.stderr[-4000:]
    return subprocess.run([exe], capture_output=True, text=True, timeout=600)
