"""The CPU code under AddressSanitizer and UndefinedBehaviorSanitizer: the
oracle (oracle/lda_oracle.c), the host layout planner
(paper_2007_08725_amd/csrc/layout.cpp), the whole-number Q' sums shared with
the device and the host threads of the exports (csrc/readback.h) are built with
-fsanitize=address,undefined (host compilers only; no device code is involved)
and driven by tests/sanitize/*.  Any sanitizer report fails the run."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-g", "-O1"]
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")


def _run(cmd, **kw):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600, **kw)
    assert r.returncode == 0, "%s\n%s\n%s" % (" ".join(cmd), r.stdout[-3000:], r.stderr[-3000:])
    return r


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not installed")
def test_oracle_under_sanitizers(tmp_path):
    exe = str(tmp_path / "oracle_checks")
    _run(["gcc", "-std=c11", "-ffp-contract=off", *SAN, "-I", os.path.join(ROOT, "oracle"),
          os.path.join(HERE, "sanitize", "oracle_checks.c"), os.path.join(ROOT, "oracle", "lda_oracle.c"),
          "-lm", "-o", exe])
    r = _run([exe], env=ENV)
    assert "oracle checks passed" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="g++ or the HIP headers are not installed")
def test_layout_planner_under_sanitizers(tmp_path):
    exe = str(tmp_path / "layout_checks")
    csrc = os.path.join(ROOT, "paper_2007_08725_amd", "csrc")
    _run(["g++", "-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", csrc,
          os.path.join(HERE, "sanitize", "layout_checks.cpp"), os.path.join(csrc, "layout.cpp"), "-o", exe])
    r = _run([exe], env=ENV)
    assert "layout checks passed" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="g++ or the HIP headers are not installed")
def test_q_sums_do_not_depend_on_the_order(tmp_path):
    exe = str(tmp_path / "q_sum_checks")
    _run(["g++", "-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
          os.path.join(ROOT, "paper_2007_08725_amd", "csrc"), os.path.join(HERE, "sanitize", "q_sum_checks.cpp"),
          "-o", exe])
    r = _run([exe], env=ENV)
    assert "Q' sum checks passed" in r.stdout


def test_kernels_add_no_floating_point_atomics():
    """Draws and LLPT promise the same bits on every run: an atomic sum of floating-point values has the order of the
    waves' timing, so the kernels' atomics are whole numbers (their operands' types are declared in the sources)."""
    csrc = os.path.join(ROOT, "paper_2007_08725_amd", "csrc")
    for name in sorted(os.listdir(csrc)):
        if not name.endswith((".hip", ".h", ".cpp")):
            continue
        text = open(os.path.join(csrc, name)).read()
        assert "unsafeAtomicAdd" not in text and "__builtin_amdgcn_ds_atomic_fadd" not in text, name
        doubles = set(re.findall(r"\b(?:double|float)\s*\*\s*(?:__restrict__\s*)?(\w+)", text))
        for target in re.findall(r"atomicAdd\(\s*&?\s*(?:\w+(?:\.|->))*(\w+)", text):
            assert target not in doubles, "%s: atomicAdd on %s" % (name, target)


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="g++ or the HIP headers are not installed")
def test_read_back_threads_survive_failed_allocations(tmp_path):
    exe = str(tmp_path / "crew_checks")
    _run(["g++", "-std=c++17", *SAN, "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
          os.path.join(ROOT, "paper_2007_08725_amd", "csrc"), os.path.join(HERE, "sanitize", "crew_checks.cpp"),
          "-o", exe])
    r = _run([exe], env=ENV)
    assert "crew checks passed" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="g++ or the HIP headers are not installed")
def test_read_back_leaves_nothing_behind(tmp_path):
    exe = str(tmp_path / "readback_checks")
    _run(["g++", "-std=c++17", *SAN, "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
          os.path.join(ROOT, "paper_2007_08725_amd", "csrc"), os.path.join(HERE, "sanitize", "readback_checks.cpp"),
          "-o", exe])
    r = _run([exe], env=ENV)
    assert "read-back checks passed" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="g++ or the HIP headers are not installed")
def test_certified_draws_that_stand_are_the_exact_ones(tmp_path):
    exe = str(tmp_path / "certified_checks")
    _run(["g++", "-std=c++17", *SAN, "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
          os.path.join(ROOT, "paper_2007_08725_amd", "csrc"), os.path.join(HERE, "sanitize", "certified_checks.cpp"),
          "-o", exe])
    r = _run([exe], env=ENV)
    assert "certified draw checks passed" in r.stdout, r.stdout
