"""What the host records for the kernels, checked without a GPU: rpod_abi.cpp and
warm_abi.cpp compiled host-only with AddressSanitizer and UndefinedBehaviorSanitizer
against the stand-ins of tests/host_records/checks.cpp. The grid of every Gram
reduction and the record of the factorisation it ends in, the bounds of the FP32
passes' 32-bit offsets, and every part of an adaptive plan's program: a stop after
the first, a middle and the last block runs exactly one finish."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_15350_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)), reason="hipcc / clang++ not installed")
def test_records(tmp_path):
    flags = ["-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g", "-Xarch_host", "-fsanitize=address",
             "-Xarch_host", "-fsanitize=undefined"]
    sources = [os.path.join(CSRC, "rpod_abi.cpp"), os.path.join(CSRC, "warm_abi.cpp"),
               os.path.join(HERE, "host_records", "checks.cpp")]
    objs = [str(tmp_path / (os.path.splitext(os.path.basename(s))[0] + ".o")) for s in sources]
    procs = [subprocess.Popen([HIPCC, *flags, "-c", s, "-o", o], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                              text=True) for s, o in zip(sources, objs)]
    for p in procs:
        out, _ = p.communicate(timeout=600)
        assert p.returncode == 0, out
    exe = str(tmp_path / "checks")
    link = subprocess.run([CLANG, "-fsanitize=address,undefined", *objs, "-o", exe], capture_output=True, text=True)
    assert link.returncode == 0, link.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600,
                         env=dict(os.environ, UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1"))
    report = run.stdout + run.stderr
    assert run.returncode == 0 and "PASSED" in run.stdout and "runtime error" not in report, report[-4000:]
    shutil.rmtree(tmp_path, ignore_errors=True)
