"""The library's double-precision modular arithmetic, compiled for the host and checked against exact 128-bit
integer arithmetic: value congruence and the stated magnitude bounds of every primitive (lazy product,
lazy reduction, exact multiply-accumulate in doubles and in integers, splits, sixteen-point forward / inverse passes), on random
and boundary-seeking inputs, for the primes the workloads use; and both fused conversions on the tables of the built library."""

import os
import shutil
import subprocess

import pytest

import paper_2512_11269_amd as K

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_arith", "arith_selftest.hip")


def _library():
    """Linker arguments for the built library."""
    K.load_library()
    where, name = os.path.split(os.path.abspath(K.library_path()))
    return ["-L" + where, "-l:" + name, "-Wl,-rpath," + where]


def test_device_arithmetic_is_exact_on_host(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "arith_selftest")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off", SRC, "-o", exe] + _library(),
                          stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip().endswith("OK")


def test_device_arithmetic_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    """The same host build with AddressSanitizer and UBSan on the host side (the GPU side is never run)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "arith_selftest_san")
    subprocess.check_call([hipcc, "-O1", "-g", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off", "-Xarch_host",
                           "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined",
                           SRC, "-o", exe] + _library(), stderr=subprocess.DEVNULL)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("LD_PRELOAD", None)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.strip().endswith("OK") and "runtime error" not in out.stderr and "AddressSanitizer" not in out.stderr
