"""The library's host code around the device (assembly, products, GMRES, refinement, serving with
several workers) under AddressSanitizer + UndefinedBehaviorSanitizer and under ThreadSanitizer,
against a CPU stand-in of the HIP runtime (tests/hip_stand_in.cpp) that also checks the runtime's
rules for streams under capture.  No device calls."""
import os
import subprocess

import pytest

from paper_1807_03097_amd import workloads as W
from test_host_sanitizers import CLANGXX, DRIVER_FLAGS, HIPCC, ROOT, _write_geom

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANGXX)),
                                reason="hipcc / clang++ not available")


@pytest.mark.slow
@pytest.mark.parametrize("variant,servers", [("asan", 12), ("tsan", 6)])
def test_serving_host_code_under_sanitizers(tmp_path, variant, servers):
    from paper_1807_03097_amd import build as B
    lib = B.build(variant=variant, incremental=True)
    libdir, flags = os.path.dirname(lib), ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", *DRIVER_FLAGS[variant]]
    soname = "libamdhip64.so.7"
    stand_in, exe = str(tmp_path / soname), str(tmp_path / "serve_driver")
    inc = os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include")
    for cmd in ([CLANGXX, *flags, "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", f"-I{inc}", f"-Wl,-soname,{soname}", "-o", stand_in,
                 os.path.join(ROOT, "tests", "hip_stand_in.cpp")],
                [CLANGXX, *flags, "-o", exe, os.path.join(ROOT, "tests", "serve_driver.cpp"), f"-L{libdir}",
                 f"-l:libigaefie_{variant}.so", f"-Wl,-rpath,{libdir}", stand_in, "-lpthread"]):
        cp = subprocess.run(cmd, capture_output=True, text=True)
        assert cp.returncode == 0, cp.stderr[-3000:]
    env = dict(os.environ, LD_LIBRARY_PATH=str(tmp_path), ASAN_OPTIONS="detect_leaks=1:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1", TSAN_OPTIONS="halt_on_error=1:second_deadlock_stack=1")
    gpath = str(tmp_path / "sphere.geom")
    _write_geom(gpath, W.cube_sphere())
    r = subprocess.run([exe, gpath, str(servers)], env=env, capture_output=True, text=True, timeout=900)
    out = r.stdout + r.stderr
    print(out[-3000:])
    assert r.returncode == 0, out[-3000:]
    assert "all done" in out
    assert " 0 operations on the legacy stream, 0 blocking streams captured, 0 allocations left" in out
    for bad in ("ERROR: AddressSanitizer", "runtime error:", "WARNING: ThreadSanitizer", "ERROR: LeakSanitizer", "stand-in: legacy"):
        assert bad not in out
