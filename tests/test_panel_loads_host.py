"""The device's panel loads (tile_f32.h, tile_bf16.h, tile_bytes.h, common.h) compiled
for the CPU and run under AddressSanitizer and UndefinedBehaviorSanitizer: no read
leaves the stored matrix, and every element arrives, with zeros beyond K."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_panel_loads_on_the_cpu(tmp_path):
    from paper_2305_18236_amd import build
    cc = build.hipcc()
    clangxx = os.path.join(os.path.dirname(cc), "..", "llvm", "bin", "clang++")
    if not os.path.exists(clangxx):
        pytest.skip("no clang++")
    obj, exe = str(tmp_path / "panel.o"), str(tmp_path / "panel")
    subprocess.run([cc, f"--offload-arch={build.ARCH}", "--offload-host-only", "-O1", "-g", "-std=c++17",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=undefined",
                    "-DMG_DEVICE=__host__ __device__ inline", "-I" + build.CSRC, "-c",
                    os.path.join(ROOT, "tests", "sanitize", "panel_driver.hip"), "-o", obj], check=True)
    lib = os.path.join(os.path.dirname(os.path.dirname(cc)), "lib")
    subprocess.run([clangxx, "-fsanitize=address,undefined", obj, "-o", exe, "-L" + lib, "-lamdhip64",
                    "-Wl,-rpath," + lib], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], env=env, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
