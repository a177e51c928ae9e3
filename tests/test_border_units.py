"""The units of the adjoint's mirror pass, run on the host with the kernel's
own index code under AddressSanitizer: every pixel that padding folds onto
once, in every channel.  No GPU is needed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang")
def test_units_visit_every_folded_pixel_once(tmp_path):
    exe = str(tmp_path / "border")
    subprocess.check_call([CLANG, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-std=c++17", "-O2", "-g",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wno-unused-result",
                           "-I", os.path.join(ROOT, "paper_2511_04261_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "border_driver.cpp"), "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.stdout + r.stderr)[-4000:]
