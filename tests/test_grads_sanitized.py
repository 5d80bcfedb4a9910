"""The host code of the training pass under AddressSanitizer and
UndefinedBehaviorSanitizer (no GPU needed): its source is compiled for the host
only and driven by tests/sanitize_grads_main.c along its argument checks and
over every size of its scratch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang"


@pytest.mark.skipif(shutil.which("hipcc") is None or not os.path.exists(CLANG), reason="ROCm compilers not available")
def test_training_pass_host_code_is_clean(tmp_path):
    san = ["-Xarch_host", "-fsanitize=address,undefined", "-Xarch_host", "-fno-sanitize-recover=all"]
    obj, drv, exe = (str(tmp_path / n) for n in ("train.o", "drv.o", "grads_sanitized"))
    r = subprocess.run(["hipcc", "--cuda-host-only", "-fgpu-rdc", "-O1", "-g", "-std=c++17", "-fPIC", *san, "-c",
                        os.path.join(ROOT, "paper_1408_3526_amd", "csrc", "rmdf_mlp_train.hip"), "-o", obj],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    subprocess.check_call([CLANG, "-std=c99", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "include"), "-c",
                           os.path.join(ROOT, "tests", "sanitize_grads_main.c"), "-o", drv])
    r = subprocess.run(["hipcc", "-fgpu-rdc", "--offload-arch=gfx950", *san, obj, drv, "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, (r.stdout[-3000:], r.stderr[-4000:])
    assert "sanitized grads ok" in r.stdout, r.stdout[-3000:]
    assert "runtime error" not in r.stderr
