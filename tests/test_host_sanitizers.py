"""The library's host code under AddressSanitizer and UndefinedBehaviorSanitizer: the packer (Alg. 1 and
the other grouping arms), the partition search and re-computation plan, the GEMM plans and buffer layouts, and the validation half of the
device entry points are compiled with g++ -fsanitize=address,undefined against stub launchers that
abort, and a driver walks them (tests/host_sanitize/).  Host only: no GPU code is built or run."""
import os
import shutil
import subprocess

import pytest

import paper_2407_20761_amd as ob

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_20761_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "host_sanitize")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the ROCm headers")
def test_host_code_is_clean_under_asan_and_ubsan(tmp_path):
    exe = str(tmp_path / "host_sanitize")
    srcs = [os.path.join(HERE, "driver.cpp"), os.path.join(HERE, "stubs.cpp")] + \
           [os.path.join(CSRC, f) for f in ("packer.cpp", "planner.cpp", "gemm_plan.cpp", "attention_plan.cpp", "api.cpp", "connector_api.cpp")]
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *srcs, "-L/opt/rocm/lib", "-lamdhip64",
           "-Wl,-rpath,/opt/rocm/lib", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "all checks passed" in r.stdout
    # the build under the sanitizers lays its buffers out as the shipped library does
    sizes = [line.split() for line in r.stdout.splitlines() if line.startswith(("block", "connector"))]
    assert len(sizes) == 37
    for kind, *v in sizes:
        v = [int(t) for t in v]
        if kind == "block":
            desc = ob.ob_block_desc(*v[:5], ob.OB_LAYERNORM, ob.OB_GELU, ob.OB_MASK_SEG_CAUSAL, ob.OB_BF16, 0, 1e4, 1e-5, 1)
            want = [ob.ob_block_saved_bytes(desc, v[5]), ob.ob_block_workspace_bytes(desc, v[5])]
        else:
            desc = ob.make_connector_desc(v[0], 4096, 32, 1e-5)
            want = [ob.ob_connector_saved_bytes(desc, v[1]), ob.ob_connector_workspace_bytes(desc, v[1])]
        assert v[-2:] == want, (kind, v)
