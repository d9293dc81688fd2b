"""The pressure sums of the kernels with several lanes per particle, built for the
host with AddressSanitizer and UndefinedBehaviorSanitizer, against the equations
written out in long double: every split, normal mode and list source.  No GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_group_sums_on_the_host(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = tmp_path / "host_group_sums"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none", "-Wl,--defsym=__hip_fatbin=0",
                    "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    os.path.join(ROOT, "tests", "host_group_sums.cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert res.stdout.startswith("ok 36000"), res.stdout
