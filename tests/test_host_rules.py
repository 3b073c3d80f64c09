"""Rules of the host runtime that choose between paths (tests/sanitize/
rule_checks.cpp), built with the host sources and sanitizers, no GPU."""
import os
import subprocess

import pytest

from test_sanitizers import CLANG, CSRC, HERE, HIPCC, HOST_SOURCES, ROCM, SAN


@pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)), reason="needs hipcc and clang++")
def test_rules(tmp_path):
    from paper_1010_4135_amd import lbm3d
    if lbm3d.lbm3d_device_count() > 0:
        pytest.skip("host rules: run where no GPU is visible")
    jobs, objs = [], []
    for path in [os.path.join(CSRC, s) for s in HOST_SOURCES] + [os.path.join(HERE, "rule_checks.cpp")]:
        obj = str(tmp_path / (os.path.basename(path) + ".o"))
        cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-g"] + SAN + ["-c", path, "-o", obj]
        jobs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT))
        objs.append(obj)
    for j in jobs:
        out, _ = j.communicate()
        assert j.returncode == 0, out.decode()[-3000:]
    exe = str(tmp_path / "rule_checks")
    r = subprocess.run([CLANG] + objs + ["-fsanitize=address,undefined", "-L" + os.path.join(ROCM, "lib"), "-lamdhip64",
                                         "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    supp = tmp_path / "lsan.supp"
    supp.write_text("leak:libamdhip64\nleak:libhsa-runtime64\nleak:librocprofiler\n")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, LSAN_OPTIONS=f"suppressions={supp}"))
    assert r.returncode == 0 and "rule checks passed" in r.stdout, (r.stdout[-2000:], r.stderr[-6000:])
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr, r.stderr[-6000:]
