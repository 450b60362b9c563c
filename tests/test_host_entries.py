"""Index arithmetic and planning rules of the HIP library near 2^31 nonzeros
(CPU only): tests/sanitize/host_entries.cpp is built by hipcc with the
sanitizers on its host code and makes no GPU call."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_10722_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LINKED = ["pmp_binned.hip", "pmp_binned_plan.hip", "pmp_adjoint.hip", "pmp_prune.hip", "pmp_batch.hip",
          "pmp_api.hip"]   # pmp_kernels.hip is included by the program


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_host_entries_under_sanitizers(tmp_path):
    exe = str(tmp_path / "entries_asan")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17",
                        "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                        "-Xarch_host", "-fno-sanitize-recover=all",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip",
                        os.path.join(ROOT, "tests", "sanitize", "host_entries.cpp"),
                        *[os.path.join(CSRC, f) for f in LINKED], "-o", exe],
                       capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout[-4000:] + r.stderr[-4000:]
    assert "runtime error" not in r.stderr
