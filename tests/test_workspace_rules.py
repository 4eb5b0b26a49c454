"""The host rules that size the workspace for batches smaller than the call's own, over every number of tokens (no GPU)."""
import os
import subprocess

import pytest

from paper_2410_09687_amd import moin

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "include", "hip")), reason="no HIP headers")
def test_no_smaller_batch_asks_for_more_rows_than_reported(tmp_path):
    moin.load()
    exe, pkg = str(tmp_path / "rows"), os.path.dirname(moin.LIB_PATH)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                        os.path.join(ROOT, "tests", "host", "workspace_rows_main.cpp"), "-L" + pkg, "-l:libmoin.so",
                        "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", f"-Wl,-rpath,{pkg}:{os.path.join(ROCM, 'lib')}", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "workspace rows agree" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
