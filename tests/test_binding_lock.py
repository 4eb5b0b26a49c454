"""An exception that leaves a library call finds the interpreter's lock held again (no GPU)."""
import os
import subprocess
import sys
import sysconfig

import torch

from paper_2410_09687_amd import moin

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_lock_is_held_when_a_call_throws(tmp_path):
    moin.load()
    pkg, at = os.path.dirname(moin.LIB_PATH), os.path.dirname(torch.__file__)
    r = subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(at, "include"),
                        "-I" + sysconfig.get_paths()["include"], f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                        os.path.join(ROOT, "tests", "host", "binding_lock_main.cpp"), "-o", str(tmp_path / "binding_lock.so"),
                        "-L" + os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-L" + pkg, "-l:libmoin.so",
                        "-Wl,-rpath," + pkg], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    code = "import torch, binding_lock\ntry:\n    binding_lock.throwing()\nexcept Exception as e:\n    print('raised', type(e).__name__)\n"
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert r.returncode == 0 and "raised" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])
    print(r.stdout)
