"""The build steps on a host (nothing is compiled: the commands are recorded)."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORD = """
import concurrent.futures, importlib.util, os, sys, types
if {absent}:
    sys.modules["torch"] = None                 # import torch raises ImportError
spec = importlib.util.spec_from_file_location("b", {path!r})
b = importlib.util.module_from_spec(spec)
spec.loader.exec_module(b)
ran, moved = [], []
def run(cmd):
    if {broken} and any("torch_bind" in x for x in cmd):
        raise RuntimeError("binding")
    ran.append(cmd)
    return types.SimpleNamespace(stdout="", stderr="")
b._run, b.BUILD, b.hipcc = run, {tmp!r}, lambda: "hipcc"
b.os = types.SimpleNamespace(**{{k: getattr(os, k) for k in ("path", "makedirs", "environ")}}, replace=lambda a, c: moved.append(c))
try:
    b.build()
except RuntimeError as e:
    print("failed:", e)
print("compiled:", sum("-c" in c for c in ran), "library:", b.LIB in moved, "binding:", b.BIND in moved)
"""


@pytest.mark.parametrize("absent,broken,said", [
    (True, False, "compiled: 12 library: True binding: False"),
    (False, False, "compiled: 13 library: True binding: True"),
    (False, True, "failed: binding\ncompiled: 12 library: True binding: False"),     # (a torch whose headers do not fit)
])
def test_the_library_is_built_without_torch(tmp_path, absent, broken, said):
    """libspecfp8.so is a plain C ABI: torch is needed for the binding only."""
    code = RECORD.format(absent=absent, broken=broken, tmp=str(tmp_path),
                         path=os.path.join(ROOT, "paper_2606_18502_amd", "build.py"))
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    assert res.stdout.strip() == said
