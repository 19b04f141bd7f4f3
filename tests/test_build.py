"""CPU: the C library builds without torch; only the host module of the Python package needs it."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCRIPT = """
import importlib.util, sys, types
class NoTorch:                                   # torch can be neither imported nor found
    def find_spec(self, name, path=None, target=None):
        if name.split(".")[0] == "torch":
            raise ModuleNotFoundError(name)
sys.meta_path.insert(0, NoTorch())
spec = importlib.util.spec_from_file_location("build", %r)
b = importlib.util.module_from_spec(spec)
spec.loader.exec_module(b)
ran, done = [], types.SimpleNamespace(returncode=0, stdout="", stderr="")
b.subprocess.run = lambda cmd, **kw: ran.append(cmd) or done
b.os.replace = b.os.makedirs = lambda *a, **kw: None
b.build(host=False)
tools = {c[0].rsplit("/", 1)[-1] for c in ran}
assert tools == {"hipcc"} and len(ran) == len(b.sources()) + 1, (tools, len(ran))
assert not any("torch" in a for c in ran for a in c)
print("alone ok")
"""


def test_the_library_needs_no_torch():
    script = SCRIPT % os.path.join(ROOT, "paper_2201_13195_amd", "build.py")
    p = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True)
    assert p.returncode == 0 and "alone ok" in p.stdout, p.stderr
