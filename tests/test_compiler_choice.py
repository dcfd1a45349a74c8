"""Which compiler makes a plan's code, and under which name it is cached (no GPU needed)."""
import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLAN = "b.Plan('8x0e+8x1o', '1x0e+1x1o', '8x0e+8x1o', device=-2).close()"


def compiled(cache, before, **env):
    """File name -> bytes of the code objects that a new process makes, which runs `before` first."""
    cache.mkdir()
    code = f"{before}\nfrom paper_2501_13986_amd import binding as b\n{PLAN}"
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, env={**os.environ, "CGTP_CACHE_DIR": str(cache), **env}, check=True)
    return {f.name: f.read_bytes() for f in cache.iterdir()}


def test_the_code_of_a_plan_does_not_depend_on_torch(tmp_path):
    alone, after_torch = compiled(tmp_path / "a", ""), compiled(tmp_path / "t", "import torch")
    assert alone and alone.keys() == after_torch.keys()
    assert all(alone[name] == after_torch[name] for name in alone)


def test_another_compiler_has_keys_of_its_own(tmp_path):
    """The linked compiler in a process with torch is torch's: where its code differs, so does every name."""
    own, linked = compiled(tmp_path / "o", "import torch"), compiled(tmp_path / "l", "import torch", CGTP_OWN_COMPILER="0")
    assert own and linked
    shared = own.keys() & linked.keys()
    assert all(own[name] == linked[name] for name in shared)
