"""Under which compiler's name a plan's code is cached, and whose code is taken (no GPU needed)."""
import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLAN = "b.Plan('8x0e+8x1o', '1x0e+1x1o', '8x0e+8x1o', device=-2).close()"


def compiled(cache, before):
    """File name -> bytes of the code objects in the cache after a new process, which runs `before` first, has made a plan."""
    os.makedirs(cache, exist_ok=True)
    code = f"{before}\nfrom paper_2501_13986_amd import binding as b\n{PLAN}"
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, env={**os.environ, "CGTP_CACHE_DIR": str(cache)}, check=True)
    return {f: open(os.path.join(cache, f), "rb").read() for f in os.listdir(cache)}


def test_code_of_two_compilers_never_has_one_name(tmp_path):
    """A process that has imported torch compiles with torch's compiler."""
    alone, with_torch = compiled(tmp_path / "a", ""), compiled(tmp_path / "t", "import torch")
    assert alone and with_torch
    assert all(alone[name] == with_torch[name] for name in alone.keys() & with_torch.keys())


def test_code_of_the_installed_compiler_is_taken_where_it_is_cached(tmp_path):
    alone = compiled(tmp_path, "")
    assert compiled(tmp_path, "import torch") == alone
