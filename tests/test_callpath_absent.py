"""The binding without its native call path: it loads, says so once, and every call goes through Python."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

import pytest
import torch

from paper_2412_21124_amd import binding as B
from paper_2412_21124_amd import build as nt_build

CLIENT = """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2412_21124_amd import binding as B
    assert B.normtest_tile_coords(4) == 16384
    B.lib()
print(B.__file__)
print(sum("marshalled in Python" in str(w.message) for w in seen))
assert B._fast is None
import torch
g, v, b = torch.zeros(3, 64), torch.zeros(64), torch.zeros(B.RESULT_BYTES, dtype=torch.uint8)
for call in (lambda: B.normtest_step(g, v, v, v, B.make_hyper(), workspace=b, result=b), lambda: B.normtest_adamw_gbar(v, v, v, v, B.make_hyper())):
    try:
        call()
    except ValueError as e:
        assert "no CPU path" in str(e)
    else:
        raise AssertionError("accepted")
"""


def _client(root):
    """The client's lines, run on the package in `root` where no compiler is found."""
    env = dict(os.environ, PATH=str(root / "nowhere"), PYTHONPATH=str(root))
    done = subprocess.run([sys.executable, "-c", CLIENT], cwd=root, env=env, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return done.stdout.splitlines()


@pytest.mark.parametrize("there", ["nothing", "no module", "another torch's"])
def test_loads_without(tmp_path, there):
    B.lib()   # built
    package = tmp_path / "paper_2412_21124_amd"
    shutil.copytree(os.path.dirname(nt_build.LIB), package, ignore=shutil.ignore_patterns("_callpath*", "__pycache__"))
    shutil.copytree(nt_build.INCLUDE, tmp_path / "include")
    if there == "no module":
        (package / os.path.basename(nt_build.callpath_file())).write_bytes(b"not a shared object")
    elif there == "another torch's":   # as it was named before, and for another version: neither is looked at
        for name in ("_callpath.so", "_callpath.torch-0.0.0.so"):
            shutil.copy(nt_build.callpath_file(), package / name)
    where, warned = _client(tmp_path)
    assert where.startswith(str(tmp_path)) and warned == "1"


# what fails while it is made ready is not used either: a call may only see a module whose init() has returned
def test_half_loaded_module_is_not_used(tmp_path, monkeypatch):
    B.lib()
    seen = tmp_path / "callpath.py"
    seen.write_text("def init(*a):\n    raise RuntimeError('not today')\n")
    monkeypatch.setattr(nt_build, "ensure_callpath", lambda: str(seen))
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_fast", None)
    with pytest.warns(RuntimeWarning, match="not today"):
        B.lib()
    assert B._fast is None and B.normtest_tile_coords(4) == 16384


# and one that can be loaded is, under a name that no other Python or torch takes
def test_loaded_module_is_this_builds():
    B.lib()
    name = os.path.basename(B._fast.__file__)
    assert torch.__version__ in name and name.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
