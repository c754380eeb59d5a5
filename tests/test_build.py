"""The package from its sources alone: nothing that is built may be needed to import what builds it."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sources(tmp_path_factory):
    root = tmp_path_factory.mktemp("sources")
    for d in ("paper_2402_03694_amd", "include"):
        shutil.copytree(os.path.join(ROOT, d), root / d, ignore=shutil.ignore_patterns("*.so", "*.so.*", "__pycache__"))
    shutil.copy(os.path.join(ROOT, "__graft_entry__.py"), root)
    return root


def _child(root, code):
    env = {k: v for k, v in os.environ.items() if k != "SERVEFLOW_LIB"}
    res = subprocess.run([sys.executable, "-c", code], cwd=root, env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    return res.stdout


def test_sources_alone_import_and_say_what_is_missing(sources):
    out = _child(sources, """
import __graft_entry__
from paper_2402_03694_amd import binding, build
assert build.is_stale()
for call in (binding.lib, binding.load_marshal):
    try:
        call()
    except (OSError, ImportError) as e:
        assert "build" in str(e), e
    else:
        raise SystemExit("loaded what is not there")
print("fine")
""")
    assert out.endswith("fine\n")


def test_tensor_check_is_built_and_bound_to_its_torch(sources):
    out = _child(sources, """
import os
import torch
from paper_2402_03694_amd import binding, build
open(build.LIB, "w").close()                  # (stands for the library)
assert build.is_stale()
path = build.build_marshal()
assert not build.is_stale() and os.listdir(build.HERE).count(os.path.basename(path)) == 1
native = binding.load_marshal()
assert native.ptr(None) is None
for form in (native.ptr, binding.check_ptr):
    try:
        form(torch.zeros(3))
    except TypeError as e:
        assert "device tensor" in str(e)
    else:
        raise SystemExit("took a tensor of the host")
torch.__version__ = "0.0"
assert build.is_stale()
print("fine")
""")
    assert out.endswith("fine\n")
