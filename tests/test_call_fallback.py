"""The binding without its native caller (CPU only): it builds, loads and
calls through ctypes where the module cannot be compiled or imported."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2608_12123_amd import build
from paper_2608_12123_amd import rc_cohort as rc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# In a child process: the state of the parent's binding stays as it is.
CHILD = """
import sys
{block}
from paper_2608_12123_amd import rc_cohort as rc
assert rc.rc_status_string(0) == "RC_OK"
assert (rc._call is None) == {none}
b = rc.RcBuffers()
assert rc.rc_cohort_run_chain(None, b, -1, 1, 0, 0, 1, stream=0, check=False) == rc.RC_E_INVALID
assert rc.rc_cohort_run_chain_noalloc(None, b, 1 << 32, 1, 0, 0, 1, stream=0, check=False) == rc.RC_E_INVALID
try:
    rc.rc_cohort_run_chain(None, b, 0, 1, 0, 0, 1, stream=0)
    raise SystemExit("accepted")
except rc.RcError:
    pass
"""


@pytest.mark.parametrize("block,none", [("", False), ("sys.modules['paper_2608_12123_amd._rc_call'] = None", True)])
def test_loads_without_the_native_caller(block, none):
    res = subprocess.run([sys.executable, "-c", CHILD.format(block=block, none=none)], cwd=ROOT,
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr


def test_host_only_library_keeps_its_error(tmp_path, monkeypatch):
    """A library without the chain entry points: the call says so."""
    class HostOnly:
        def __getattr__(self, name):
            raise AttributeError(name)
    monkeypatch.setattr(rc, "_lib", HostOnly())
    monkeypatch.setattr(rc, "_call", None)
    with pytest.raises(AttributeError):
        rc.rc_cohort_run_chain(None, rc.RcBuffers(), 0, 1, 0, 0, 1, stream=0)


def test_module_is_named_for_the_interpreter():
    assert os.path.basename(build.CALL_LIB) == "_rc_call" + sysconfig.get_config_var("EXT_SUFFIX")


@pytest.mark.parametrize("compiler", ["missing", "failing"])
def test_build_goes_on_without_a_compiler(tmp_path, monkeypatch, compiler):
    cc = str(tmp_path / "cc")
    if compiler == "failing":
        with open(cc, "w") as f:
            f.write("#!/bin/sh\nexit 1\n")
        os.chmod(cc, 0o755)
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setattr(build, "CALL_LIB", str(tmp_path / "_rc_call.test.so"))
    monkeypatch.setattr(build.shutil, "which", lambda name: cc if name == "cc" else None)
    monkeypatch.setattr(build, "hipcc", lambda: cc)
    (tmp_path / "_rc_call.so").write_bytes(b"of other sources")
    with pytest.warns(UserWarning, match="ctypes"):
        assert build.build_call() is None
    assert not [f for f in os.listdir(tmp_path) if f.startswith("_rc_call")]
