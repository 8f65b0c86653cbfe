"""The binding with and without its native argument marshalling: the library loads and answers either way (no GPU)."""
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest

from paper_2302_02390_amd import binding as qb
from paper_2302_02390_amd import build as lib_build

SUFFIX = sysconfig.get_config_var("EXT_SUFFIX")
# another torch's module: whoever attaches it has not looked at its version
OTHER_TORCH = "torch_version = '0.0.0 elsewhere'\ndef attach(*args):\n    raise AssertionError('attached')\n"
PROGRAM = """
from paper_2302_02390_amd import binding as qb
assert qb.spec_version() == 3 and qb.codes_bytes(1025, 4, 1024) == 1024 and qb.meta_bytes(1025, 1024) == 16
assert qb.status_string(-1) == "invalid argument"
assert all(getattr(qb, name) is f and f.__module__ == qb.__name__ for name, f in qb._IN_PYTHON.items())
try:
    import torch
    qb.qsdp_quantize_grad(torch.zeros(64), 4, 32, 1, 0, None, None)
except TypeError as e:
    assert "contiguous" in str(e)
else:
    raise AssertionError("a tensor on the CPU was accepted")
"""


def test_the_built_tree_uses_the_native_functions():
    qb.lib()
    assert os.path.exists(lib_build.MARSHAL) and lib_build.MARSHAL.endswith(SUFFIX)
    assert all(getattr(qb, name) is not f for name, f in qb._IN_PYTHON.items())


@pytest.mark.parametrize("module", [None, ("_marshal" + SUFFIX, b"no shared object"),
                                    ("_marshal.py", OTHER_TORCH.encode()), ("_marshal.py", b"")])
def test_a_library_without_a_module_for_this_torch(tmp_path, module):
    package = tmp_path / "paper_2302_02390_amd"
    package.mkdir()
    for name in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(lib_build.HERE, name), package)
    os.symlink(os.path.join(lib_build.HERE, "libqsdp.so"), package / "libqsdp.so")
    if module is not None:
        (package / module[0]).write_bytes(module[1])
    run = subprocess.run([sys.executable, "-c", PROGRAM], cwd=tmp_path, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr


@pytest.mark.parametrize("why", ["torch", "compiler", "headers"])
def test_a_build_without_what_the_module_needs(tmp_path, monkeypatch, capsys, why):
    """The library and the bench's kernels are built all the same, and no module of an earlier build stays."""
    commands = []

    def run(cmd, **kwargs):
        if cmd[0] == "g++" and why == "compiler":
            raise FileNotFoundError("g++")
        commands.append(cmd)
        return subprocess.CompletedProcess(cmd, int(cmd[0] == "g++" and why == "headers"), "", "Python.h: no such file")

    for name, value in (("HERE", str(tmp_path)), ("OBJ", str(tmp_path / "ob")), ("LIB", str(tmp_path / "libqsdp.so")),
                        ("MARSHAL", str(tmp_path / ("_marshal" + SUFFIX))), ("_compile", lambda unit: unit[0])):
        monkeypatch.setattr(lib_build, name, value)
    monkeypatch.setattr(lib_build.subprocess, "run", run)
    if why == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    (tmp_path / ("_marshal" + SUFFIX)).write_bytes(b"")
    assert lib_build.build() == str(tmp_path / "libqsdp.so")
    assert any(lib_build.BENCH_LIB in c for c in commands) and not list(tmp_path.glob("_marshal*"))
    assert "not built" in capsys.readouterr().err


class _Argument(int):
    """A number that notices when it is asked for an address, and a tensor's stand-in that has one."""
    asked = 0

    @property
    def data_ptr(self):
        _Argument.asked += 1
        raise AttributeError("data_ptr")


class _OnDevice:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address

    def get_device(self):
        return 0


def test_the_general_launch_asks_pointers_alone_for_their_address(monkeypatch):
    qb.lib()
    calls = []
    library = type("L", (), {name: staticmethod(lambda *args: calls.append(args) or 0) for name in qb.EXPORTS})
    monkeypatch.setattr(qb, "_lib", library)
    monkeypatch.setattr(qb, "_raw_stream", lambda device: 77)
    monkeypatch.setattr(qb.torch.cuda, "current_device", lambda: 0)
    for name, (_, kinds) in qb._SIGNATURES.items():
        if kinds and kinds[-1] is qb._vp:
            pointer = [kind is qb._vp for kind in kinds[:-1]]
            for absent in (False, True):
                args = [(None if absent else _OnDevice(i)) if p else _Argument(i) for i, p in enumerate(pointer)]
                qb._IN_PYTHON["_launch"](_OnDevice(5), name, *args)
                assert calls[-1] == tuple(None if p and absent else i for i, p in enumerate(pointer)) + (77,)
    assert len(calls) > 70 and _Argument.asked == 0
