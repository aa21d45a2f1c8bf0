"""Addresses of tensors for the C entry points (csrc/marshal.cpp): the Python rule holds for whatever is not plainly a device
tensor, errors included.  CPU only (device tensors go through it in every GPU test)."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2210_05064_amd import binding as ver


class Like:
    def __init__(self, p, cuda=True, contiguous=True):
        self.p, self.is_cuda, self.c = p, cuda, contiguous

    def is_contiguous(self):
        return self.c

    def data_ptr(self):
        return self.p


class Sub(torch.Tensor):
    is_cuda = True

    def data_ptr(self):
        return 2 ** 63 + 5


@pytest.mark.parametrize("take", [ver._ptr, lambda t: ver._ptr_array([t])[0], lambda t: ver.pack_args(obs=t).obs])
def test_addresses(take):
    assert take(None) is None
    assert take(Sub()) == 2 ** 63 + 5
    for bad in (torch.zeros(4), torch.zeros(4, 4).t()):
        with pytest.raises(AssertionError, match="device, contiguous tensors only"):
            take(bad)


def test_look_alikes_and_other_objects():
    assert ver._ptr(Like(77)) == 77
    assert list(ver._ptr_array((Like(1), None, Like(2 ** 64 - 1)))) == [1, None, 2 ** 64 - 1]
    for bad in (Like(1, cuda=False), Like(1, contiguous=False)):
        with pytest.raises(AssertionError):
            ver._ptr(bad)
    with pytest.raises(AttributeError):
        ver._ptr(3)


def test_a_list_that_changes_meanwhile():
    """The addresses are those of the list as it was handed over: an object that lengthens it adds nothing to the buffer."""
    class Grows(Like):
        def data_ptr(self):
            tensors.append(Like(99))
            return self.p
    tensors = [Grows(5)]
    buf = (C.c_void_p * 8)()
    ver._marshal.fill(buf, tensors)
    assert list(buf) == [5] + [None] * 7


def test_pack_args_fields():
    a = ver.pack_args(N=3, S=7, obs=None, h0=Sub(), D=4, workspace=None)
    assert (a.N, a.S, a.D, a.obs, a.h0, a.workspace, a.workspace_bytes) == (3, 7, 4, None, 2 ** 63 + 5, None, 0)
    assert ver.pack_args(obs=1234).obs == 1234
    with pytest.raises(TypeError, match="unknown ver_pack_args field nonsense"):
        ver.pack_args(N=1, nonsense=Sub())
    with pytest.raises(ValueError):
        ver._marshal.fill((C.c_void_p * 1)(), [None, None])


@pytest.mark.parametrize("elsewhere", [True, False])
def test_sources_that_were_not_built(tmp_path, elsewhere):
    """Without _marshal.so: a library built elsewhere (VER_LIB) is enough; else the error says what to run."""
    package = tmp_path / "paper_2210_05064_amd"
    package.mkdir()
    for f in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(os.path.dirname(ver.__file__), f), package)
    if not elsewhere:
        os.symlink(ver.LIB_PATH, package / "libver.so")
    env = {k: v for k, v in os.environ.items() if k != "VER_LIB"}
    if elsewhere:
        env["VER_LIB"] = ver.LIB_PATH
    code = """if True:
        from paper_2210_05064_amd import binding as ver
        class T:
            is_cuda = True
            is_contiguous = lambda self: True
            data_ptr = lambda self: 77
        a = ver.pack_args(N=3, rnn_h=None, workspace=None)
        assert ver._ptr(T()) == 77 and list(ver._ptr_array([T(), None])) == [77, None] and (a.N, a.rnn_h, a.workspace) == (3, None, None)
    """
    run = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env=env, capture_output=True, text=True)
    if elsewhere:
        assert run.returncode == 0, run.stderr
    else:
        assert "ImportError" in run.stderr and "_marshal.so is missing: run `python -m" in run.stderr, run.stderr
