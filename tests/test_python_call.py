"""The direct way from Python into the calls made once per step (csrc/zi_python.c): which forms of arguments it takes,
and that it refuses what the general way refuses, with the same words (no GPU: every call here ends in the library's
argument checks)."""
import ctypes
import importlib.machinery
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi
from paper_2104_07857_amd import binding
from paper_2104_07857_amd import build as zb

OUT, WS = torch.zeros(4, dtype=torch.float64), torch.zeros(262144, dtype=torch.uint8)


@pytest.fixture(scope="module")
def calls():
    if not zb.call_can_be_built():
        pytest.skip("no Python.h or no gcc: every call goes through ctypes")
    binding.lib()
    assert binding._call_step is not binding._not_taken, zb.CALL_PATH + " is not built"
    return binding._call_norm, binding._call_norm_noalloc, binding._call_step


def _list(n=8):
    x = [torch.zeros(n) for _ in range(3)]
    return zi.make_tensors([(x[0], x[1], x[2], torch.zeros(n, dtype=torch.bfloat16), None, n)])


class _Stream:
    cuda_stream = 0


class _Raises:
    def data_ptr(self):
        raise RuntimeError("no")


def test_module_is_named_for_this_interpreter(calls):
    """Another Python finds neither this file nor one without a version in its name."""
    from paper_2104_07857_amd import _zi_call
    assert os.path.samefile(_zi_call.__file__, zb.CALL_PATH)
    assert zb.CALL_PATH.endswith(importlib.machinery.EXTENSION_SUFFIXES[0]) and importlib.machinery.EXTENSION_SUFFIXES[0] != ".so"
    assert not os.path.exists(os.path.join(zb.HERE, "_zi_call.so"))


@pytest.mark.parametrize("why", ["no headers", "no compiler", "compiler fails", "compiler vanishes"])
def test_build_goes_on_without_the_module(why, tmp_path, monkeypatch, capsys):
    """Without the module every call goes through ctypes: one that cannot be built is reported, an older one goes away."""
    here, old = tmp_path / ("_zi_call" + importlib.machinery.EXTENSION_SUFFIXES[0]), tmp_path / "_zi_call.so"
    here.write_bytes(b"old")
    old.write_bytes(b"old")
    monkeypatch.setattr(zb, "HERE", str(tmp_path))
    monkeypatch.setattr(zb, "CALL_PATH", str(here))

    def run(*args, **kwargs):
        assert why.startswith("compiler")
        if why == "compiler vanishes":
            raise FileNotFoundError("gcc")
        return subprocess.CompletedProcess(args, 1, "", "no such luck")

    monkeypatch.setattr(zb.subprocess, "run", run)
    monkeypatch.setattr(zb, "has_python_headers", lambda: why != "no headers")
    monkeypatch.setattr(zb.shutil, "which", lambda name: None if why == "no compiler" else "/usr/bin/" + name)
    assert zb.build_call() is None
    assert "ctypes" in capsys.readouterr().err and not here.exists() and not old.exists()


def test_usual_forms_are_taken(calls):
    norm, noalloc, step = calls
    tl, cfg = _list(), zi.make_config()
    for out in (OUT, OUT.data_ptr(), None):
        for stream in (None, 0, _Stream()):
            # (dtype 7 does not exist: the library answers before it touches anything)
            assert norm(tl, 7, 1.0, out, WS, None, stream) == zi.ZI_ERR_INVALID_ARG
            assert norm(tl, 7, 1.0, out, WS.data_ptr(), 262144, stream) == zi.ZI_ERR_INVALID_ARG
            assert step(tl, 7, cfg, out, stream) == zi.ZI_ERR_INVALID_ARG
    assert norm(tl, 7, 1.0, OUT, WS, None, None) < 0 and "dtype 7" in zi.zi_last_error()
    assert step(tl, 0, zi.make_config(step=0), None, None) < 0 and "step" in zi.zi_last_error()
    many = zi.make_tensors([(a, a, a, a, None, 5) for a in (4096, 8192)])
    assert step(many, 0, cfg, None, None) < 0 and "tensor 0: p and m overlap" in zi.zi_last_error()
    del noalloc


@pytest.mark.parametrize("change", [
    dict(tensors=[(4096, 8192, 12288, 16384, None, 8)]), dict(tensors=(3, 4)), dict(tensors=((zi.zi_file_tensor * 2)(), 2)),
    dict(tensors=((zi.zi_adamw_config * 2)(), 2)), dict(tensors=(zi.zi_tensor(), 1)), dict(dt=np.int32(0)), dict(dt=0.0), dict(dt=1 << 40),
    dict(cfg=None), dict(cfg=zi.zi_tensor()), dict(norm=_Raises()), dict(norm="x"), dict(norm=-1), dict(stream="x"), dict(norm=np.zeros(4))])
def test_other_forms_go_the_general_way(calls, change):
    a = dict(tensors=_list(), dt=0, cfg=zi.make_config(), norm=None, stream=None)
    a.update(change)
    assert calls[2](a["tensors"], a["dt"], a["cfg"], a["norm"], a["stream"]) is None
    if "cfg" not in change:
        assert calls[0](a["tensors"], a["dt"], 1.0, OUT if a["norm"] is None else a["norm"], WS, None, a["stream"]) is None
        assert calls[1](a["tensors"], a["dt"], 1.0, OUT if a["norm"] is None else a["norm"], a["stream"]) is None
    assert calls[0](_list(), 0, 1, OUT, WS, None, None) is None and calls[0](_list(), 0, 1.0, OUT, 4096, None, None) is None


@pytest.mark.parametrize("call", [
    lambda: zi.zi_adamw_step(_list(), 9, zi.make_config()),
    lambda: zi.zi_adamw_step(_list(), 0, zi.make_config(beta1=1.0)),
    lambda: zi.zi_adamw_step(_list(), 0, None),
    lambda: zi.zi_adamw_step(_list(), 0, zi.make_config(), 12),
    lambda: zi.zi_adamw_step(((zi.zi_adamw_config * 2)(), 2), 0, zi.make_config()),
    lambda: zi.zi_adamw_step(_list(), 0, zi.make_config(), "norm"),
    lambda: zi.zi_grad_norm(_list(), 0, -1.0, OUT, WS),
    lambda: zi.zi_grad_norm(_list(), 0, 1.0, None, WS),
    lambda: zi.zi_grad_norm(_list(), 0, 1.0, OUT, WS[:100]),
    lambda: zi.zi_grad_norm(_list(), 0, 1.0, OUT, np.zeros(4)),
    lambda: zi.zi_grad_norm(_list(), 0, 1.0, OUT, None),
    lambda: zi.zi_grad_norm(_list(), 0, "1", OUT, WS)])
def test_what_is_refused_stays_refused(calls, call, monkeypatch):
    def raised():
        try:
            call()
        except Exception as e:                                                            # noqa: BLE001
            return type(e), str(e)
        return None

    direct = raised()
    for name in ("_call_norm", "_call_norm_noalloc", "_call_step"):
        monkeypatch.setattr(binding, name, binding._not_taken)
    assert direct is not None and direct == raised()


def test_nothing_is_kept(calls):
    tl, cfg, out = _list(), zi.make_config(), torch.zeros(4, dtype=torch.float64)
    before = [sys.getrefcount(x) for x in (tl, tl[0], cfg, out, WS)]
    for _ in range(100):
        calls[0](tl, 7, 1.0, out, WS, None, None)
        calls[2](tl, 7, cfg, out, None)
        calls[2](tl, 7, None, out, None)
    assert [sys.getrefcount(x) for x in (tl, tl[0], cfg, out, WS)] == before
    ctypes.resize(cfg, ctypes.sizeof(cfg))            # a buffer still held would refuse this
