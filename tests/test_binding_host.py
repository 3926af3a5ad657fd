"""The binding's gathering of tensor lists: the compiled one, the one in Python that stands in for it, and which of
them a process gets."""
import importlib
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2509_04084_amd import _build
from paper_2509_04084_amd import lowdiff as ld

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ld.load()
GATHERS = [pytest.param(ld._gather, id="loaded"), pytest.param(ld._gather_tensors, id="python")]


def unpack(answer):
    ptr, sizes, device, bad = answer
    return np.frombuffer(ptr, np.uint64).tolist(), np.frombuffer(sizes, np.int64).tolist(), device, bad


def test_the_compiled_gather_is_the_one_in_use():
    assert ld._gather is not ld._gather_tensors
    assert ld._gather.__module__ is None or "marshal" in str(ld._gather.__module__)


@pytest.mark.parametrize("gather", GATHERS)
def test_gather_of_host_tensors(gather):
    i32 = [torch.zeros(n, dtype=torch.int32) for n in (4, 0, 7)]
    # pageable host memory fits neither a device list nor a page-locked one
    for pinned in (False, True):
        assert unpack(gather(i32, torch.int32, pinned)) == ([0, 0, 0], [4, 0, 7], -1, 0)
    assert unpack(gather([], torch.int32, False)) == ([], [], -2, -1)
    assert unpack(gather((), torch.int32, True)) == ([], [], -2, -1)
    assert unpack(gather(tuple(i32), torch.int32, False)) == unpack(gather(i32, torch.int32, False))
    stack = torch.zeros(3, 5, dtype=torch.int32)       # any sequence of tensors
    assert unpack(gather(stack, torch.int32, False))[1] == [5, 5, 5]
    for wrong in ([i32[0], None], [np.zeros(3)], 7):
        with pytest.raises(TypeError):
            gather(wrong, torch.int32, False)
    with pytest.raises(TypeError):
        gather(i32, "int32", False)


@pytest.mark.gpu
@pytest.mark.parametrize("gather", GATHERS)
def test_gather_of_device_and_page_locked_tensors(gather):
    dev = "cuda:0"
    a = [torch.zeros(n, dtype=torch.bfloat16, device=dev) for n in (8, 0, 3)]
    assert unpack(gather(a, torch.bfloat16, False)) == ([t.data_ptr() for t in a], [8, 0, 3], 0, -1)
    view = a[0][3:]                                     # contiguous, at an offset
    strided = a[0][::2]
    assert unpack(gather([view, strided, a[2]], torch.bfloat16, False)) == (
        [view.data_ptr(), 0, a[2].data_ptr()], [5, 4, 3], 0, 1)
    other = torch.zeros(5, device=dev)                  # a wrong type in the middle: the first one is told
    assert unpack(gather([a[0], other, strided], torch.bfloat16, False)) == ([a[0].data_ptr(), 0, 0], [8, 5, 4], 0, 1)
    locked, paged = torch.zeros(6, dtype=torch.bfloat16).pin_memory(), torch.zeros(6, dtype=torch.bfloat16)
    assert unpack(gather([locked, locked], torch.bfloat16, True)) == ([locked.data_ptr()] * 2, [6, 6], -1, -1)
    assert unpack(gather([locked], torch.bfloat16, False)) == ([0], [6], -1, 0)
    assert unpack(gather([a[0], locked, paged], torch.bfloat16, True)) == (
        [a[0].data_ptr(), locked.data_ptr(), 0], [8, 6, 6], -2, 2)


@pytest.mark.gpu
@pytest.mark.parametrize("gather", GATHERS)
def test_entry_points_refuse_what_gather_reports(gather, monkeypatch):
    monkeypatch.setattr(ld, "_gather", gather)
    dev = "cuda:0"
    bf = lambda n, **kw: torch.zeros(n, dtype=torch.bfloat16, **kw)
    src = [bf(8, device=dev), bf(3, device=dev)]
    ld.ld_snapshot_layers(src, [bf(8, device=dev), bf(3).pin_memory()])      # both kinds of destination in one call
    torch.cuda.synchronize()
    with pytest.raises(TypeError, match="pinned"):
        ld.ld_snapshot_layers(src, [bf(8, device=dev), bf(3)])
    with pytest.raises(TypeError, match="src"):
        ld.ld_snapshot_layers([src[0], bf(3).pin_memory()], [bf(8, device=dev), bf(3, device=dev)])
    with pytest.raises(ValueError, match="differ in size"):
        ld.ld_snapshot_layers(src, [bf(8, device=dev), bf(4, device=dev)])
    w = torch.zeros(64, device=dev)
    i, v = torch.zeros(1, dtype=torch.int32, device=dev), torch.zeros(1, device=dev)
    with pytest.raises(ValueError, match="different devices"):
        ld.ld_merge_sparse(w, [i, i.cpu()], [v, v], 0.1)
    with pytest.raises(TypeError, match="val"):
        ld.ld_merge_sparse(w, [i, i], [v, v.double()], 0.1)
    ld.ld_merge_sparse(w, [], [], 0.1)


def test_gather_is_built_once_more_and_done_without(monkeypatch):
    builds = []

    def fails(name, package=None):
        raise ImportError("built for another torch")

    real = importlib.import_module
    monkeypatch.setattr(ld.importlib, "import_module", fails)
    monkeypatch.setattr(_build, "build_marshal", lambda force=True: builds.append(force))
    assert ld._load_gather() is ld._gather_tensors and builds == [True]

    def no_compiler(force=True):
        builds.append(force)
        raise RuntimeError("g++ failed")

    monkeypatch.setattr(_build, "build_marshal", no_compiler)
    assert ld._load_gather() is ld._gather_tensors and builds == [True, True]
    # a module that loads after it was built anew is used
    monkeypatch.setattr(ld.importlib, "import_module", lambda n, p=None: real(n, p) if len(builds) == 3 else fails(n))
    monkeypatch.setattr(_build, "build_marshal", lambda force=True: builds.append(force))
    assert ld._load_gather() is not ld._gather_tensors and len(builds) == 3


def test_a_module_of_another_torch_does_not_load():
    code = ("import sys, torch; torch.__version__ = '0.0'\n"
            f"sys.path.insert(0, {os.path.dirname(_build.MARSHAL)!r})\n"
            "try:\n    import _marshal\nexcept ImportError as e:\n    print('refused', e)\n")
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert res.stdout.startswith("refused _marshal was built for torch " + torch.__version__), res.stdout + res.stderr


def test_processes_that_build_at_once_have_files_of_their_own(monkeypatch):
    outs = []
    monkeypatch.setattr(_build.subprocess, "run", lambda cmd, **kw: outs.append(cmd[cmd.index("-o") + 1]) or
                        subprocess.CompletedProcess(cmd, 0, "", ""))
    monkeypatch.setattr(_build.os, "replace", lambda a, b: outs.append((a, b)))
    for pid in (11, 12):
        monkeypatch.setattr(_build.os, "getpid", lambda: pid)
        _build.build_marshal()
        _build.build_library()
    made, moved = outs[0::2], outs[1::2]
    assert len(set(made)) == 4 and [m[0] for m in moved] == made
    assert {m[1] for m in moved} == {_build.MARSHAL, _build.LIB}
