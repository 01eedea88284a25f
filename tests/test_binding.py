"""The binding's look at a tensor: in native code where that was built for this torch and Python, else the same in Python."""
import warnings

import numpy as np
import pytest

from paper_2605_16637_amd import binding


def test_marshal_is_native_where_built_for_this_torch():
    from paper_2605_16637_amd import build
    import os
    if not os.path.exists(binding.MARSHAL_PATH):
        build.build()
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        address = binding._load_marshal()
    assert address is not binding._ptr_other and address(None) is None


@pytest.mark.parametrize("what", ["missing", "no module", "another torch"])
def test_marshal_that_cannot_be_used_leaves_the_work_to_python(monkeypatch, tmp_path, what):
    if what == "another torch":
        monkeypatch.setattr(binding, "marshal_built_for", lambda: "torch 1.0, cpython-36")
    else:
        path = tmp_path / "hx_marshal.so"
        if what == "no module":
            path.write_bytes(b"not an ELF file")
        monkeypatch.setattr(binding, "MARSHAL_PATH", str(path))
    with pytest.warns(RuntimeWarning, match="hx_marshal"):
        assert binding._load_marshal() is binding._ptr_other


def test_library_is_built_without_what_marshal_needs(monkeypatch, capsys):
    import subprocess
    from paper_2605_16637_amd import build
    done = []

    def compile_(cmd, verbose, out=None):
        if cmd[0] != "hipcc":
            raise subprocess.CalledProcessError(1, cmd)
        done.append(cmd[cmd.index("-o") + 1])
        return out

    monkeypatch.setattr(build, "_compile", compile_)
    assert build.build() == build.LIB and done == [build.CALIB_LIB, build.LIB]
    assert build.MARSHAL_LIB in capsys.readouterr().out


def outcome(look, *args):
    try:
        got = look(*args)
    except Exception as e:
        return type(e), str(e)
    return None if got is None else got.value


# Whatever a tensor is and is asked for, native code and Python say the same of it.
def looked_at(device):
    import torch
    t = torch.arange(24, dtype=torch.int32, device=device)
    i32, f32 = torch.int32, torch.float32

    class Sub(torch.Tensor):
        pass

    raw = binding.RawArray(4096, 24, i32)
    return [(None,), (None, i32, 5), (t,), (t, i32), (t, i32, 24), (t, i32, 25), (t, i32, 0), (t, i32, -1), (t, i32, True), (t, None, 7),
            (t, f32), (t, f32, 24), (t, i32, np.int64(24)), (t, i32, np.int64(25)), (t, i32, 2.5),
            (t, i32, 2**63 - 1), (t, i32, 2**63), (t, i32, 2**70), (t, i32, -2**70), (t, "int32"), (t, i32, "24"),
            (t[3:], i32, 21), (t[3:], i32, 22), (t[::2],), (t.view(4, 6).t(),), (t.view(4, 6)[:, :1],), (t.view(1, 24).t(), i32, 24),
            (t[:0], i32, 0), (t[:0], i32, 1), (t.float(), f32, 24), (t.float().requires_grad_(), f32, 24),
            (torch.nn.Parameter(t.float()), f32, 24), (t.as_subclass(Sub), i32, 24), (t.as_subclass(Sub), i32, 25),
            (torch.empty(24, dtype=i32, device="meta"), i32, 24), (raw, i32, 24), (raw, i32, 25), (raw, f32), (np.arange(24), i32, 24), (5, i32),
            (), (t, i32, 24, 1)]


def native_and_python_agree(device):
    address = binding._load_marshal()
    assert address is not binding._ptr_other
    outcomes = []
    for args in looked_at(device):
        outcomes.append(outcome(binding._ptr_other, *args))
        assert outcome(address, *args) == outcomes[-1], args
    return outcomes


def test_native_and_python_agree_on_host_tensors():
    assert [x for x in native_and_python_agree("cpu") if not isinstance(x, tuple)] == [None, None, 4096]      # the last the raw array


@pytest.mark.gpu
def test_native_and_python_agree_on_device_tensors():
    outcomes = native_and_python_agree("cuda:0")
    assert sum(isinstance(x, int) for x in outcomes) >= 14
