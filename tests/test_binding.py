"""The binding's look at a tensor: in native code where that was built for this torch and Python, else the same in Python."""
import warnings

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
