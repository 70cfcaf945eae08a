"""Forms that the general path refuses stay refused where the compiled binding
is asked first (None means the default operator and the default kernels only
inside the binding's own arguments), and the package works without a binding
that fits."""
import pathlib
import sys
import types

import pytest

from paper_2305_00515_amd import build

torch = pytest.importorskip("torch")


def test_none_is_not_handed_to_the_binding(sobel_lib, monkeypatch):
    monkeypatch.setattr(sobel_lib, "_bind_u8", lambda *a: ("taken", None))
    src = torch.zeros(8, 8, dtype=torch.uint8)
    for call in (sobel_lib.sobel4x5_u8_op, sobel_lib.sobel4x5_u8_weighted):
        assert call(src, 1) == ("taken", None)
        with pytest.raises(TypeError):
            call(src, None)


@pytest.mark.gpu
def test_none_is_no_operator_and_no_weights(sobel_lib, gpu):
    src = torch.zeros(8, 8, dtype=torch.uint8, device=gpu)
    with pytest.raises(TypeError):
        sobel_lib.sobel4x5_u8_weighted(src, None)
    with pytest.raises(Exception) as e:
        sobel_lib.sobel4x5_u8_op(src, None)
    assert e.type.__name__ == "ArgumentError"      # ctypes', from the library call


def test_an_unfit_binding_is_left_out(sobel_lib, monkeypatch):
    """One of another torch, or one that does not load: the package works
    through the library alone, and says so."""
    name = sobel_lib.__package__ + "._bind"
    if not (sobel_lib._PKG / "_bind.so").exists():
        pytest.skip("no binding built")
    assert sobel_lib._load_bind() is not None
    for stand_in in (None, types.SimpleNamespace(built_for="torch 0.1, Python 2.7"), types.SimpleNamespace()):
        monkeypatch.setitem(sys.modules, name, stand_in)
        monkeypatch.delattr(sys.modules[sobel_lib.__package__], "_bind", raising=False)
        with pytest.warns(RuntimeWarning, match="Build again"):
            assert sobel_lib._load_bind() is None


@pytest.mark.parametrize("why", ["no headers", "compile fails", "no compiler"])
def test_the_library_is_built_without_the_binding(tmp_path, monkeypatch, why):
    monkeypatch.setattr(build, "LIB", tmp_path / "lib.so")
    monkeypatch.setattr(build, "BIND", tmp_path / "_bind.so")
    build.BIND.write_text("of an earlier build")
    monkeypatch.setattr(build, "hipcc", lambda: "hipcc")
    run = build._run

    def fake(cmd, verbose):
        if cmd[0] != "hipcc":
            return run(cmd, verbose)
        pathlib.Path(cmd[cmd.index("-o") + 1]).write_text("x")
        return 0

    def command(out):
        if why == "no headers":
            raise ImportError("torch")
        return ["false"] if why == "compile fails" else [str(tmp_path / "no-such-compiler")]

    monkeypatch.setattr(build, "_run", fake)
    monkeypatch.setattr(build, "bind_command", command)
    assert build.build() == build.LIB and build.LIB.exists()
    assert not build.BIND.exists()
