"""Forms that the general path refuses stay refused where the compiled binding
is asked first: None means the default operator and the default kernels only
inside the binding's own arguments."""
import pytest

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
