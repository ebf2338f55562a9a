"""What the Python binding refuses, keeps and needs before any kernel is launched (no GPU needed)."""
import pytest

from paper_2309_04875_amd import hb


class _Everything:
    """Short cuts that would serve whatever they are given."""
    def __getattr__(self, name):
        return lambda *args: 7


@pytest.mark.parametrize("call", [hb.hb_relu_batch_ex, hb.hb_drelu_batch_ex])
def test_a_batch_without_its_layout_is_refused(call, monkeypatch):
    monkeypatch.setattr(hb, "_native", _Everything())
    monkeypatch.setattr(hb, "_stream_handle", lambda stream: None)
    assert call([], hb.HB_DEALER_PER_GATE) == 7
    with pytest.raises(TypeError):
        call([], None)
