"""The Python binding's own shortcuts: what they may not accept or remember."""

import ctypes

import pytest

import paper_2510_16045_amd as ams


def test_packed_bytes_takes_integers_only_whatever_was_asked_before():
    assert ams.ams_packed_bytes(ams.FP425, 16, 128) == 16 * 128 * 17 // 32 * 4  # K padded to four records
    for args in ((ams.FP425, 16.0, 128), (float(ams.FP425), 16, 128), (ams.FP425, [16], 128)):
        with pytest.raises(ctypes.ArgumentError):
            ams.ams_packed_bytes(*args)


def test_packed_bytes_of_a_changed_ctypes_integer():
    n = ctypes.c_int64(16)
    small = ams.ams_packed_bytes(ams.FP425, n, 128)
    n.value = 32
    assert ams.ams_packed_bytes(ams.FP425, n, 128) == 2 * small


def test_stream_without_torchs_private_name(monkeypatch):
    torch = pytest.importorskip("torch")

    class Stream:
        cuda_stream = 123

    monkeypatch.setattr(ams, "_current_stream", None)  # bound anew, and as before afterwards
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert ams._stream() == 123


@pytest.mark.gpu
def test_stream_is_the_current_one():
    torch = pytest.importorskip("torch")
    side = torch.cuda.Stream()
    assert ams._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert ams._stream() == side.cuda_stream
