"""RandKStep zeroes its output before it gathers unless the gradients overlap it:
the overlap is one of memory, not of storage objects."""
import pytest

torch = pytest.importorskip("torch")
pytest.importorskip("paper_2109_12497_amd", reason="libuq.so not built")

from paper_2109_12497_amd.step import overlap  # noqa: E402


def test_views_of_one_allocation():
    buf = torch.zeros(1000)
    assert overlap(buf[:100], buf[99:200]) and overlap(buf, buf[500:])
    assert not overlap(buf[:100], buf[100:200])
    rows = buf[:900].view(3, 300)
    assert overlap(rows[:, :100], buf[250:260])  # inside the span, between two rows
    assert not overlap(rows[:2, :100], buf[400:])
    assert not overlap(buf[:0], buf)


def test_memory_shared_under_another_storage():
    buf = torch.zeros(1000)
    other = torch.from_dlpack(buf[64:])
    assert other.untyped_storage().data_ptr() != buf.untyped_storage().data_ptr()
    assert overlap(other, buf) and not overlap(other, buf[:64])
    assert not overlap(torch.zeros(1000), buf)
