"""The views an array keeps of its own buffers are views of the memory the buffers hold now: after another tensor
took a buffer's place, and after the buffer itself was given other memory."""
import torch

from paper_2102_02344_amd import arrays
from paper_2102_02344_amd import binding as hb


def _arena():
    a = arrays.ParamArena.__new__(arrays.ParamArena)
    a.B, a._index, a.seg_offsets = 2, {"x": 0, "y": 1}, [0, 3, 8]
    a.theta, a.lowp, a.grad = torch.arange(16.0), None, torch.zeros(16)
    return a


def _other_memory(a):
    yield setattr(a, "theta", torch.full((16,), 1.0))
    a.theta.data = torch.full((16,), 2.0)
    yield
    a.theta.set_(torch.full((16,), 3.0))
    yield


def test_segments_follow_their_buffer():
    a = _arena()
    assert a.w("y").tolist() == list(range(6, 16)) and a.w("y") is a.w("y")
    for k, _ in enumerate(_other_memory(a), 1):
        for v in (a.w("y"), a.master("y")):
            assert v.data_ptr() == a.theta[6:].data_ptr() and v.tolist() == [float(k)] * 10


def test_cuts_follow_their_buffer():
    a = _arena()
    buf = a.theta
    assert a._cut(buf, 5).tolist() == list(range(5)) and a._cut(buf, 5) is a._cut(buf, 5)
    buf.data = torch.full((16,), 4.0)
    assert a._cut(buf, 5).data_ptr() == buf.data_ptr() and a._cut(buf, 5).tolist() == [4.0] * 5


def test_strides_are_read_on_every_call():
    """Numbers that can change in place are not remembered by the object that holds them."""
    step = torch.tensor(7)
    s = (step, step, torch.tensor(3), torch.tensor(1))
    assert list(hb._strides(s)) == [7, 7, 3, 1]
    step.fill_(9)
    assert list(hb._strides(s)) == [9, 9, 3, 1] and list(hb._strides([1, 2, 3], 3)) == [1, 2, 3]
    assert hb._strides((4, 3, 2, 1)) is hb._strides((4, 3, 2, 1)) and hb._strides(None) is None
