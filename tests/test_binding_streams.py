"""The stream table and the trigger records as the binding passes them (no device memory is touched)."""
import ctypes

import pytest

torch = pytest.importorskip("torch")


def test_stream_table():
    from paper_2201_11133_amd import gwd
    a, b = torch.zeros(1001, 2), torch.zeros(4000, 2)[::4]
    c0, c1 = torch.zeros(77), torch.zeros(77)
    d = torch.zeros(2, 90)[:, ::3]
    arr, lengths = gwd.make_streams([a, b, (c0, c1), [d[0], d[1]]])
    want = [(a.data_ptr(), a.data_ptr() + 4, 2, 1001), (b.data_ptr(), b.data_ptr() + 4, 8, 1000),
            (c0.data_ptr(), c1.data_ptr(), 1, 77), (d[0].data_ptr(), d[1].data_ptr(), 3, 30)]
    assert [(s.ch[0], s.ch[1], s.elem_stride, s.length) for s in arr] == want
    assert lengths == [1001, 1000, 77, 30] and all(type(n) is int for n in lengths)
    empty, none = gwd.make_streams([])
    assert len(empty) == 0 and none == []


@pytest.mark.parametrize("bad", [(0,), (5,), (5, 3), (2, 5, 2)])
def test_refused_streams(bad):
    from paper_2201_11133_amd import gwd
    with pytest.raises(AssertionError):
        gwd.make_streams([torch.zeros(*bad)])
    with pytest.raises(AssertionError):
        gwd.make_streams([torch.zeros(6, 4)[:, ::2]])
    with pytest.raises(AssertionError):
        gwd.make_streams([(torch.zeros(5), torch.zeros(4))])
    with pytest.raises(AssertionError):
        gwd.make_streams([(torch.zeros(5), torch.zeros(10)[::2])])
    with pytest.raises(AssertionError):
        gwd.make_streams([(torch.zeros(5), torch.zeros(5, dtype=torch.float64))])


def test_trigger_records():
    from paper_2201_11133_amd import gwd
    assert ctypes.sizeof(gwd.Trigger) == gwd._TRIGGER.size
    buf = (gwd.Trigger * 4)()
    for i in range(4):
        buf[i].stream, buf[i].sample, buf[i].logit, buf[i].prob = i, 10 ** 12 + i, -0.1 * i, 1.0 / (i + 3)
    for n in (0, 1, 4):
        assert gwd._trigger_records(buf, n) == [(t.stream, t.sample, t.logit, t.prob) for t in list(buf)[:n]]
