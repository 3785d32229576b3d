"""The native per-step calls against the C ABI called through ctypes: the same
outputs, shapes, types, columns, streams and errors."""
import numpy as np
import pytest
import torch

from paper_2310_05205_amd import gear
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu

COLS = [("obs", "bfloat16", (3, 5)), ("action", torch.int32, ()), ("u", torch.uint8, (7,)), ("d", torch.float64, (2,))]


@pytest.fixture
def table():
    t = gear.Table(COLS, 50, 9)
    g = torch.Generator().manual_seed(1)
    rows = [torch.randint(0, 256, (50, 9 * e), dtype=torch.uint8, generator=g) for e in t.elem_bytes]
    t.insert(rows, np.arange(1, 51, dtype=np.uint32))
    t.raw = rows
    yield t
    t.close()


def _ctypes_select(t, strategy, B, L, seed, beta):
    idx = torch.empty(B, dtype=torch.int64, device=cuda())
    start = torch.empty(B, dtype=torch.int32, device=cuda())
    w = torch.empty(B, dtype=torch.float32, device=cuda())
    gear.gear_select(t.handle, strategy, B, L, seed, beta, idx.data_ptr(), start.data_ptr(), w.data_ptr(),
                     torch.cuda.current_stream().cuda_stream)
    return idx, start, w


def test_outputs_equal_the_c_calls(table):
    t = table
    for seed in (5, -3, (1 << 64) + 9, np.int64(12), 7.0):
        for strategy in (gear.GEAR_PRIORITIZED, gear.GEAR_UNIFORM, gear.GEAR_TOPK):
            got, want = t.select(strategy, 33, 4, seed, 0.5, weights=True), _ctypes_select(t, strategy, 33, 4, seed, 0.5)
            for a, b in zip(got, want):
                assert a.dtype == b.dtype and torch.equal(a, b)
    assert t.select(gear.GEAR_FIFO, np.int32(4), 4, 1)[2] is None
    idx, start, _ = t.select(gear.GEAR_UNIFORM, 33, 4, 5)
    raw = t.collect(idx, start, 4)
    typed = t.collect_fields(idx, start, 4)
    assert list(typed) == ["obs", "action", "u", "d"] and isinstance(raw, list)
    for (name, dtype, shape), r, e, src in zip(COLS, raw, t.elem_bytes, t.raw):
        assert r.shape == (33, 4 * e) and r.dtype == torch.uint8
        cols = host(start)[:, None].astype(np.int64) * e + np.arange(4 * e)
        assert np.array_equal(host(r), src.numpy()[host(idx)[:, None], cols])
        v = typed[name]
        assert v.shape == (33, 4) + shape and v.dtype == getattr(torch, str(dtype).replace("torch.", ""))
        assert v.is_contiguous() and torch.equal(v.view(torch.uint8).reshape(33, -1), r)
    i2, s2, w2, f2 = t.select_collect_fields(gear.GEAR_UNIFORM, 33, 4, 5, fields=["u", "obs"], weights=True)
    assert torch.equal(i2, idx) and torch.equal(s2, start) and bool((w2 == 1).all()) and list(f2) == ["u", "obs"]
    assert torch.equal(f2["u"], typed["u"]) and torch.equal(f2["obs"].view(torch.int16), typed["obs"].view(torch.int16))
    i3, s3, w3, r3 = t.select_collect(gear.GEAR_UNIFORM, 33, 4, 5, col_ids=(2, 2))
    assert w3 is None and len(r3) == 2 and torch.equal(r3[0], raw[2]) and torch.equal(r3[1], raw[2])
    out = {"u": torch.zeros(33, 28, dtype=torch.uint8, device=cuda())}
    reused = t.collect_fields(idx, start, 4, fields=["u"], out=out)
    assert reused["u"].data_ptr() == out["u"].data_ptr() and torch.equal(out["u"], raw[2])


def test_anything_with_an_address_is_accepted(table):
    class Words:
        def __init__(self, x):
            self.x, self.shape = x, x.shape

        def data_ptr(self):
            return self.x.data_ptr()

    t = table
    idx, start, _ = t.select(gear.GEAR_FIFO, 10, 9, 0)
    for a, b in zip(t.collect(idx, start, 9), t.collect(Words(idx), Words(start), 9)):
        assert torch.equal(a, b)
    t.update_priorities(Words(idx), Words(torch.full((10,), 99, dtype=torch.int32, device=cuda())))
    assert (t.priorities()[host(idx)] == 99).all()


def test_stream_argument_orders_the_call(table):
    t = table
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    idx, start, _ = t.select(gear.GEAR_UNIFORM, 20, 3, 4, stream=s)
    raw = t.collect(idx, start, 3, stream=s)
    t.update_priorities(idx, torch.ones(20, dtype=torch.int32, device=cuda()), stream=s)
    s.synchronize()
    torch.cuda.current_stream().wait_stream(s)
    for a, b in zip(raw, t.collect(idx, start, 3)):
        assert torch.equal(a, b)
    assert t.sync() == 0


def test_errors_are_those_of_the_library(table):
    t = table
    idx, start, _ = t.select(gear.GEAR_UNIFORM, 5, 3, 4)
    for call, code in ((lambda: t.select(9, 5, 3, 0), gear.GEAR_E_INVAL),
                       (lambda: t.select(gear.GEAR_UNIFORM, 5, 10, 0), gear.GEAR_E_INVAL),
                       (lambda: t.select(gear.GEAR_UNIFORM, 0, 3, 0), gear.GEAR_E_INVAL),
                       (lambda: t.select(gear.GEAR_PRIORITIZED, 5, 3, 0, float("nan")), gear.GEAR_E_INVAL),
                       (lambda: t.select(gear.GEAR_FIFO, 51, 3, 0), gear.GEAR_E_INSUFFICIENT),
                       (lambda: t.collect(idx, start, 10), gear.GEAR_E_INVAL),
                       (lambda: t.collect(idx, start, 3, col_ids=[-1]), gear.GEAR_E_INVAL),
                       (lambda: t.select_collect(gear.GEAR_PRIORITIZED, 5, 3, 0), gear.GEAR_E_INVAL)):
        with pytest.raises(gear.GearError) as e:
            call()
        assert e.value.code == code
    for call, kind in ((lambda: t.collect(idx, start, 3, col_ids=[4]), IndexError),
                       (lambda: t.collect_fields(idx, start, 3, fields=["nothing"]), KeyError),
                       (lambda: t.select(gear.GEAR_UNIFORM, -1, 3, 0), RuntimeError),
                       (lambda: t.select(gear.GEAR_UNIFORM, 5.5, 3, 0), TypeError),
                       (lambda: t.select(gear.GEAR_UNIFORM, 5, 3, "x"), ValueError)):
        with pytest.raises(kind):
            call()
    t.close()
    with pytest.raises(gear.GearError):
        t.select(gear.GEAR_UNIFORM, 5, 3, 0)
