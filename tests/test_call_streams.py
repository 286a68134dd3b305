"""A call given a stream allocates the tensors it makes itself on that stream,
and a batch orders and keeps its buffers for every stream that launches it:
the caching allocator hands out a freed block as soon as the stream it was
allocated on allows.  On the CPU, with the stream and library calls replaced
by records of them."""
import contextlib

import numpy as np
import pytest

torch = pytest.importorskip("torch")


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle
        self.waited = []

    def wait_event(self, e):
        self.waited.append(e)

    def record_event(self):
        return ("event of", self.cuda_stream)


class Lib:
    """Every call succeeds; the stream argument (the last) is recorded."""

    def __init__(self, real):
        self.real, self.ran = real, []

    def __getattr__(self, name):
        if name in ("hmsv_workspace_bytes", "hmsv_strerror"):
            return getattr(self.real, name)
        return lambda *a: (self.ran.append(name), 0)[1]


@pytest.fixture
def cpu(monkeypatch):
    import paper_1707_09683_amd as hm
    from paper_1707_09683_amd import batch
    now = [Stream(1)]
    made = []

    @contextlib.contextmanager
    def on(stream):
        now.append(stream)
        yield
        now.pop()

    def record(fn):
        def f(*a, **k):
            made.append(now[-1].cuda_stream)
            return fn(*a, **k)
        return f

    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: now[-1])
    monkeypatch.setattr(torch.cuda, "device", lambda d: contextlib.nullcontext())
    for name in ("empty", "zeros", "full"):
        monkeypatch.setattr(torch, name, record(getattr(torch, name)))
    lib = Lib(hm._lib)
    monkeypatch.setattr(hm, "_lib", lib)
    monkeypatch.setattr(batch, "_lib", lib)
    return hm, batch, made


def inputs(hm):
    db = hm.Database.__new__(hm.Database)
    db._h, db.nseq = None, 5
    prof = hm.Profile(torch.ones((32, 7), dtype=torch.uint8), torch.ones((32, 7), dtype=torch.int8), 3)
    p7 = hm.P7Profile(torch.ones((32, 7), dtype=torch.int16), torch.ones((7, 7), dtype=torch.int16), 0)
    return db, prof, p7


@pytest.mark.parametrize("side", [False, True], ids=["current", "other"])
def test_own_tensors_come_from_the_calls_stream(cpu, side):
    hm, _, made = cpu
    db, prof, p7 = inputs(hm)
    score, flags = torch.from_numpy(np.zeros(5, np.uint8)), torch.from_numpy(np.zeros(5, np.uint8))
    s16 = torch.from_numpy(np.zeros(5, np.int16))
    i32 = torch.from_numpy(np.zeros(5, np.int32))
    stream = Stream(2) if side else None
    for call in (lambda: hm.msv_score(prof, db, stream=stream),
                 lambda: hm.ssv_score(prof, db, stream=stream),
                 lambda: hm.score_range("msv", prof, db, 1, 2, score, flags, stream=stream),
                 lambda: hm.p7_score(p7, db, stream=stream),
                 lambda: hm.select(db, score, flags, "msv", 9, stream=stream),
                 lambda: hm.p7_score_selected(p7, db, i32, i32, s16, flags, stream=stream),
                 lambda: hm.pipeline("msv", prof, p7, db, 9, stream=stream)):
        made.clear()
        call()
        assert made and set(made) == {2 if side else 1}, made


def test_batch_orders_other_streams(cpu, monkeypatch):
    hm, batch, _ = cpu
    db, prof, _ = inputs(hm)
    kept = []
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: kept.append((t.data_ptr(), s)))
    b = batch.Batch([("msv", prof), ("ssv", prof)], db)
    b.launch()
    assert not kept
    other = Stream(3)
    for _ in range(2):
        b.launch(other)
    assert other.waited == [("event of", 1)]
    assert {p for p, s in kept if s is other} == {t.data_ptr() for t in
                                                  (*b.scores, *b.flags, *b.workspaces)}
    assert len(kept) == 6
