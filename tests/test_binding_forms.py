"""The binding's calls of a serving loop: tensors, plain addresses and None, stream objects and raw handles, in any mixture, reach
the library as the same call, and none of them is taken up twice."""
import itertools

import pytest

from paper_2604_24013_amd import binding as cf


class Tensor:
    def __init__(self, at):
        self.at, self.asked = at, 0

    def data_ptr(self):
        self.asked += 1
        return self.at


class Stream:
    def __init__(self, handle):
        self.handle, self.asked = handle, 0

    @property
    def cuda_stream(self):
        self.asked += 1
        return self.handle


class Handle(int):
    pass


class Library:
    """Writes down what it is called with."""
    def __getattr__(self, name):
        return lambda *args: self.seen.append((name, args)) or self.status

    def __init__(self):
        self.seen, self.status = [], cf.CF_OK


@pytest.fixture
def lib(monkeypatch):
    lib = Library()
    monkeypatch.setattr(cf, "_lib", lib)
    return lib


POINTERS = {"rs_step": 4, "rs_step_noalloc": 4, "ag_step": 3}
FORMS = {"tensor": Tensor, "address": int, "handle": Handle}


@pytest.mark.parametrize("name", POINTERS)
@pytest.mark.parametrize("stream", [Stream, int, Handle, None])
def test_steps_take_every_form(lib, name, stream):
    n, desc = POINTERS[name], object()
    for forms in itertools.product(FORMS, repeat=n):
        args = [FORMS[f](0x1000 * (i + 1)) for i, f in enumerate(forms)]
        s = stream(0x77) if stream else None
        getattr(cf, name)(desc, 3, *args, s)
        (called, got), = lib.seen
        assert called == "commfuse_" + name and got[:2] == (desc, 3)
        assert [int(a) for a in got[2:-1]] == [0x1000 * (i + 1) for i in range(n)] and (got[-1] if s is None else int(got[-1])) == (0x77 if stream else None)
        if "handle" not in forms and stream is not Handle:            # (an int of another class is looked at again)
            assert all(a.asked == 1 for a in args + [s] if isinstance(a, (Tensor, Stream)))
        lib.seen.clear()


@pytest.mark.parametrize("first,second", itertools.product([Stream, int, Handle, None], repeat=2))
def test_schedules_take_every_form(lib, first, second):
    desc, bufs = object(), object()
    streams = [f(0x70 + i) if f else None for i, f in enumerate((first, second))]
    cf.run_schedule(desc, cf.CF_KIND_AG, bufs, *streams, cf.CF_SERIAL)
    (called, got), = lib.seen
    assert called == "commfuse_run_schedule" and got[:3] == (desc, cf.CF_KIND_AG, bufs) and got[5] == cf.CF_SERIAL
    assert [s if s is None else int(s) for s in got[3:5]] == [0x70 + i if f else None for i, f in enumerate((first, second))]
    if Handle not in (first, second):
        assert all(s.asked == 1 for s in streams if isinstance(s, Stream))


@pytest.mark.parametrize("recv", [None, 0x3000])
def test_a_missing_operand_is_null(lib, recv):
    cf.rs_step(object(), 0, None, 0x2000, recv, Tensor(0x4000), 0)
    assert lib.seen[0][1][2:6] == (None, 0x2000, recv, 0x4000) and not lib.seen[0][1][6]


def test_a_failing_status_is_raised(monkeypatch, lib):
    lib.status = cf.CF_ERR_MISALIGNED
    monkeypatch.setattr(cf, "last_error", lambda: "text")
    for call in (lambda: cf.rs_step(object(), 0, 1, 2, None, 3), lambda: cf.ag_step(object(), 0, 1, 2, 3),
                 lambda: cf.run_schedule(object(), 0, object(), None, None)):
        with pytest.raises(cf.CommFuseError) as ei:
            call()
        assert ei.value.status == cf.CF_ERR_MISALIGNED
