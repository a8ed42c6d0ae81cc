"""Buffer handling of Lattice.step (host logic, CPU).

The library is replaced by a stand-in on CPU tensors whose step adds 1 to
every element of the buffer it reads, so the state after n steps is A + n.
The reference is the plain form of the same call: n steps that alternate
between a copy of A and out."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

SHAPE = (1, 9, 1, 3, 4)


class FakeLibrary:
    """lbm_step as the library does it: the buffers must differ."""

    def __init__(self):
        self.calls = []

    def lbm_state_elems(self, ctx):
        return 108

    def lbm_param_elems(self, ctx):
        return 0

    def lbm_step(self, ctx, A, B, theta, nsteps, stream):
        a, b = (torch.frombuffer((ctypes.c_float * 108).from_address(p.value), dtype=torch.float32)
                for p in (A, B))
        self.calls.append(nsteps)
        if A.value == B.value:
            return 1
        for _ in range(nsteps):
            b.copy_(a + 1)
            a, b = b, a
        return 0

    def lbm_last_error(self):
        return b"A and B must differ"


@pytest.fixture
def lattice(monkeypatch):
    from paper_2403_18466_amd import lbm

    def ptr(t, dtype, numel=None, name="array", allow_none=False):
        if t is None:
            return None
        if not t.is_contiguous() or t.dtype != dtype or t.numel() != numel:
            raise ValueError(name)
        return ctypes.c_void_p(t.data_ptr())

    lib = FakeLibrary()
    monkeypatch.setattr(lbm, "load_library", lambda: lib)
    monkeypatch.setattr(lbm, "_ptr", ptr)
    monkeypatch.setattr(lbm, "_stream", lambda s: None)
    L = object.__new__(lbm.Lattice)
    L.cfg = lbm.Config(nx=4, ny=3)
    L.ctx, L.device, L.lib = None, torch.device("cpu"), lib
    L.n_state, L.n_param = 108, 0
    return L


def plain(A, nsteps, out=None):
    a = A.clone()
    b = torch.empty(SHAPE) if out is None else out
    for _ in range(nsteps):
        b.copy_((a + 1).reshape(b.shape))
        a, b = b, a
    return a


@pytest.mark.parametrize("nsteps", [0, 1, 2, 3, 6])
@pytest.mark.parametrize("shape", [SHAPE, (9, 3, 4), (108,)])
def test_result_shape(lattice, shape, nsteps):
    """States are taken by their number of elements: the result has A's shape
    after an even number of steps and out's after an odd one."""
    A = torch.arange(108.0).reshape(shape)
    A0 = A.clone()
    want = plain(A0, nsteps)
    got = lattice.step(A, None, nsteps)
    assert torch.equal(A, A0)
    assert got.shape == want.shape
    assert torch.equal(got, want)


@pytest.mark.parametrize("nsteps", [1, 2, 3])
@pytest.mark.parametrize("first", [0, 108, 54])
def test_out_in_the_same_memory(lattice, first, nsteps):
    """out as a tensor of another storage on A's memory (an array taken over
    by another library): all of A, none of it, half of it."""
    base = torch.arange(3 * 108.0)
    A = base[108:216].reshape(SHAPE)
    out = torch.from_dlpack(base[first:first + 108])
    want = plain(A, nsteps)
    got = lattice.step(A, None, nsteps, out=out)
    assert torch.equal(got.reshape(SHAPE), want)
    if nsteps % 2 == 1:
        assert got.data_ptr() == out.data_ptr()


@pytest.mark.parametrize("nsteps", [1, 2, 10])
def test_arguments_are_marshalled_once(lattice, monkeypatch, nsteps):
    """On small grids a call's time is the host's: every step after the first
    goes in one library call, and each argument is checked and the stream
    looked up once."""
    from paper_2403_18466_amd import lbm
    streams, names = [], []
    check = lbm._ptr
    monkeypatch.setattr(lbm, "_stream", lambda s: streams.append(s))
    monkeypatch.setattr(lbm, "_ptr", lambda t, *a, **k: (names.append(id(t)), check(t, *a, **k))[1])
    A = torch.arange(108.0).reshape(SHAPE)
    got = lattice.step(A, None, nsteps)
    assert torch.equal(got, A + nsteps)
    assert sum(lattice.lib.calls) == nsteps and len(lattice.lib.calls) <= 2
    assert len(streams) == 1
    names = [n for n in names if n != id(None)]
    assert len(names) == len(set(names))
