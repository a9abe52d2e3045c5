"""Which stream's memory the Python binding takes for arrays that a call allocates and
drops (no GPU: torch's allocator and streams, and the library, are stand-ins that record).
The caching allocator orders a block's reuse on the stream that was current when it was
allocated, so such an array has to come from the stream that the kernels run on."""
import contextlib
import types

import pytest

import paper_2607_05061_amd as kv


class _Stream:
    def __init__(self, ptr):
        self.cuda_stream = ptr


class _External(_Stream):
    def __init__(self, ptr, device=None):
        super().__init__(ptr)


class _Tensor:
    """A device tensor that knows the stream it was allocated on; never dereferenced."""
    n = 0

    def __init__(self, shape, dtype, device, pool=None):
        self.shape, self.dtype, self.device, self.pool = tuple(shape), dtype, device, pool
        _Tensor.n += 1
        self.ptr = _Tensor.n << 40

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return self.ptr

    def numel(self):
        r = 1
        for x in self.shape:
            r *= x
        return r

    def record_stream(self, s):
        pass

    def element_size(self):
        return {"bf16": 2, "f32": 4, "i32": 4, "u8": 1}[self.dtype]


class _World:
    def __init__(self, monkeypatch, capturing=False):
        self.device = types.SimpleNamespace(type="cuda", index=0)
        self.main, self.side = _Stream(0x1000), _Stream(0x2000)
        self.current, self.allocated, self.calls = self.main, [], []
        world = self

        @contextlib.contextmanager
        def stream(s):
            before, world.current = world.current, s
            try:
                yield
            finally:
                world.current = before

        def empty(shape, dtype=None, device=None):
            t = _Tensor((shape,) if isinstance(shape, int) else shape, dtype, device, world.current)
            world.allocated.append(t)
            return t

        cuda = types.SimpleNamespace(
            Stream=_Stream, ExternalStream=_External, stream=stream, current_stream=lambda device=None: world.current,
            default_stream=lambda device=None: _Stream(0), current_device=lambda: 0,
            is_current_stream_capturing=lambda: capturing and world.current.cuda_stream == world.side.cuda_stream)
        fake = types.SimpleNamespace(Tensor=_Tensor, empty=empty, cuda=cuda, bfloat16="bf16", float32="f32", int32="i32",
                                     uint8="u8")
        real = kv.lib()

        class _Lib:
            kvpop_running_topk_workspace_size = staticmethod(real.kvpop_running_topk_workspace_size)

            def __getattr__(self, name):
                if name.startswith("kvpop_internal"):
                    return getattr(real, name)

                def call(*args):
                    world.calls.append((name, args))
                    return kv.KVPOP_OK
                return call

        lib = _Lib()
        monkeypatch.setattr(kv, "_torch", lambda: fake)
        monkeypatch.setattr(kv, "lib", lambda: lib)

    def given(self, shape, dtype):
        return _Tensor(shape, dtype, self.device)

    def scores_call(self, stream, T=4096, **more):
        """kvpop_future_attn_scores of a size whose heads are spread, on a stream that is not
        the current one, into the caller's own array: what it allocated, and its `out`."""
        q, k = self.given((1, 8, T, 128), "bf16"), self.given((1, 2, T, 128), "bf16")
        lse, sc = self.given((1, 8, T), "f32"), self.given((1, 2, T), "f32")
        got, mass = kv.kvpop_future_attn_scores(q, k, lse, 0.1, scores=sc, stream=stream, **more)
        assert got is sc
        (name, args), = self.calls
        assert name == "kvpop_future_attn_scores" and args[12] == (stream or self.current).cuda_stream
        return self.allocated, args[10], mass


def test_masses_of_spread_scores_come_from_the_launch_stream(monkeypatch):
    w = _World(monkeypatch)
    allocated, out, mass = w.scores_call(w.side)
    assert mass is None and [t.pool for t in allocated] == [w.side]
    assert out == allocated[0].data_ptr() and allocated[0].shape == (1, 8, 4096)
    assert w.current is w.main


def test_masses_on_the_current_stream(monkeypatch):
    w = _World(monkeypatch)
    allocated, out, _ = w.scores_call(None)
    assert [t.pool for t in allocated] == [w.main] and out == allocated[0].data_ptr()


@pytest.mark.parametrize("ptr", [0x2000, 0])
def test_a_stream_may_be_any_object_with_a_handle(monkeypatch, ptr):
    w = _World(monkeypatch)
    allocated, _, _ = w.scores_call(types.SimpleNamespace(cuda_stream=ptr))
    assert [t.pool.cuda_stream for t in allocated] == [ptr] and isinstance(allocated[0].pool, _Stream)


def test_nothing_is_allocated_under_capture(monkeypatch):
    """A captured launch would go on writing into an array that is freed on return."""
    w = _World(monkeypatch, capturing=True)
    allocated, out, _ = w.scores_call(w.side)
    assert allocated == [] and out is None


def test_nothing_is_allocated_where_the_epilogue_is_fused(monkeypatch):
    w = _World(monkeypatch)
    allocated, out, _ = w.scores_call(w.side, T=100)
    assert allocated == [] and out is None


def test_masses_the_caller_asks_for_are_returned(monkeypatch):
    w = _World(monkeypatch, capturing=True)
    allocated, out, mass = w.scores_call(w.side, write_mass=True)
    assert allocated == [mass] and out == mass.data_ptr()


@pytest.mark.parametrize("explicit", [True, False])
def test_top_k_workspace_comes_from_the_launch_stream(monkeypatch, explicit):
    w = _World(monkeypatch)
    r = w.given((1, 8, 4096), "f32")
    out = kv.kvpop_running_topk(r, 4, 256, 2016, stream=w.side if explicit else None)
    (name, args), = w.calls
    assert name == "kvpop_running_topk"
    scratch = [t for t in w.allocated if all(t is not o for o in out.values())]
    assert [t.pool for t in scratch] == [w.side if explicit else w.main]
    assert args[11] == scratch[0].data_ptr() and args[12] == scratch[0].numel()
    assert all(o.pool is w.main for o in out.values())
