"""The layer calls' argument conversion (csrc/pycall.cpp): what the library is handed, argument by
argument, against the same calls through ctypes (both reach host functions that record it), and what is
refused before any device work, whatever the argument forms."""
import contextlib
import ctypes as C
import gc
import weakref

import numpy as np
import pytest

import paper_2604_07173_amd as L


class Seg:
    """A Segments object without device memory: the C structure and a scratch tensor's face."""

    def __init__(self):
        from paper_2604_07173_amd import binding
        self.c, self.ws = binding._Segments(), Buffer(512)
        self.c.P, self.c.tile_rows, self.c.n_keys = 4, 16, 4


class Buffer:
    def __init__(self, n, address=4096):
        self.n, self.address = n, address

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.n

    def element_size(self):
        return 1


def calls(pool, seg, x, ys, lds, ws):
    yield "build_segments", lambda: L.lora_build_segments(pool, x, None, 4, seg, stream=0)
    yield "apply", lambda: L.lora_apply(pool, 0, 0, x, 8, None, seg, ys[0], 8, x, stream=0)
    yield "apply_group", lambda: L.lora_apply_group(pool, 0, 0, x, 8, None, seg, ys, lds, ws, stream=0)
    yield "build_apply_group", lambda: L.lora_build_apply_group(pool, 0, 0, x, 8, None, x, None, 4, seg, ys, lds, ws,
                                                                stream=0)
    yield "moe_apply", lambda: L.lora_moe_apply(pool, 0, 0, x, 8, x, seg, x, x, 8, ws, stream=0)
    yield "moe_build_apply", lambda: L.lora_moe_build_apply(pool, 0, 0, x, 8, x, x, x, 4, seg, x, x, 8, ws, stream=0)
    yield "moe_down_combine", lambda: L.lora_moe_down_combine(pool, 0, x, 8, x, x, seg, x, 2, x, 8, ws, stream=0)
    yield "load_adapter_layer", lambda: L.lora_pool_load_adapter_layer(pool, 0, 0, x, stream=0)


@pytest.mark.parametrize("pool", [None, 0, C.c_void_p(None)])
def test_a_missing_pool_is_refused_by_every_call(pool):
    x, ws = Buffer(64), Buffer(1 << 16)
    for name, call in calls(pool, Seg(), x, [x], [8], ws):
        with pytest.raises(L.LoraError) as e:
            call()
        assert e.value.status == -5, name


def test_argument_forms_and_mistakes():
    x, ws, seg = Buffer(64), Buffer(1 << 16), Seg()

    def group(ys, lds, layer=0, segments=seg, stream=0, ldx=8):
        return L.lora_apply_group(None, layer, 0, x, ldx, None, segments, ys, lds, ws, stream=stream)

    for ys, lds in ([x], [8]), ((x, 4096), (np.int64(8), 8.0)), ([], []), ([x] * 9, [8] * 9), ([x, x], [8]):
        with pytest.raises(L.LoraError):              # converted, then refused for the missing pool
            group(ys, lds)
    with pytest.raises(IndexError):
        group([x], [8, 8])
    with pytest.raises(AttributeError):
        group([x], [8], segments=x)
    with pytest.raises(AttributeError):
        group([object()], [8])
    with pytest.raises(TypeError):
        group([x], [8], ldx="8")
    with pytest.raises(OverflowError):
        group([x], [8], layer=1 << 40)

    class Stream:
        cuda_stream = 0

    with pytest.raises(L.LoraError):
        group([x], [8], stream=Stream())


ENTRIES = ("lora_build_segments", "lora_apply", "lora_apply_group", "lora_build_apply_group", "lora_moe_apply",
           "lora_moe_build_apply", "lora_moe_down_combine", "lora_pool_load_adapter_layer")


@contextlib.contextmanager
def recorded():
    """The extension module bound to host functions that note their arguments; yields (calls, ctypes
    functions with the library's prototypes at the same addresses)."""
    from paper_2604_07173_amd import binding
    lib = L.load_library()
    calls, keep, addresses, through_ctypes = [], [], {}, {}
    for name in ENTRIES:
        types = getattr(lib, name).argtypes
        group = "apply_group" in name

        def note(*args, name=name, types=types, group=group):
            got = []
            for t, v in zip(types, args):
                if t is C.POINTER(binding._Segments):
                    v = (C.addressof(v.contents), v.contents.P, v.contents.n_keys)
                elif t in (C.POINTER(C.c_void_p), C.POINTER(C.c_int64)):
                    v = [v[i] for i in range(min(args[3], 8))]
                got.append(v)
            calls.append((name, got))
            return 0

        proto = C.CFUNCTYPE(C.c_int, *types)
        keep.append(proto(note))
        addresses[name] = C.cast(keep[-1], C.c_void_p).value
        through_ctypes[name] = proto(addresses[name])
    binding._calls().bind(addresses, binding._stream)
    try:
        yield calls, through_ctypes
    finally:
        binding._calls().bind({n: C.cast(getattr(lib, n), C.c_void_p).value for n in binding.EXPORTED_SYMBOLS},
                              binding._stream)


def test_every_argument_arrives_where_ctypes_puts_it():
    b = [Buffer(1000 + i, 0x7F0000000000 + 4096 * i) for i in range(12)]         # addresses beyond 32 bits
    a = [v.address for v in b]
    big, seg, pool = 1 << 40, Seg(), 0x5500_0000_1000
    ref, sws = C.byref(seg.c), (4096, 512)
    two = (C.c_void_p * 2)(a[3], a[4]), (C.c_int64 * 2)(big, 24)
    f32 = L.LORA_DTYPE_F32
    with recorded() as (calls, ct):
        pairs = [
            (lambda: L.lora_build_segments(pool, b[0], b[1], 7, seg, stream=9),
             lambda: ct["lora_build_segments"](pool, a[0], a[1], 7, ref, *sws, 9)),
            (lambda: L.lora_apply(pool, 2, 3, b[0], big, b[1], seg, b[2], 16, b[3], f32, stream=9),
             lambda: ct["lora_apply"](pool, 2, 3, a[0], big, a[1], ref, a[2], 16, f32, a[3], 9)),
            (lambda: L.lora_apply_group(pool, 2, 3, b[0], 16, b[1], seg, [b[3], a[4]], (np.int64(big), 24), b[5], f32, 9),
             lambda: ct["lora_apply_group"](pool, 2, 3, 2, a[0], 16, a[1], ref, *two, f32, a[5], 1005, 9)),
            (lambda: L.lora_build_apply_group(pool, 2, 3, b[0], 16, b[1], b[6], b[7], 7, seg, (b[3], b[4]), [big, 24], b[5],
                                              stream=9),
             lambda: ct["lora_build_apply_group"](pool, 2, 3, 2, a[0], 16, a[1], a[6], a[7], 7, ref, *sws, *two, 0, a[5],
                                                  1005, 9)),
            (lambda: L.lora_moe_apply(pool, 2, 1, b[0], 16, b[1], seg, b[2], b[3], big, b[4], 77, stream=9),
             lambda: ct["lora_moe_apply"](pool, 2, 1, a[0], 16, a[1], ref, a[2], a[3], big, a[4], 77, 9)),
            (lambda: L.lora_moe_build_apply(pool, 2, 1, b[0], 16, b[1], b[5], b[6], 7, seg, b[2], None, big, b[4], stream=9),
             lambda: ct["lora_moe_build_apply"](pool, 2, 1, a[0], 16, a[1], a[5], a[6], 7, ref, *sws, a[2], None, big, a[4],
                                                1004, 9)),
            (lambda: L.lora_moe_down_combine(pool, 2, b[0], 16, b[1], b[5], seg, b[6], 4, b[2], big, b[4], 78, stream=9),
             lambda: ct["lora_moe_down_combine"](pool, 2, a[0], 16, a[1], a[5], ref, a[6], 4, a[2], big, a[4], 78, 9)),
            (lambda: L.lora_pool_load_adapter_layer(pool, 5, 2, b[0], stream=9),
             lambda: ct["lora_pool_load_adapter_layer"](pool, 5, 2, a[0], 9)),
        ]
        for short, long_way in pairs:
            short()
            assert long_way() == 0
            (name, got), (name2, want) = calls[-2:]
            assert name == name2 and got == want, name
        assert {name for name, _ in calls} == set(ENTRIES)


def test_segments_live_as_long_as_the_call():
    """A Segments object that hands out its structure anew each time: the call's own one is still there,
    with its contents, while the library runs."""
    from paper_2604_07173_amd import binding
    made = []

    class Fresh(Seg):
        @property
        def c(self):
            s = binding._Segments()
            s.P, s.n_keys = 1234, 56
            made.append(weakref.ref(s))
            return s

        @c.setter
        def c(self, value):
            pass

    lib, alive = L.load_library(), []
    types = lib.lora_build_segments.argtypes

    def look(*args):
        gc.collect()
        alive.append(made[-1]() is not None)
        return 0

    stub = C.CFUNCTYPE(C.c_int, *types)(look)
    addresses = {n: C.cast(getattr(lib, n), C.c_void_p).value for n in binding.EXPORTED_SYMBOLS}
    try:
        binding._calls().bind(dict(addresses, lora_build_segments=C.cast(stub, C.c_void_p).value), binding._stream)
        L.lora_build_segments(None, 4096, None, 4, Fresh(), stream=0)
    finally:
        binding._calls().bind(addresses, binding._stream)
    assert alive == [True] and made[-1]() is None


def test_nine_outputs_are_refused_by_the_library_not_written_past():
    x, ws, seg = Buffer(64), Buffer(1 << 16), Seg()
    with pytest.raises(L.LoraError) as e:
        L.lora_build_apply_group(None, 0, 0, x, 8, None, x, None, 4, seg, [x] * 4000, [8] * 4000, ws, stream=0)
    assert e.value.status == -5


@pytest.mark.gpu
def test_too_many_outputs_are_refused_for_a_registered_pool():
    """More outputs than a group may have, up to and beyond the module's own table of them: refused for
    their number, by both group calls, before anything is enqueued."""
    import torch
    desc = L.PoolDesc(2, 1, 1, [(8, 8)] * 8, 16)
    slab = torch.zeros(L.lora_pool_bytes(desc), dtype=torch.uint8, device="cuda")
    pool = L.lora_register_pool(desc, slab)
    seg, P = L.Segments(4), 4
    aid = torch.zeros(P, dtype=torch.int32, device="cuda")
    x, y = torch.zeros(P, 8, dtype=torch.bfloat16, device="cuda"), torch.ones(P, 8, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    L.lora_build_segments(pool, aid, None, P, seg)
    for n in (0, 4, 8, 9, 4000):
        for call in (lambda: L.lora_apply_group(pool, 0, 0, x, 8, None, seg, [y] * n, [8] * n, ws),
                     lambda: L.lora_build_apply_group(pool, 0, 0, x, 8, None, aid, None, P, seg, [y] * n, [8] * n, ws)):
            with pytest.raises(L.LoraError) as e:
                call()
            assert e.value.status == -1, n
    torch.cuda.synchronize()
    assert bool((y == 1).all())


def test_current_stream_without_torchs_private_calls(monkeypatch):
    """A torch that has renamed the calls behind torch.cuda.current_stream(): the handle comes from the
    Stream object, as before there was a short way."""
    import torch
    from paper_2604_07173_amd import binding

    class Current:
        cuda_stream = 0x77

    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Current())
    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name)
    L.load_library()
    assert binding._stream(None) == 0x77
    with pytest.raises(L.LoraError) as e:
        L.lora_pool_load_adapter_layer(None, 0, 0, Buffer(64))
    assert e.value.status == -5
