"""The layer calls' argument conversion (csrc/pycall.cpp) against the same calls through ctypes: the
library refuses both with the same status before any device work, whatever the argument forms."""
import ctypes as C

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


def test_nine_outputs_are_refused_by_the_library_not_written_past():
    x, ws, seg = Buffer(64), Buffer(1 << 16), Seg()
    with pytest.raises(L.LoraError) as e:
        L.lora_build_apply_group(None, 0, 0, x, 8, None, x, None, 4, seg, [x] * 4000, [8] * 4000, ws, stream=0)
    assert e.value.status == -5


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
