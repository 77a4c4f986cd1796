"""The Python binding's argument checks (csrc/bind.cpp): what a call refuses before anything is launched, and what stands in
for the classes of the package.  The calls without a GPU stop at the first check, or in the library, at a missing pointer."""
import ctypes as C

import numpy as np
import pytest

import paper_2503_22879_amd as q
from paper_2503_22879_amd import binding

SHAPE = dict(batch=1, seqlen=8, nheads=4, headdim=8, d_state=8, ngroups=2, chunk=4, n_head_clusters=1, n_chan_clusters=1,
             flags=0)


def _host_scales():
    return q.HostScales(np.ones(2, np.float32), np.full(2, 2, np.int32), np.full(2, 8, np.int32), np.ones(2, np.float32),
                        np.ones(2, np.float32))


def _prefill(shape=None, scales=None, x=None, **kw):
    """A prefill with every tensor missing: refused by the library for the missing x unless the binding refuses it first."""
    q.quamba_ssd_prefill(q.Shape(**SHAPE) if shape is None else shape,
                         q.DeviceScales(_host_scales(), device="cpu") if scales is None else scales,
                         x, None, None, None, None, None, None, None, **{"stream": 0, **kw})


class Asked(Exception):
    pass


def test_a_complete_call_reaches_the_library():
    with pytest.raises(q.QuambaError) as e:
        _prefill()
    assert e.value.status == -1                       # x is missing
    class Named(q.Shape):
        pass
    with pytest.raises(q.QuambaError):
        _prefill(shape=Named(**SHAPE))


@pytest.mark.parametrize("shape", [bytes(40), np.zeros(10, np.int32), (C.c_int32 * 10)(), 7, "shape", None])
def test_the_shape_is_a_shape(shape):
    """Ten 32-bit numbers are not a Shape, whatever object holds them."""
    with pytest.raises(TypeError):
        q.quamba_ssd_prefill(shape, q.DeviceScales(_host_scales(), device="cpu"), *([None] * 8), stream=0)


def test_scales_other_than_device_scales_are_asked_for_their_struct():
    class Elsewhere(q.DeviceScales):
        def struct(self):
            raise Asked

    class Bytes:
        def struct(self):
            return bytes(40)

    with pytest.raises(Asked):
        _prefill(scales=Elsewhere(_host_scales(), device="cpu"))
    with pytest.raises(TypeError):
        _prefill(scales=Bytes())
    with pytest.raises(AttributeError):
        _prefill(scales=object())
    as_tuple = q.DeviceScales(_host_scales(), device="cpu")
    as_tuple.tensors = tuple(as_tuple.tensors)
    for scales in (_host_scales(), as_tuple):         # accepted: the call stops at the missing x
        with pytest.raises(q.QuambaError):
            _prefill(scales=scales)


def test_gates_other_than_a_gate_are_asked_for_their_struct():
    seen = []

    class Own(q.Gate):
        def struct(self, *shapes):
            seen.append(shapes)
            return super().struct(*shapes)

    class Bytes:
        def struct(self, *shapes):
            return bytes(40)

    with pytest.raises(q.QuambaError):                # goes on to the missing x
        _prefill(gate=Own(z_scale=0.5))
    assert seen == [((1, 8, 4, 8), (1, 8, 4), 4)]
    with pytest.raises(TypeError):
        _prefill(gate=Bytes())
    with pytest.raises(AttributeError):
        _prefill(gate=object())
    st = q.Gate(z_scale=0.5, dt_scale=0.25).struct((1, 8, 4, 8), (1, 8, 4), 4)
    assert isinstance(st, binding._GateStruct) and (st.z, st.z_scale, st.dt_q, st.dt_scale, st.dt_bias) == \
        (None, 0.5, None, 0.25, None)


def test_a_stream_may_be_a_ctypes_pointer():
    class Stream:
        cuda_stream = C.c_void_p(0)

    for stream in (C.c_void_p(0), C.c_void_p(64), C.pointer(C.c_int(1)), (C.c_char * 8)(), Stream(), 64):
        with pytest.raises(q.QuambaError):            # accepted: the call stops at the missing x
            _prefill(stream=stream)
    for stream in (object(), 1.5, [0]):
        with pytest.raises((TypeError, C.ArgumentError)):
            _prefill(stream=stream)


def _decode_arguments(torch):
    """A one-token step of 2 sequences, 4 heads of 8 channels, 8 states."""
    shape = q.Shape(**{**SHAPE, "batch": 2})
    dev = dict(device="cuda")
    a = dict(x=torch.ones(2, 4, 8, dtype=torch.int8, **dev), B=torch.ones(2, 2, 8, dtype=torch.int8, **dev),
             Cm=torch.ones(2, 2, 8, dtype=torch.int8, **dev), dt=torch.ones(2, 4, **dev), A=torch.zeros(4, **dev),
             D=torch.zeros(4, **dev), state=torch.zeros(2, 4, 8, 8, **dev),
             y=torch.zeros(2, 4, 8, dtype=torch.float16, **dev))
    return shape, q.DeviceScales(_host_scales()), a


@pytest.mark.gpu
@pytest.mark.parametrize("name,wrong", [
    ("x", lambda t: t.to("cpu")), ("x", lambda t: t.short()), ("x", lambda t: t.view(8, 8)), ("x", lambda t: t[:1]),
    ("x", lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)), ("x", lambda t: t.tolist()), ("x", lambda t: t.data_ptr()),
    ("B", lambda t: t.half()), ("dt", lambda t: t.double()), ("dt", lambda t: t[:, :3].contiguous()), ("A", lambda t: t.cpu()),
    ("state", lambda t: t[..., ::2]), ("state", lambda t: t.half()), ("state", lambda t: t.cpu()), ("y", lambda t: t.float()),
    ("y", lambda t: t.view(2, 32))])
def test_device_tensors_are_checked(gpu_lib, name, wrong):
    """Device, type, shape and strides of every tensor, before anything is launched: the state stays as it was."""
    import torch
    shape, scales, a = _decode_arguments(torch)
    bad = {**a, name: wrong(a[name])}
    with pytest.raises((ValueError, TypeError)):
        q.quamba_ssd_decode_step(shape, scales, *bad.values())
    assert not a["state"].any() and not a["y"].any()
    q.quamba_ssd_decode_step(shape, scales, *a.values())
    assert (a["state"] == 1).all() and (a["y"] == 8).all()      # dt x B = 1, sum of 8 C h = 8


@pytest.mark.gpu
@pytest.mark.parametrize("name,wrong", [("z", lambda t: t.cpu()), ("z", lambda t: t.view(8, 8)), ("dt_q", lambda t: t.float()),
                                        ("dt_bias", lambda t: t[:2]), ("dt_bias", lambda t: t.half()),
                                        ("z_scale", lambda v: None), ("z_scale", lambda v: "scale")])
def test_side_inputs_are_checked(gpu_lib, name, wrong):
    import torch
    shape, scales, a = _decode_arguments(torch)
    g = dict(z=torch.ones(2, 4, 8, dtype=torch.int8, device="cuda"), z_scale=0.5,
             dt_q=torch.ones(2, 4, dtype=torch.int8, device="cuda"), dt_scale=0.25, dt_bias=torch.zeros(4, device="cuda"))
    with pytest.raises((ValueError, TypeError)):
        q.quamba_ssd_decode_step(shape, scales, *a.values(), gate=q.Gate(**{**g, name: wrong(g[name])}))
    assert not a["state"].any()
    q.quamba_ssd_decode_step(shape, scales, *a.values(), gate=q.Gate(**g))
    assert a["state"].any()


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["current", "object", "number", "pointer"])
def test_the_call_is_enqueued_on_the_stream_it_is_given(gpu_lib, how):
    """Its input is written on that stream behind a wait of some milliseconds: a launch on another stream would read what
    was there before."""
    import torch
    s = torch.cuda.Stream()
    src = torch.randn(64, 1024, device="cuda").half()
    y, out, want = torch.zeros_like(src), torch.empty(64, 1024, dtype=torch.int8, device="cuda"), \
        torch.empty(64, 1024, dtype=torch.int8, device="cuda")
    q.quamba_hadamard_quantize(src, 1.0, want)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        torch.cuda._sleep(20_000_000)
        y.copy_(src)
        if how == "current":
            q.quamba_hadamard_quantize(y, 1.0, out)
    if how != "current":
        q.quamba_hadamard_quantize(y, 1.0, out, stream={"object": s, "number": s.cuda_stream,
                                                        "pointer": C.c_void_p(s.cuda_stream)}[how])
    s.synchronize()
    assert want.any() and torch.equal(out, want)
