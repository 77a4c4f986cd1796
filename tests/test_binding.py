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
