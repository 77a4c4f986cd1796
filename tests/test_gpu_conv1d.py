"""GPU parity of the W8A8 causal convolution in front of the scan (quamba_conv1d_q8) against the oracle, through the
C ABI: the int8 codes of x, B and C and the carried conv state bit for bit."""
import ctypes as C

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import make_problem, make_conv_inputs, to_shape, host_scales

pytestmark = pytest.mark.gpu


def _split(codes, s):
    HP, GN = s.nheads * s.headdim, s.ngroups * s.d_state
    b, L, _ = codes.shape
    return (codes[:, :, :HP].reshape(b, L, s.nheads, s.headdim), codes[:, :, HP:HP + GN].reshape(b, L, s.ngroups, s.d_state),
            codes[:, :, HP + GN:].reshape(b, L, s.ngroups, s.d_state))


def _gpu(q, s, sc, inp, state_in=None, want_state=True, alias=False, offset=0):
    import torch
    b, L = inp["xBC"].shape[:2]
    shape = to_shape(q, s.with_(batch=b, seqlen=L))
    dsc = q.DeviceScales(host_scales(q, sc))
    Ct = inp["xBC"].shape[2]

    def dev(a):
        if offset == 0:
            return torch.from_numpy(np.ascontiguousarray(a)).cuda()
        buf = torch.zeros(a.size + offset, dtype=torch.from_numpy(a).dtype, device="cuda")   # unaligned view
        v = buf[offset:].view(a.shape)
        v.copy_(torch.from_numpy(np.ascontiguousarray(a)))
        return v
    xo = torch.full((b, L, s.nheads, s.headdim), 99, dtype=torch.int8, device="cuda")
    Bo = torch.full((b, L, s.ngroups, s.d_state), 99, dtype=torch.int8, device="cuda")
    Co = torch.full((b, L, s.ngroups, s.d_state), 99, dtype=torch.int8, device="cuda")
    st_in = None if state_in is None else torch.from_numpy(state_in.copy()).cuda()
    st_out = st_in if alias else (torch.full((b, 3, Ct), 99, dtype=torch.int8, device="cuda") if want_state else None)
    q.quamba_conv1d_q8(shape, dsc, dev(inp["xBC"]), torch.from_numpy(inp["weight"]).cuda(),
                       None if inp["bias"] is None else torch.from_numpy(inp["bias"]).cuda(), inp["in_w_scale"],
                       xo, Bo, Co, conv_state_in=st_in, conv_state_out=st_out)
    return xo.cpu().numpy(), Bo.cpu().numpy(), Co.cpu().numpy(), None if st_out is None else st_out.cpu().numpy()


def _check(q, s, sc, inp, state_in=None, **kw):
    os_ = oracle.output_scales(sc, s.nheads, s.headdim, s.ngroups, s.d_state)
    ref, ref_state = oracle.ref_conv1d_q8(inp["xBC"], inp["weight"], inp["in_w_scale"], inp["bias"], os_, state_in)
    rx, rB, rC = _split(ref, s)
    gx, gB, gC, gstate = _gpu(q, s, sc, inp, state_in, **kw)
    for name, g, r in (("x", gx, rx), ("B", gB, rB), ("C", gC, rC)):
        bad = np.argwhere(g != r)
        assert bad.size == 0, f"{name}: {len(bad)} codes differ, first at {bad[0]}: {g[tuple(bad[0])]} vs {r[tuple(bad[0])]}"
    if gstate is not None:
        assert np.array_equal(gstate, ref_state)
    return ref, ref_state


def test_codes_bit_exact_small_layer(gpu_lib):
    """Several channel blocks, several segments and a ragged last one; all three outputs and the state."""
    s = W.CONFIGS["m2_130m"].with_(batch=2, seqlen=77)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=1, calib_tokens=256)
    inp = make_conv_inputs(s, seed=1)
    ref, _ = _check(gpu_lib, s, sc, inp)
    assert len(np.unique(ref)) > 120 and (ref == 127).any()


def test_8b_shape_with_carried_state_in_pieces(gpu_lib):
    """The 8B layer's 10240 channels; a sequence run at once equals the same sequence run in pieces (decode-sized ones
    too) through the carried state, and both equal the oracle."""
    s = W.CONFIGS["m2_8b_b1"].with_(batch=2, seqlen=150)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=2, calib_tokens=256)
    inp = make_conv_inputs(s, seed=2)
    ref, ref_state = _check(gpu_lib, s, sc, inp)
    state = None
    for lo, hi in [(0, 1), (1, 3), (3, 64), (64, 149), (149, 150)]:
        piece = dict(inp, xBC=np.ascontiguousarray(inp["xBC"][:, lo:hi]))
        r, state = _check(gpu_lib, s, sc, piece, state)
        assert np.array_equal(r, ref[:, lo:hi])
    assert np.array_equal(state, ref_state)


def test_many_elements_against_the_exact_sequence(gpu_lib):
    """21 million outputs compared one by one.  The kernel takes most codes from the hardware's approximate exponential
    and reciprocal and falls back to the stated exact sequence wherever the two could round differently; a bound that
    was too optimistic would show here as single codes off by one."""
    s = W.CONFIGS["m2_8b_b1"].with_(batch=2, seqlen=1024)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=12, calib_tokens=256)
    inp = make_conv_inputs(s, seed=12)
    ref, _ = _check(gpu_lib, s, sc, inp)
    assert len(np.unique(ref)) > 200


def test_decode_step_updates_state_in_place(gpu_lib):
    s = W.CONFIGS["m2_8b_decode"].with_(batch=5, seqlen=1)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=3, calib_tokens=256)
    Ct = s.nheads * s.headdim + 2 * s.ngroups * s.d_state
    state = np.random.default_rng(3).integers(-128, 128, size=(5, 3, Ct), dtype=np.int8)
    for step in range(4):
        inp = make_conv_inputs(s, seed=3, stream=60 + step)
        _, state = _check(gpu_lib, s, sc, inp, state, alias=True)


@pytest.mark.parametrize("batch,H,P,N,m,n,state", [(1, 24, 64, 128, 4, 4, True), (3, 6, 16, 16, 3, 6, True),
                                                   (5, 5, 48, 32, 1, 1, False), (1030, 8, 64, 128, 2, 3, True)])
def test_one_token_kernel(gpu_lib, batch, H, P, N, m, n, state):
    """One token per sequence: channel counts that fill no whole wave, cluster counts on both sides of the four that are
    looked up at once, no carried state, several sequences per thread (1030 x 768 channels) with a ragged last group."""
    s = W.LayerShape("step", batch, 1, H, P, N, 1, 16, m, n)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=13, calib_tokens=128)
    Ct = H * P + 2 * N
    st = np.random.default_rng(13).integers(-128, 128, size=(batch, 3, Ct), dtype=np.int8) if state else None
    _check(gpu_lib, s, sc, make_conv_inputs(s, seed=13), st, alias=state)


@pytest.mark.parametrize("batch,L,H,P,N,m,n", [(2, 2, 24, 64, 128, 4, 4),      # shorter than the halo
                                               (1, 45, 6, 16, 16, 3, 6),       # six ranges; segments of 4, a last one of 1
                                               (9, 291, 6, 64, 128, 2, 3),     # ... a last one of 3
                                               (15, 900, 6, 64, 16, 2, 3),     # segments of 8, the last of 4
                                               (16, 3085, 14, 64, 64, 2, 2),   # segments of 32, the last of 13
                                               (64, 3085, 4, 16, 16, 2, 2)])   # one channel block, the last of 13
def test_segments_and_carried_state(gpu_lib, batch, L, H, P, N, m, n):
    """Short and the longest segments of the vector kernel, with ragged last ones, from a carried state.  (Longer ones
    than 8 tokens from 6144 waves of 8 up, 32 where 28 still make more than 6144.)"""
    s = W.LayerShape("seg", batch, L, H, P, N, 1, 16, m, n)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=14, calib_tokens=128)
    st = np.random.default_rng(14).integers(-128, 128, size=(batch, 3, H * P + 2 * N), dtype=np.int8)
    _check(gpu_lib, s, sc, make_conv_inputs(s, seed=14), st)


@pytest.mark.parametrize("batch,L,H,P,N,m,n,bias", [(64, 2049, 6, 48, 16, 3, 7, True),   # ranges that end inside a thread
                                                    (16, 4096, 18, 64, 32, 1, 1, False)])  # a second, ragged block; no bias
def test_channel_ranges_and_blocks_of_large_calls(gpu_lib, batch, L, H, P, N, m, n, bias):
    """Segments of 32 tokens: more channel ranges than four, ends of ranges inside the channels of a
    thread, no bias, and a channel block that fills no whole wave."""
    s = W.LayerShape("wide", batch, L, H, P, N, 1, 16, m, n)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=16, calib_tokens=128)
    if n > 1:
        assert (np.asarray(sc.chan_cluster_end) % 16 != 0).any()
    inp = make_conv_inputs(s, seed=16)
    st = np.random.default_rng(16).integers(-128, 128, size=(batch, 3, H * P + 2 * N), dtype=np.int8) if bias else None
    _check(gpu_lib, s, sc, inp if bias else dict(inp, bias=None), st)


@pytest.mark.parametrize("L,scale,bias,s_in", [
    (1531, 1.0, 1.0, 1.0),       # segments of 16 tokens, the last of 11
    (1150, 1.0, 30.0, 1.0),      # of 12, the last of 10; large biases
    (2301, 1e-3, 1.0, 1e-3),     # of 24, the last of 21; small outputs: a wider margin around the rounding boundaries
    (45, 1e-4, 100.0, 1.0),      # a margin of most of a code
    (45, 1e-9, 1.0, 1.0),        # wider than a code: the exact sequence throughout
    (45, 1e-3, 0.0, 1e36)])      # constants beyond the range of fp32
def test_margin_around_the_rounding_boundaries(gpu_lib, L, scale, bias, s_in):
    """The codes are the exact sequence's whatever the constants the fast evaluation's error bound depends on."""
    s = W.LayerShape("margin", 64, L, 4, 16, 16, 1, 16, 2, 2)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=17, calib_tokens=128)
    for name in ("x_scales", "B_scales", "C_scales"):
        setattr(sc, name, (np.asarray(getattr(sc, name)) * np.float32(scale)).astype(np.float32))
    inp = make_conv_inputs(s, seed=17)
    _check(gpu_lib, s, sc, dict(inp, bias=inp["bias"] * np.float32(bias),
                                in_w_scale=float(np.float32(inp["in_w_scale"] * s_in))))


def test_large_call_is_its_sequences(gpu_lib):
    """More codes than are left in the caches (96 MiB) against calls of a few of the sequences, codes bit for bit."""
    import torch
    s = W.CONFIGS["m2_130m"].with_(batch=16, seqlen=4001)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=18, calib_tokens=128)
    inp = make_conv_inputs(s.with_(batch=1, seqlen=8), seed=18)
    dsc = gpu_lib.DeviceScales(host_scales(gpu_lib, sc))
    Ct = inp["xBC"].shape[2]
    assert 16 * 4001 * Ct > 96 << 20
    g = torch.Generator(device="cuda").manual_seed(18)
    x = torch.randint(-128, 128, (16, 4001, Ct), generator=g, device="cuda", dtype=torch.int8)
    w, bias = torch.from_numpy(inp["weight"]).cuda(), torch.from_numpy(inp["bias"]).cuda()

    def run(part):
        b = part.shape[0]
        out = [torch.full((b, 4001, h, p), 99, dtype=torch.int8, device="cuda")
               for h, p in ((s.nheads, s.headdim), (s.ngroups, s.d_state), (s.ngroups, s.d_state))]
        out.append(torch.full((b, 3, Ct), 99, dtype=torch.int8, device="cuda"))
        gpu_lib.quamba_conv1d_q8(to_shape(gpu_lib, s.with_(batch=b)), dsc, part, w, bias, inp["in_w_scale"], *out[:3],
                                 conv_state_out=out[3])
        return out
    whole, parts = run(x), [run(x[i:i + 4].contiguous()) for i in range(0, 16, 4)]
    for i, t in enumerate(whole):
        assert torch.equal(t, torch.cat([p[i] for p in parts]))


@pytest.mark.parametrize("L", [2, 7, 16])
def test_short_sequence_with_one_buffer_as_both_states(gpu_lib, L):
    s = W.CONFIGS["m2_130m"].with_(batch=3, seqlen=L)
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=15, calib_tokens=128)
    Ct = s.nheads * s.headdim + 2 * s.ngroups * s.d_state
    st = np.random.default_rng(15).integers(-128, 128, size=(3, 3, Ct), dtype=np.int8)
    _check(gpu_lib, s, sc, make_conv_inputs(s, seed=15), st, alias=True)


def test_no_bias_no_state_output(gpu_lib):
    s = W.CONFIGS["m2_130m"].with_(batch=1, seqlen=40)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=4, calib_tokens=256)
    inp = dict(make_conv_inputs(s, seed=4), bias=None)
    _check(gpu_lib, s, sc, inp, want_state=False)


def test_any_shape_kernel_odd_sizes_and_unaligned_input(gpu_lib):
    """headdim and d_state that are no multiples of 16, and a 16-friendly shape whose input starts 1 byte off."""
    s = W.LayerShape("odd", 2, 45, 6, 20, 24, 2, 16, 2, 2)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=5, calib_tokens=128)
    st = np.random.default_rng(5).integers(-128, 128, size=(2, 3, 6 * 20 + 2 * 2 * 24), dtype=np.int8)
    _check(gpu_lib, s, sc, make_conv_inputs(s, seed=5), st)
    s2 = W.CONFIGS["m2_130m"].with_(batch=1, seqlen=33)
    sc2, _, _ = make_problem(s2.with_(seqlen=8), seed=6, calib_tokens=256)
    _check(gpu_lib, s2, sc2, make_conv_inputs(s2, seed=6), offset=1)


@pytest.mark.parametrize("L", [1, 5])
@pytest.mark.parametrize("G,H,P,N", [(1, 8, 65552, 16), (4, 262160, 16, 16), (8, 8, 16, 65552)])
def test_widest_heads_and_groups(gpu_lib, G, H, P, N, L):
    """Heads of more than 2^16 channels, groups of as many heads or states: by the rounded-up reciprocal alone some channels' head or
    group is one too high.  Four channels to a thread all the same."""
    d = max(P, N, H // G)
    step = 1 if d == H // G else 4
    c = np.arange(0, (H if step == 1 else 8 * d), step)
    assert ((c * -(-2**32 // d) >> 32) != c // d).any()
    s = W.LayerShape("wide", 1, L, H, P, N, G, 16, 1, 2 if G == 1 else 1)
    takes = gpu_lib.load_library()._ZN6quamba26conv1d_takes_four_channelsERK18quamba_ssd_shape_t
    takes.restype = C.c_bool
    assert takes(C.byref(to_shape(gpu_lib, s)))
    g = np.random.default_rng(H + L)
    Ct = H * P + 2 * G * N
    scales = lambda: np.float32(0.01) * (1 + np.arange(G, dtype=np.float32))
    sc = oracle.Scales(1, 1, scales(), np.full(G, H // G, np.int32), np.full(G, P, np.int32), scales(), scales())
    if G == 1:  # ... nor its place in the head
        sc = oracle.Scales(1, 2, np.float32([0.01, 0.03]), sc.head_cluster_end, np.array([P - 3, P], np.int32), sc.B_scales, sc.C_scales)
    inp = {"xBC": g.integers(-127, 128, (1, L, Ct), dtype=np.int8), "weight": g.integers(-127, 128, (Ct, 4), dtype=np.int8),
           "bias": g.standard_normal(Ct).astype(np.float32), "in_w_scale": 1e-4}
    _check(gpu_lib, s, sc, inp, g.integers(-128, 128, (1, 3, Ct), dtype=np.int8))


def test_extreme_codes_and_saturation(gpu_lib):
    """All-extreme inputs and filters: the largest window sums (4 * 128 * 128), both signs, deep exp underflow."""
    s = W.CONFIGS["m2_130m"].with_(batch=1, seqlen=35)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=7, calib_tokens=256)
    Ct = s.nheads * s.headdim + 2 * s.ngroups * s.d_state
    g = np.random.default_rng(7)
    inp = {"xBC": g.choice(np.array([-128, 127], np.int8), size=(1, 35, Ct)),
           "weight": g.choice(np.array([-128, 127], np.int8), size=(Ct, 4)),
           "bias": (g.standard_normal(Ct) * 5).astype(np.float32), "in_w_scale": 3e-3}
    ref, _ = _check(gpu_lib, s, sc, inp)
    assert (ref == 127).any() and (ref <= 0).any()


def test_rejects_aliased_state_on_long_sequences(gpu_lib):
    import torch
    s = W.CONFIGS["m2_130m"].with_(batch=1, seqlen=64)
    sc, _, _ = make_problem(s.with_(seqlen=8), seed=8, calib_tokens=128)
    inp = make_conv_inputs(s, seed=8)
    Ct = inp["xBC"].shape[2]
    with pytest.raises(gpu_lib.QuambaError):
        _gpu(gpu_lib, s, sc, inp, np.zeros((1, 3, Ct), np.int8), alias=True)


def test_bench_size_sampled_tokens(gpu_lib):
    """The bench launch (4 x 4096 tokens x 10240 channels): tokens sampled over the launch checked bit for bit; the
    oracle recomputes each sampled token from its own 4-token window."""
    import torch
    s = W.CONFIGS["m2_8b_b4"]
    sc, _, _ = make_problem(s.with_(batch=1, seqlen=8), seed=9, calib_tokens=256)
    inp = make_conv_inputs(s, seed=9)
    gx, gB, gC, gstate = _gpu(gpu_lib, s, sc, inp)
    got = np.concatenate([gx.reshape(s.batch, s.seqlen, -1), gB.reshape(s.batch, s.seqlen, -1),
                          gC.reshape(s.batch, s.seqlen, -1)], axis=2)
    os_ = oracle.output_scales(sc, s.nheads, s.headdim, s.ngroups, s.d_state)
    for t in [0, 1, 2, 3, 31, 32, 33, 1000, 2047, 2048, 4064, 4095]:
        lo = max(0, t - 3)
        win = np.ascontiguousarray(inp["xBC"][:, lo:t + 1])
        ref, _ = oracle.ref_conv1d_q8(win, inp["weight"], inp["in_w_scale"], inp["bias"], os_)
        assert np.array_equal(got[:, t], ref[:, -1]), f"token {t}"
    assert np.array_equal(gstate, inp["xBC"][:, -3:])
    assert not (got == 99).all(axis=2).any()
