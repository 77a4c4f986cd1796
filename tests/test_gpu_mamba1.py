"""GPU parity of the 8-bit Mamba1 selective scan (quamba_mamba1_scan, quamba_mamba1_decode_step) against the fp64
oracle, through the C ABI: y within 2e-3 of the largest |y| (fp32 scan, fp16 output), states within 1e-4."""
import ctypes as C

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import make_mamba1_problem, make_mamba1_gate, host_scales

pytestmark = pytest.mark.gpu

Y_TOL = 2e-3
S_TOL = 1e-4


def _shape(q, b, D, N, L, nranges, flags=0):
    return q.Shape(batch=b, seqlen=L, nheads=1, headdim=D, d_state=N, ngroups=1, chunk=1, n_head_clusters=1,
                   n_chan_clusters=nranges, flags=flags)


def _form(q, b, D, N, L, flags=0):
    """The kernel that the library chooses for a scan on this device (Mamba1Form in csrc/quamba_internal.h)."""
    f = q.load_library()._ZN6quamba16mamba1_scan_formERK18quamba_ssd_shape_t
    return ["any", "16 lanes", "32 lanes", "64 lanes", "8 channels", "24 channels", "halves"][f(C.byref(_shape(q, b, D, N, L, 4, flags)))]


def _run(q, sc, p, b, D, N, L, nranges=4, flags=0, init=None, with_D=True, want_state=True):
    import torch
    shape = _shape(q, b, D, N, L, nranges, flags)
    dsc = q.DeviceScales(host_scales(q, sc))
    t = {k: torch.from_numpy(np.ascontiguousarray(p[k])).cuda() for k in ("x", "B", "C", "dt", "A", "D")}
    y = torch.full((b, D, L), float("nan"), dtype=torch.float16, device="cuda")
    fin = torch.full((b, D, N), float("nan"), device="cuda") if want_state else None
    ini = None if init is None else torch.from_numpy(init.astype(np.float32)).cuda()
    q.quamba_mamba1_scan(shape, dsc, t["x"], t["B"], t["C"], t["dt"], t["A"], t["D"] if with_D else None, y,
                         init_state=ini, final_state=fin)
    return y.cpu().numpy().astype(np.float64), None if fin is None else fin.cpu().numpy().astype(np.float64)


def _check(q, b, D, N, L, seed, nranges=4, flags=0, with_init=False, with_D=True):
    sc, p = make_mamba1_problem(b, D, N, L, seed, nranges)
    init = np.random.default_rng(seed).normal(0, 0.05, size=(b, D, N)).astype(np.float32) if with_init else None
    yref, sref = oracle.ref_mamba1_scan(p["xs"], sc.B_scales[0], sc.C_scales[0], p["x"], p["B"], p["C"], p["dt"], p["A"],
                                        p["D"] if with_D else None, init)
    y, fin = _run(q, sc, p, b, D, N, L, nranges, flags, init, with_D)
    assert np.isfinite(y).all() and np.isfinite(fin).all()
    ey = np.abs(y - yref).max() / np.abs(yref).max()
    es = np.abs(fin - sref).max() / np.abs(sref).max()
    assert ey <= Y_TOL, f"y error {ey:.3e}"
    assert es <= S_TOL, f"state error {es:.3e}"
    return ey, es


def test_wave_scan_kernel_several_tiles_and_a_ragged_one(gpu_lib):
    """2608 tokens = five full tiles of 512 (32 lanes) and one of 48; channels not a multiple of the 16 a workgroup owns
    (lanes of the last workgroup without a channel)."""
    ey, es = _check(gpu_lib, b=2, D=8198, N=16, L=2608, seed=1, with_init=True)
    print(f"mamba1 scan, 8198 channels x 2608 tokens: y {ey:.2e} state {es:.2e}")


def test_wave_scan_kernel_small_shapes(gpu_lib):
    """One workgroup per compute unit is all there is: tiles of 1024 tokens (64 lanes), and one tile of 16."""
    ey, es = _check(gpu_lib, b=1, D=203, N=16, L=1040, seed=2)
    print(f"mamba1 scan, 203 channels x 1040 tokens: y {ey:.2e} state {es:.2e}")
    _check(gpu_lib, b=3, D=64, N=16, L=16, seed=3, with_init=True, with_D=False)       # one lane of tokens


@pytest.mark.parametrize("D,L", [(40, 15), (33, 16), (37, 17), (70, 255), (40, 256), (33, 257), (40, 511), (16, 512),
                                 (20, 513), (9, 1023), (9, 1025), (2060, 1037), (8177, 700)])
def test_sequence_lengths_around_lanes_and_tiles(gpu_lib, D, L):
    """Rows that start at any byte and end inside a lane's 16 tokens, on every tile width: one token less and more than a
    lane (16), and than a tile of 16, 32 and 64 lanes; 2060 channels give the 32-lane kernel with workgroups of 24
    channels several tiles, 8177 of 700 tokens the 16-lane kernel."""
    _check(gpu_lib, b=2, D=D, N=16, L=L, seed=L, with_init=L % 2 == 1, with_D=L % 3 != 0)


def test_any_shape_kernel_and_cross_check(gpu_lib):
    _check(gpu_lib, b=2, D=70, N=16, L=45, seed=4, with_init=True, flags=gpu_lib.FLAG_GENERIC_KERNEL)  # forced, odd length
    _check(gpu_lib, b=1, D=33, N=24, L=64, seed=5, nranges=3)                           # other d_state
    _check(gpu_lib, b=1, D=130, N=16, L=256, seed=6, flags=gpu_lib.FLAG_GENERIC_KERNEL)  # forced, fast-path shape


def test_pieces_through_the_state_equal_one_run(gpu_lib):
    import torch
    b, D, N, L = 2, 256, 16, 2048
    sc, p = make_mamba1_problem(b, D, N, L, seed=7)
    y_all, s_all = _run(gpu_lib, sc, p, b, D, N, L)
    st = None
    ys = []
    for lo, hi in [(0, 1024), (1024, 1040), (1040, 2048)]:
        piece = dict(p, **{k: np.ascontiguousarray(p[k][:, :, lo:hi]) for k in ("x", "B", "C", "dt")})
        y, st = _run(gpu_lib, sc, piece, b, D, N, hi - lo, init=st)
        ys.append(y)
    yp = np.concatenate(ys, axis=2)
    scale = np.abs(y_all).max()
    assert np.abs(yp - y_all).max() <= 2 * 4.9e-4 * scale              # two fp16 roundings of nearly equal fp32 values
    assert np.abs(st - s_all).max() <= 1e-5 * np.abs(s_all).max()


def test_limits(gpu_lib):
    """dt = 0: y = D x exactly to fp16 rounding and the state does not move; strong decay: y -> dt C.B x + D x."""
    b, D, N, L = 1, 128, 16, 1024
    sc, p = make_mamba1_problem(b, D, N, L, seed=8)
    p0 = dict(p, dt=np.zeros_like(p["dt"]))
    init = np.random.default_rng(8).normal(0, 1, size=(b, D, N)).astype(np.float32)
    y, fin = _run(gpu_lib, sc, p0, b, D, N, L, init=np.zeros_like(init))
    want = (p["D"].astype(np.float64)[None, :, None] * p["x"] * p["xs"].astype(np.float64)[None, :, None]).astype(np.float16)
    assert np.array_equal(y.astype(np.float16), want) and not fin.any()
    _, fin2 = _run(gpu_lib, sc, dict(p0, D=np.zeros_like(p["D"])), b, D, N, L, init=init)
    assert np.array_equal(fin2.astype(np.float32), init)


def test_2p8b_shape_sampled(gpu_lib):
    """The Mamba1-2.8B-shaped layer the bench times (5120 channels, 16 states, 4 x 4096 tokens): the oracle scans 24
    sampled channels of every sequence in full."""
    import torch
    b, D, N, L = 4, 5120, 16, 4096
    sc, p = make_mamba1_problem(b, D, N, L, seed=9)
    y, fin = _run(gpu_lib, sc, p, b, D, N, L)
    pick = np.unique(np.concatenate([np.arange(0, D, 223), [D - 1, D - 2, 1]]))
    yref, sref = oracle.ref_mamba1_scan(p["xs"][pick], sc.B_scales[0], sc.C_scales[0], p["x"][:, pick], p["B"], p["C"],
                                        p["dt"][:, pick], p["A"][pick], p["D"][pick])
    ey = np.abs(y[:, pick] - yref).max() / np.abs(yref).max()
    es = np.abs(fin[:, pick] - sref).max() / np.abs(sref).max()
    assert ey <= Y_TOL and es <= S_TOL, (ey, es)
    assert np.isfinite(y).all()
    print(f"mamba1 scan 2.8B shape: y {ey:.2e} state {es:.2e}")


def test_decode_steps(gpu_lib):
    import torch
    q = gpu_lib
    for (b, D, N) in [(5, 5120, 16), (7, 203, 16), (3, 77, 24)]:  # 203: a last workgroup with idle lanes
        sc, p = make_mamba1_problem(b, D, N, 6, seed=10)
        shape = _shape(q, b, D, N, 1, 4)
        dsc = q.DeviceScales(host_scales(q, sc))
        st_ref = np.random.default_rng(10).normal(0, 0.1, size=(b, D, N))
        st = torch.from_numpy(st_ref.astype(np.float32)).cuda()
        st_ref = st_ref.astype(np.float32).astype(np.float64)
        A, Dk = torch.from_numpy(p["A"]).cuda(), torch.from_numpy(p["D"]).cuda()
        y = torch.empty((b, D), dtype=torch.float16, device="cuda")
        for t in range(6):
            sl = {k: np.ascontiguousarray(p[k][:, :, t]) for k in ("x", "B", "C", "dt")}
            q.quamba_mamba1_decode_step(shape, dsc, *(torch.from_numpy(sl[k]).cuda() for k in ("x", "B", "C", "dt")),
                                        A, Dk, st, y)
            yref, st_ref = oracle.ref_mamba1_scan(p["xs"], sc.B_scales[0], sc.C_scales[0], sl["x"][:, :, None],
                                                  sl["B"][:, :, None], sl["C"][:, :, None], sl["dt"][:, :, None], p["A"],
                                                  p["D"], st_ref)
            ey = np.abs(y.cpu().numpy().astype(np.float64) - yref[:, :, 0]).max() / np.abs(yref).max()
            es = np.abs(st.cpu().numpy().astype(np.float64) - st_ref).max() / np.abs(st_ref).max()
            assert ey <= Y_TOL and es <= S_TOL, (t, ey, es)


def _gate(q, g, use_z, use_dt, sl=None):
    import torch
    pick = (lambda v: torch.from_numpy(np.ascontiguousarray(v if sl is None else v[:, :, sl])).cuda())
    return q.Gate(z=pick(g["z"]) if use_z else None, z_scale=g["z_scale"] if use_z else 0.0,
                  dt_q=pick(g["dt_q"]) if use_dt else None, dt_scale=g["dt_scale"] if use_dt else 0.0,
                  dt_bias=torch.from_numpy(g["dt_bias"]).cuda() if use_dt else None)


def _dt_of_codes(g):
    """The oracle's softplus takes the bias along the last axis: channels last, then back to time last."""
    return np.moveaxis(oracle.dt_from_codes(np.moveaxis(g["dt_q"], 1, -1), g["dt_scale"], g["dt_bias"]), -1, 1)


@pytest.mark.parametrize("use_z,use_dt", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("b,D,N,L,flags", [(2, 203, 16, 2608, 0),    # 64 lanes per channel, several tiles
                                           (2, 70, 16, 45, 0),       # 16 lanes, one tile
                                           (2, 8177, 16, 700, 0),    # 16 lanes, several tiles
                                           (2, 2060, 16, 1037, 0),   # 32 lanes, 24 channels
                                           (2, 8198, 16, 1029, 0),   # 32 lanes, 16 channels
                                           (2, 8198, 16, 1301, 0),   # ... and 64 lanes behind, several tiles of both
                                           (1, 33, 24, 64, 0),       # any shape
                                           (1, 130, 16, 256, 1)])    # ... forced
def test_scan_with_side_inputs(gpu_lib, b, D, N, L, flags, use_z, use_dt):
    """Step size from int8 codes of its pre-activation plus a per-channel bias, and / or the output gate on int8 z
    (Section 3.2), on every width of the wave-scan kernel (several tiles and a ragged one, rows that start at odd
    addresses) and the any-shape kernel: the oracle's scan on the oracle's own step size, followed by the oracle's gate.
    Of the larger layers the oracle scans channels sampled over the workgroups."""
    import torch
    q = gpu_lib
    sc, p = make_mamba1_problem(b, D, N, L, seed=11)
    g = make_mamba1_gate(b, D, L, seed=11)
    dt_ref = _dt_of_codes(g).astype(np.float32) if use_dt else p["dt"]
    init = np.random.default_rng(11).normal(0, 0.05, size=(b, D, N)).astype(np.float32)
    pick = np.arange(D) if D < 2048 else np.unique(np.r_[0:16, np.arange(0, D, 61), D - 16:D])
    yref, sref = oracle.ref_mamba1_scan(p["xs"][pick], sc.B_scales[0], sc.C_scales[0], p["x"][:, pick], p["B"], p["C"],
                                        dt_ref[:, pick], p["A"][pick], p["D"][pick], init[:, pick])
    if use_z:
        yref = oracle.silu_gate(yref, g["z"][:, pick], g["z_scale"])
    t = {k: torch.from_numpy(np.ascontiguousarray(p[k])).cuda() for k in ("x", "B", "C", "dt", "A", "D")}
    y = torch.full((b, D, L), float("nan"), dtype=torch.float16, device="cuda")
    fin = torch.full((b, D, N), float("nan"), device="cuda")
    q.quamba_mamba1_scan(_shape(q, b, D, N, L, 4, flags), q.DeviceScales(host_scales(q, sc)), t["x"], t["B"], t["C"],
                         None if use_dt else t["dt"], t["A"], t["D"], y, init_state=torch.from_numpy(init).cuda(),
                         final_state=fin, gate=_gate(q, g, use_z, use_dt))
    yg, sg = y.cpu().numpy().astype(np.float64), fin.cpu().numpy().astype(np.float64)
    assert np.isfinite(yg).all() and np.isfinite(sg).all()
    ey = np.abs(yg[:, pick] - yref).max() / np.abs(yref).max()
    es = np.abs(sg[:, pick] - sref).max() / np.abs(sref).max()
    print(f"mamba1 scan D={D} L={L} flags={flags} z={use_z} dt_q={use_dt}: y {ey:.2e} state {es:.2e}")
    assert ey <= Y_TOL and es <= S_TOL


def test_decode_steps_with_side_inputs(gpu_lib):
    import torch
    q = gpu_lib
    for (b, D, N) in [(5, 5120, 16), (7, 203, 16), (3, 77, 24)]:  # 203: a last workgroup with idle lanes
        sc, p = make_mamba1_problem(b, D, N, 4, seed=12)
        g = make_mamba1_gate(b, D, 4, seed=12)
        dt_all = _dt_of_codes(g).astype(np.float32)
        shape = _shape(q, b, D, N, 1, 4)
        dsc = q.DeviceScales(host_scales(q, sc))
        st_ref = np.random.default_rng(12).normal(0, 0.1, size=(b, D, N)).astype(np.float32)
        st = torch.from_numpy(st_ref).cuda()
        st_ref = st_ref.astype(np.float64)
        A, Dk = torch.from_numpy(p["A"]).cuda(), torch.from_numpy(p["D"]).cuda()
        y = torch.empty((b, D), dtype=torch.float16, device="cuda")
        for t in range(4):
            sl = {k: np.ascontiguousarray(p[k][:, :, t]) for k in ("x", "B", "C")}
            q.quamba_mamba1_decode_step(shape, dsc, *(torch.from_numpy(sl[k]).cuda() for k in ("x", "B", "C")), None,
                                        A, Dk, st, y, gate=_gate(q, g, True, True, sl=t))
            yref, st_ref = oracle.ref_mamba1_scan(p["xs"], sc.B_scales[0], sc.C_scales[0], sl["x"][:, :, None],
                                                  sl["B"][:, :, None], sl["C"][:, :, None], dt_all[:, :, t:t + 1],
                                                  p["A"], p["D"], st_ref)
            yref = oracle.silu_gate(yref[:, :, 0], g["z"][:, :, t], g["z_scale"])
            ey = np.abs(y.cpu().numpy().astype(np.float64) - yref).max() / np.abs(yref).max()
            es = np.abs(st.cpu().numpy().astype(np.float64) - st_ref).max() / np.abs(st_ref).max()
            assert ey <= Y_TOL and es <= S_TOL, (t, ey, es)


def test_step_size_codes_to_fp32_accuracy(gpu_lib):
    """Every step-size code once, A = 0 and one non-zero token per channel: a state is dt x B.  dt is within three units of
    2^-24 (its own two roundings, exponential and logarithm of one unit), and three products follow: 6 * 2^-24 of the
    value.  The pre-activations code / 16 are exact and run from -8 to 8; both the wave-scan kernel and the one-thread kernel."""
    import torch
    q = gpu_lib
    D, N, L = 256, 16, 37
    one = np.ones(1, np.float32)
    sc = q.DeviceScales(q.HostScales(np.full(4, 0.37, np.float32), np.array([1], np.int32),
                                     np.array([64, 128, 192, 256], np.int32), 0.11 * one, one))
    x = np.zeros((1, D, L), np.int8)
    x[0, np.arange(D), np.arange(D) % L] = 101
    codes = np.ascontiguousarray(np.broadcast_to(np.arange(-128, 128, dtype=np.int8)[None, :, None], (1, D, L)))
    B = np.full((1, N, L), 93, np.int8)
    v = np.arange(-128, 128) / 16.0
    want = np.logaddexp(0.0, v) * (101 * np.float64(np.float32(0.37))) * (93 * np.float64(np.float32(0.11)))
    for flags in (0, q.FLAG_GENERIC_KERNEL):
        fin = torch.full((1, D, N), float("nan"), device="cuda")
        q.quamba_mamba1_scan(_shape(q, 1, D, N, L, 4, flags), sc, torch.from_numpy(x).cuda(), torch.from_numpy(B).cuda(),
                             torch.from_numpy(B).cuda(), None, torch.zeros(D, N, device="cuda"), None,
                             torch.empty((1, D, L), dtype=torch.float16, device="cuda"), final_state=fin,
                             gate=q.Gate(dt_q=torch.from_numpy(codes).cuda(), dt_scale=1.0 / 16))
        err = np.abs(fin.cpu().numpy().astype(np.float64)[0] / want[:, None] - 1.0).max()
        print(f"step sizes, flags {flags}: {err / 2 ** -24:.2f} units of 2^-24")
        assert err <= 6 * 2.0 ** -24


@pytest.mark.parametrize("D,L", [(40, 37), (40, 300), (9, 1100), (2060, 1037), (8177, 700)])
def test_infinite_and_zero_states(gpu_lib, D, L):
    """On every width of the scan: an infinite state stays infinite as long as no single decay is zero, also where the
    product over several tokens underflows (exp(-8) per token); a state of zero without inputs stays zero where that
    product overflows (A > 0)."""
    b, N = 2, 16
    sc, p = make_mamba1_problem(b, D, N, L, seed=L)
    p = dict(p, dt=np.full_like(p["dt"], 0.5), A=np.full_like(p["A"], -16.0), C=np.where(p["C"] == 0, np.int8(1), p["C"]))
    init = np.random.default_rng(L).normal(0, 0.1, size=(b, D, N)).astype(np.float32)
    init[0, 3, 2], init[1, D - 1, 15] = np.inf, -np.inf
    pick = np.unique(np.r_[0:9, D - 9:D])
    yref, sref = oracle.ref_mamba1_scan(p["xs"][pick], sc.B_scales[0], sc.C_scales[0], p["x"][:, pick], p["B"], p["C"],
                                        p["dt"][:, pick], p["A"][pick], p["D"][pick], init[:, pick])
    y, fin = _run(gpu_lib, sc, p, b, D, N, L, init=init)
    for got, ref, tol in ((y[:, pick], yref, Y_TOL), (fin[:, pick], sref, S_TOL)):
        inf = np.isinf(ref)
        assert inf.any() and np.array_equal(got[inf], ref[inf])
        assert np.abs(got[~inf] - ref[~inf]).max() <= tol * np.abs(ref[~inf]).max()
    assert np.isinf(fin).sum() == 2 and not np.isnan(fin).any() and not np.isnan(y).any()

    p = dict(p, A=-p["A"], x=np.zeros_like(p["x"]))
    y, fin = _run(gpu_lib, sc, p, b, D, N, L)
    assert not y.any() and not fin.any()


@pytest.mark.parametrize("L", [37, 300, 1100])
def test_states_that_forget_everything_at_a_ragged_end(gpu_lib, L):
    """A = -inf (exp(A_log) overflows): every token's decay is zero, so the state is the last token's input alone, whatever
    fills the lanes behind the end of the sequence."""
    b, D, N = 1, 40, 16
    sc, p = make_mamba1_problem(b, D, N, L, seed=L)
    p["A"][::3, 5] = -np.inf
    with np.errstate(invalid="ignore"):
        yref, sref = oracle.ref_mamba1_scan(p["xs"], sc.B_scales[0], sc.C_scales[0], p["x"], p["B"], p["C"], p["dt"], p["A"],
                                            p["D"])
    assert (p["dt"] > 0).all() and np.isfinite(sref).all()
    y, fin = _run(gpu_lib, sc, p, b, D, N, L)
    assert np.abs(y - yref).max() <= Y_TOL * np.abs(yref).max()
    assert np.abs(fin - sref).max() <= S_TOL * np.abs(sref).max()


@pytest.mark.parametrize("b,D,L,form", [(1, 2085, 520, "halves"),    # no whole group, more than half a unit's worth of halves, the last one empty
                                        (1, 4096, 1024, "halves"),   # ... as many groups as compute units
                                        (3, 2736, 513, "halves"),    # two groups per unit and one: two halves behind them
                                        (3, 4090, 900, "halves"),    # ... and a group per unit
                                        (1, 8192, 600, "16 lanes"),  # two groups per unit, whose tiles of 512 tokens would be half empty
                                        (1, 8192, 1000, "32 lanes"),  # ... and would not, no halves
                                        (3, 1537, 600, "24 channels"),  # the last workgroup with one
                                        (4, 1536, 513, "24 channels"),  # as many workgroups as compute units
                                        (2, 6400, 900, "8 channels")])  # 8 states at a time
@pytest.mark.parametrize("sides", [False, True])
def test_how_channels_are_shared_out(gpu_lib, b, D, L, form, sides):
    """Groups of 16 channels, those behind the last full round as halves of 8 channels on 64 lanes each, and workgroups of 24 and
    of 8 channels, at the edges of their rules on 256 compute units, at the same bars."""
    assert _form(gpu_lib, b, D, 16, L) == form
    test_scan_with_side_inputs(gpu_lib, b, D, 16, L, 0, sides, sides)


@pytest.mark.parametrize("b,D,L,form", [(2, 5120, 1003, "halves"), (2, 5120, 4096, "halves"), (6, 1536, 1003, "halves"),
                                        (6, 1536, 2561, "halves"), (2, 1536, 4096, "halves"), (3, 5120, 600, "16 lanes"),
                                        (3, 4099, 1537, "8 channels"), (2, 6400, 1003, "8 channels"), (3, 1537, 700, "24 channels")])
@pytest.mark.parametrize("infinite", [False, True])
def test_equal_sequences_of_one_call_have_equal_results(gpu_lib, b, D, L, form, infinite):
    """Sequences with the same inputs have the same outputs and final states, bit for bit, also where a launch takes some groups of
    channels on 32 lanes each and the others on 64: with small steps, whose states carry far over the ends of the tiles, and with
    infinite initial states in some channels, which leave their neighbours' results as they are."""
    import torch
    q = gpu_lib
    assert _form(q, b, D, 16, L) == form
    g = torch.Generator(device="cuda").manual_seed(D + L)
    codes = lambda *s: torch.randint(-128, 128, s, generator=g, device="cuda", dtype=torch.int8)
    rand = lambda *s: torch.rand(s, generator=g, device="cuda")
    sc, _ = make_mamba1_problem(1, D, 16, 16, seed=3)
    x, B, Cm, dt, init = codes(1, D, L), codes(1, 16, L), codes(1, 16, L), 0.006 * rand(1, D, L), rand(1, D, 16) - 0.5
    if infinite:
        init[0, ::37, 5] = float("inf")
        init[0, 5::74, 11] = -float("inf")
    x, B, Cm, dt, init = (v.expand(b, *v.shape[1:]).contiguous() for v in (x, B, Cm, dt, init))
    A, Dk = -0.5 - 1.5 * rand(D, 16), rand(D) - 0.5
    y = torch.empty((b, D, L), dtype=torch.float16, device="cuda")
    fin = torch.empty((b, D, 16), device="cuda")
    q.quamba_mamba1_scan(_shape(q, b, D, 16, L, 4), q.DeviceScales(host_scales(q, sc)), x, B, Cm, dt, A, Dk, y, init_state=init,
                         final_state=fin)
    assert infinite or (torch.isfinite(y).all() and torch.isfinite(fin).all())
    y, fin = y.view(torch.int16), fin.view(torch.int32)
    for i in range(1, b):
        assert torch.equal(y[i], y[0]) and torch.equal(fin[i], fin[0]), i


@pytest.mark.parametrize("D,L,form", [(2000, 600, "halves"), (2000, 1537, "halves"), (6400, 900, "8 channels")])
def test_infinite_and_zero_states_in_halves_and_in_workgroups_of_8_channels(gpu_lib, D, L, form):
    """... over one tile and several."""
    assert _form(gpu_lib, 2, D, 16, L) == form
    test_infinite_and_zero_states(gpu_lib, D, L)


@pytest.mark.parametrize("b,D,L,mixed", [(1, 5120, 513, True),     # a full workgroup on every unit; one token in the second tile of 32 lanes
                                         (1, 5120, 512, False),    # one tile of 32 lanes
                                         (1, 5121, 513, False),    # a channel more than 20 per unit
                                         (3, 1681, 1024, True),    # the last workgroup of a sequence with one channel
                                         (2, 2137, 1025, True),    # ... with 17: one on 64 lanes; a third tile of one token
                                         (1, 4300, 2060, True)])
@pytest.mark.parametrize("sides", [False, True])
def test_workgroups_of_20_channels_on_32_and_64_lanes(gpu_lib, b, D, L, mixed, sides):
    """16 channels on 32 lanes and 4 on 64 in one workgroup, at the edges of their rule and of their tiles."""
    mixes = gpu_lib.load_library()._ZN6quamba17mamba1_scan_mixesERK18quamba_ssd_shape_t
    mixes.restype = C.c_bool
    assert mixes(C.byref(_shape(gpu_lib, b, D, 16, L, 4))) == mixed
    test_scan_with_side_inputs(gpu_lib, b, D, 16, L, 0, sides, sides)


def test_infinite_and_zero_states_on_32_and_64_lanes(gpu_lib):
    test_infinite_and_zero_states(gpu_lib, 2500, 1600)  # two sequences: 20 channels per unit


@pytest.mark.parametrize("b,D,L", [(3, 1537, 1300), (1, 5120, 1003)])
def test_equal_sequences_on_32_and_64_lanes(gpu_lib, b, D, L):
    """... whose channels are shared out alike; and twice the same call."""
    for infinite in (False, True):
        test_equal_sequences_of_one_call_have_equal_results(gpu_lib, b, D, L, "24 channels", infinite)
