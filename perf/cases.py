"""The work a program that serves quantized Mamba models has this package do, as measurable cases.

A prompt goes through the causal convolution and the selective scan of every layer, each generated token through one
step of the same on cached states, and the layer's output through the quantized Hadamard transform in front of the
output projection.  The layer shapes are the 130M-, 2.7B- and 8B-shaped Mamba2 layers, the 2.8B-shaped Mamba1 layer and
the tiny layer that workloads/, bench.py and the tests use; the values follow the structure workloads/synth.py
describes (drawn on the GPU here, so that inputs of full size are made in milliseconds).
"""
import math

import numpy as np
import torch

import paper_2503_22879_amd as q

# heads, channels per head, states, state groups, head clusters, channel ranges, chunk
MODELS = {"tiny": (8, 64, 16, 1, 1, 4, 64),
          "130m": (24, 64, 128, 1, 4, 4, 256),
          "2p7b": (80, 64, 128, 1, 4, 4, 256),
          "8b": (128, 64, 128, 8, 4, 4, 256)}
MAMBA1_STATES = 16
MAMBA1_CHANNELS = (1536, 5120)          # the widths of the 130M- and 2.8B-shaped layers
HADAMARD_WIDTHS = (1536, 5120, 8192)    # heads x channels of the Mamba2 layers above
MAX_SCAN_WORK = 4 * 4096 * 128          # tokens x heads of the largest listed scan
MAX_MAMBA1_WORK = 4 * 4096 * 5120       # tokens x channels of the largest listed Mamba1 scan


def listed():
    return [
        # Prompt batches through the scan alone: the workload of bench.py (a full batch, outputs only), ...
        dict(name="scan 8b 4x4096", kind="scan", model="8b", batch=4, seqlen=4096, final=False),
        # ... one prompt of a small model, whose state generation then starts from (few heads: latency), ...
        dict(name="scan 130m 1x2048", kind="scan", model="130m", batch=1, seqlen=2048, final=True),
        # ... and the smallest layer (16 states), a call that takes little beyond being made.
        dict(name="scan tiny 1x256", kind="scan", model="tiny", batch=1, seqlen=256, final=False),
        # Prompts through convolution and scan, with both states kept for generation: a batch of full prompts, ...
        dict(name="prompt 2p7b 8x2048", kind="prompt", model="2p7b", batch=8, seqlen=2048, resumed=False, gated=False),
        # ... and the next piece of one long prompt, of odd length, from the states of the piece before, with the
        # output gate and the step sizes as 8-bit codes.
        dict(name="prompt 8b 1x1531 resumed", kind="prompt", model="8b", batch=1, seqlen=1531, resumed=True, gated=True),
        # One generated token per sequence through convolution, state update and Hadamard transform: a full serving
        # batch on the fp32 state, ...
        dict(name="step 8b 256", kind="step", model="8b", batch=256, cache="fp32", gated=False),
        # ... a smaller, uneven one on the 8-bit cached state with the output gate, ...
        dict(name="step 8b 100 q8", kind="step", model="8b", batch=100, cache="q8", gated=True),
        # ... and a single sequence on a small model (all side inputs as codes): the latency of a token.
        dict(name="step 130m 1", kind="step", model="130m", batch=1, cache="fp32", gated=True),
        # The transform behind a prompt batch of the 2.7B-shaped layer (order 20 * 256).
        dict(name="hadamard 5120x16384", kind="hadamard", width=5120, rows=16384),
        # The Mamba1 layer: a prompt batch, ...
        dict(name="mamba1 scan 4x4096", kind="mamba1_scan", channels=5120, batch=4, seqlen=4096, resumed=False, gated=False),
        # ... one prompt of odd length with gate and step-size codes, resumed from a state, ...
        dict(name="mamba1 scan 1x1003", kind="mamba1_scan", channels=5120, batch=1, seqlen=1003, resumed=True, gated=True),
        # ... and one generated token for a serving batch.
        dict(name="mamba1 step 256", kind="mamba1_step", channels=5120, batch=256, gated=False),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over its logarithm."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["scan", "prompt", "step", "step", "hadamard", "mamba1_scan", "mamba1_step"])
    if kind in ("scan", "prompt"):
        model = rng.choice(["tiny", "130m", "2p7b", "8b"] if kind == "scan" else ["130m", "2p7b", "8b"])
        seqlen = _log(rng, 16, 512 if model == "tiny" else 4096)
        batch = _log(rng, 1, min(16, MAX_SCAN_WORK // (seqlen * MODELS[model][0])))
        if kind == "scan":
            return dict(kind=kind, model=model, batch=batch, seqlen=seqlen, final=rng.random() < 0.5)
        return dict(kind=kind, model=model, batch=batch, seqlen=seqlen, resumed=rng.random() < 0.5, gated=rng.random() < 0.5)
    if kind == "step":
        return dict(kind=kind, model=rng.choice(["130m", "2p7b", "8b"]), batch=_log(rng, 1, 256),
                    cache=rng.choice(["fp32", "q8"]), gated=rng.random() < 0.5)
    if kind == "hadamard":
        return dict(kind=kind, width=rng.choice(HADAMARD_WIDTHS), rows=_log(rng, 1, 16384))
    channels = rng.choice(MAMBA1_CHANNELS)
    if kind == "mamba1_step":
        return dict(kind=kind, channels=channels, batch=_log(rng, 1, 256), gated=rng.random() < 0.5)
    seqlen = _log(rng, 16, 4096)
    return dict(kind=kind, channels=channels, batch=_log(rng, 1, min(4, MAX_MAMBA1_WORK // (seqlen * channels))),
                seqlen=seqlen, resumed=rng.random() < 0.5, gated=rng.random() < 0.5)


# ---------------------------------------------------------------- inputs


class _Draw:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda")

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device="cuda")


def _codes(v, scale):
    """Eq. 1: symmetric 8-bit codes with a static scale."""
    return (v / scale).round_().clamp_(-128, 127).to(torch.int8)


def _host(t):
    return t.detach().cpu().numpy()


def _softplus(v):
    return torch.nn.functional.softplus(v)


def _scales(model, x_absmax, b_absmax, c_absmax):
    """Sort-and-cluster of a Mamba2 layer from calibrated maxima: (head order, channel order, scales on the host)."""
    H, P, N, G, m, n, _ = MODELS[model]
    return q.quamba_reorder_params(H, P, G, m, n, N, _host(x_absmax), _host(b_absmax), _host(c_absmax))


def _x_scale_table(model, hs):
    """Scale of every (head, channel position) [H, P] from the cluster tables."""
    H, P, _, G, m, n, _ = MODELS[model]
    out = np.empty((H, P), np.float32)
    for h in range(H):
        g, hl = divmod(h, H // G)
        i = int(np.searchsorted(hs.head_cluster_end[g * m:(g + 1) * m], hl, side="right"))
        cell = (g * m + min(i, m - 1)) * n
        j = np.searchsorted(hs.chan_cluster_end[cell:cell + n], np.arange(P), side="right")
        out[h] = hs.x_scales[cell + np.minimum(j, n - 1)]
    return torch.from_numpy(out).cuda()


def _shape(model, batch, seqlen):
    H, P, N, G, m, n, chunk = MODELS[model]
    return q.Shape(batch=batch, seqlen=seqlen, nheads=H, headdim=P, d_state=N, ngroups=G, chunk=chunk, n_head_clusters=m,
                   n_chan_clusters=n, flags=0)


def _layer_constants(d, H):
    """A and D of a Mamba2 layer."""
    return -torch.exp(d.uniform(H) * math.log(16.0)), d.normal(H)


def _gate(d, x_shape, dt_shape, heads, with_dt):
    """8-bit side inputs: gate codes, and codes of the step size's pre-activation with its bias."""
    z = d.normal(*x_shape) * torch.exp(0.5 * d.normal(*x_shape[-2:]))
    zs = float(z.abs().max()) / 127
    if not with_dt:
        return q.Gate(z=_codes(z, zs), z_scale=zs)
    bias = 0.5 * d.normal(heads)
    pre = d.normal(*dt_shape) - 3.0 - bias
    ds = float(pre.abs().max()) / 127
    return q.Gate(z=_codes(z, zs), z_scale=zs, dt_q=_codes(pre, ds), dt_scale=ds, dt_bias=bias)


def _empty_outputs(model, batch, seqlen):
    H, P, N, G = MODELS[model][:4]
    y = torch.empty((batch, seqlen, H, P), dtype=torch.float16, device="cuda")
    state = torch.empty((batch, H, P, N), device="cuda")
    return y, state


def _workspace(shape):
    n = q.quamba_ssd_prefill_workspace_size(shape)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _prepare_scan(case, d):
    H, P, N, G = MODELS[case["model"]][:4]
    b, L = case["batch"], case["seqlen"]
    sigma = torch.exp(d.normal(H, P))
    heavy = d.uniform(H, P) < 0.01
    sigma = torch.where(heavy, 20.0 * sigma, sigma)
    prof = []
    for _ in range(2):
        gain = torch.exp(d.normal(G))
        prof.append((gain / gain.max())[:, None] * torch.exp(0.5 * d.normal(G, N)))
    # about the largest of a calibration draw of some thousand tokens
    head, chan, hs = _scales(case["model"], 3.8 * sigma, 3.8 * prof[0], 3.8 * prof[1])
    head, chan = torch.from_numpy(head).long().cuda(), torch.from_numpy(chan).long().cuda()
    sigma = torch.gather(sigma[head], 1, chan)
    table = _x_scale_table(case["model"], hs)
    shape = _shape(case["model"], b, L)
    A, D = _layer_constants(d, H)
    y, fin = _empty_outputs(case["model"], b, L)
    return dict(run=_run_scan, shape=shape, scales=q.DeviceScales(hs), x=_codes(d.normal(b, L, H, P).mul_(sigma), table),
                B=_codes(d.normal(b, L, G, N).mul_(prof[0]), torch.from_numpy(hs.B_scales).cuda()[:, None]),
                C=_codes(d.normal(b, L, G, N).mul_(prof[1]), torch.from_numpy(hs.C_scales).cuda()[:, None]),
                dt=_softplus(d.normal(b, L, H) - 3.0), A=A, D=D, y=y, fin=fin if case["final"] else None,
                ws=_workspace(shape))


def _run_scan(s):
    q.quamba_ssd_prefill(s["shape"], s["scales"], s["x"], s["B"], s["C"], s["dt"], s["A"], s["D"], None, s["y"],
                         final_state=s["fin"], workspace=s["ws"])
    return s["y"] if s["fin"] is None else (s["y"], s["fin"])


class _Conv:
    """A layer's quantized convolution, calibrated on a draw of its own and laid out in the clustered channel order, and
    the scales of the scan that follows from the same calibration."""

    def __init__(self, model, d):
        H, P, N, G = MODELS[model][:4]
        HP, GN = H * P, G * N
        self.ct = HP + 2 * GN
        self.in_scale = 4.5 / 127
        sigma = torch.exp(0.3 * d.normal(self.ct))
        w = d.normal(self.ct, 4) * (torch.exp(0.5 * d.normal(self.ct)) / sigma * 0.75)[:, None]
        bias = 0.3 * d.normal(self.ct)
        u = d.normal(512, self.ct) * sigma
        v = bias + sum(w[:, k] * u[k:512 - 3 + k] for k in range(4))
        out = torch.nn.functional.silu(v)
        self.absmax, self.rms = out.abs().amax(0), out.square().mean(0).sqrt()
        head, chan, self.hs = _scales(model, self.absmax[:HP].view(H, P), self.absmax[HP:HP + GN].view(G, N),
                                      self.absmax[HP + GN:].view(G, N))
        rows = (torch.from_numpy(head).long()[:, None] * P + torch.from_numpy(chan).long()).view(-1).cuda()
        order = torch.cat([rows, torch.arange(HP, self.ct, device="cuda")])
        w_scale = float(w.abs().max()) / 127
        self.sigma = sigma[order].contiguous()
        self.absmax, self.rms = self.absmax[order].contiguous(), self.rms[order].contiguous()
        self.weight = _codes(w[order], w_scale)
        self.bias = bias[order].contiguous()
        self.in_w_scale = float(np.float32(self.in_scale * w_scale))
        self.scales = q.DeviceScales(self.hs)

    def inputs(self, d, batch, seqlen):
        return _codes(d.normal(batch, seqlen, self.ct).mul_(self.sigma), self.in_scale)


def _scan_operands(model, batch, seqlen):
    H, P, N, G = MODELS[model][:4]
    x = torch.empty((batch, seqlen, H, P), dtype=torch.int8, device="cuda")
    B = torch.empty((batch, seqlen, G, N), dtype=torch.int8, device="cuda")
    return x, B, torch.empty_like(B)


def _draw_state(d, conv, model, batch):
    """A cached state: its rows follow the channel magnitudes of x, its columns those of B's group."""
    H, P, N, G = MODELS[model][:4]
    HP, GN = H * P, G * N
    rows = conv.absmax[:HP].view(H, P, 1)
    cols = conv.absmax[HP:HP + GN].view(G, N).repeat_interleave(H // G, 0).view(H, 1, N)
    return d.normal(batch, H, P, N).mul_(0.1 * rows * cols)


def _prepare_prompt(case, d):
    model, b, L = case["model"], case["batch"], case["seqlen"]
    H, P, N, G = MODELS[model][:4]
    conv = _Conv(model, d)
    shape = _shape(model, b, L)
    x, B, C = _scan_operands(model, b, L)
    A, D = _layer_constants(d, H)
    y, fin = _empty_outputs(model, b, L)
    gate = _gate(d, (b, L, H, P), (b, L, H), H, True) if case["gated"] else None
    return dict(run=_run_prompt, shape=shape, conv=conv, xBC=conv.inputs(d, b, L), x=x, B=B, C=C,
                conv_in=conv.inputs(d, b, 3) if case["resumed"] else None,
                conv_out=torch.empty((b, 3, conv.ct), dtype=torch.int8, device="cuda"),
                init=_draw_state(d, conv, model, b) if case["resumed"] else None,
                dt=None if case["gated"] else _softplus(d.normal(b, L, H) - 3.0), gate=gate, A=A, D=D, y=y, fin=fin,
                ws=_workspace(shape))


def _run_prompt(s):
    c = s["conv"]
    q.quamba_conv1d_q8(s["shape"], c.scales, s["xBC"], c.weight, c.bias, c.in_w_scale, s["x"], s["B"], s["C"],
                       conv_state_in=s["conv_in"], conv_state_out=s["conv_out"])
    q.quamba_ssd_prefill(s["shape"], c.scales, s["x"], s["B"], s["C"], s["dt"], s["A"], s["D"], s["init"], s["y"],
                         final_state=s["fin"], workspace=s["ws"], gate=s["gate"])
    return s["y"], s["fin"], s["conv_out"], s["x"], s["B"], s["C"]


def _prepare_step(case, d):
    model, b = case["model"], case["batch"]
    H, P, N, G = MODELS[model][:4]
    conv = _Conv(model, d)
    shape = _shape(model, b, 1)
    x, B, C = _scan_operands(model, b, 1)
    A, D = _layer_constants(d, H)
    q8 = case["cache"] == "q8"
    gate = _gate(d, (b, H, P), (b, H), H, not q8) if case["gated"] else None
    dt = None if case["gated"] and not q8 else _softplus(d.normal(b, H) - 3.0)
    state, state_scales = _draw_state(d, conv, model, b), None
    if q8:  # static scales from the largest values of a few states of a separate draw
        calib = _host(_draw_state(d, conv, model, 8).abs().amax(0))
        m, n = MODELS[model][4:6]
        state_scales = torch.from_numpy(q.quamba_state_scales(H, P, G, m, n, N, conv.hs.head_cluster_end,
                                                              conv.hs.chan_cluster_end, calib)).cuda()
        codes = torch.empty(state.shape, dtype=torch.int8, device="cuda")
        q.quamba_ssd_quantize_state(shape, conv.scales, state_scales, state, codes)
        state = codes
    # the transform's static scale: a code of 127 for 4 standard deviations of its values, from the calibrated sizes of
    # x, C and the cached state (y = C h + D x; the gate takes SiLU of a unit normal)
    HP, GN = H * P, G * N
    rows = (0.1 * conv.absmax[:HP]).view(G, -1)
    Ch = rows.square() * (conv.absmax[HP:HP + GN] * conv.rms[HP + GN:]).view(G, N).square().sum(1, keepdim=True)
    Dx = (D[:, None] * conv.rms[:HP].view(H, P)).square()
    s_y = 4.0 * float((Ch.sum() + Dx.sum()).sqrt()) * (0.6 if case["gated"] else 1.0) / 127
    return dict(run=_run_step, shape=shape, conv=conv, xBC=conv.inputs(d, b, 1), conv_state=conv.inputs(d, b, 3),
                x=x, B=B, C=C, xs=x.view(b, H, P), Bs=B.view(b, G, N), Cs=C.view(b, G, N), dt=dt, A=A, D=D, gate=gate,
                state=state, state_scales=state_scales, s_y=s_y,
                y=torch.empty((b, H, P), dtype=torch.float16, device="cuda"),
                yq=torch.empty((b, H * P), dtype=torch.int8, device="cuda"))


def _run_step(s):
    c = s["conv"]
    q.quamba_conv1d_q8(s["shape"], c.scales, s["xBC"], c.weight, c.bias, c.in_w_scale, s["x"], s["B"], s["C"],
                       conv_state_in=s["conv_state"], conv_state_out=s["conv_state"])
    if s["state_scales"] is None:
        q.quamba_ssd_decode_step(s["shape"], c.scales, s["xs"], s["Bs"], s["Cs"], s["dt"], s["A"], s["D"], s["state"],
                                 s["y"], gate=s["gate"])
    else:
        q.quamba_ssd_decode_step_q8(s["shape"], c.scales, s["state_scales"], s["xs"], s["Bs"], s["Cs"], s["dt"], s["A"],
                                    s["D"], s["state"], s["y"], gate=s["gate"])
    y = s["y"]
    q.quamba_hadamard_quantize(y.view(y.shape[0], -1), s["s_y"], s["yq"])
    return s["state"], y, s["yq"], s["conv_state"], s["x"], s["B"], s["C"]


def _prepare_hadamard(case, d):
    n, rows = case["width"], case["rows"]
    sigma = 0.05 * torch.exp(0.5 * d.normal(n))
    sigma = torch.where(d.uniform(n) < 0.005, 20.0 * sigma, sigma)
    y = d.normal(rows, n).mul_(sigma).to(torch.float16)
    s_y = 4.0 * float(sigma.square().sum().sqrt()) / 127
    return dict(run=_run_hadamard, y=y, s_y=s_y, out=torch.empty((rows, n), dtype=torch.int8, device="cuda"))


def _run_hadamard(s):
    q.quamba_hadamard_quantize(s["y"], s["s_y"], s["out"])
    return s["out"]


class _Mamba1:
    """A Mamba1 layer: channels in ascending order of magnitude, four ranges of equal width with one scale each."""

    def __init__(self, channels, d):
        sigma = torch.exp(d.normal(channels))
        sigma = torch.where(d.uniform(channels) < 0.01, 10.0 * sigma, sigma).sort().values
        ends = np.array([channels * k // 4 for k in (1, 2, 3, 4)], np.int32)
        top = 3.8 * _host(sigma)
        xs = np.array([top[e - 1] / 127 for e in ends], np.float32)
        self.gain = [torch.exp(0.5 * d.normal(MAMBA1_STATES)) for _ in range(2)]
        bc = [np.array([3.8 * float(g.max()) / 127], np.float32) for g in self.gain]
        self.scales = q.DeviceScales(q.HostScales(xs, np.array([1], np.int32), ends, bc[0], bc[1]))
        self.bc = [float(v[0]) for v in bc]
        self.sigma = sigma
        self.xs = torch.from_numpy(np.repeat(xs, np.diff(ends, prepend=0))).cuda()
        steps = torch.arange(1, MAMBA1_STATES + 1, device="cuda", dtype=torch.float32)
        self.A = -(steps * torch.exp(0.2 * d.normal(channels, MAMBA1_STATES)))
        self.D = d.normal(channels)
        self.dt_offset = 0.5 * d.normal(channels)

    def x(self, d, b, L):
        return _codes(d.normal(b, self.sigma.numel(), L).mul_(self.sigma[:, None]), self.xs[:, None])

    def bc_codes(self, d, b, L):
        return [_codes(d.normal(b, MAMBA1_STATES, L).mul_(g[:, None]), s) for g, s in zip(self.gain, self.bc)]

    def dt(self, d, b, L):
        return _softplus(d.normal(b, self.sigma.numel(), L) - 3.0 + self.dt_offset[:, None])

    def gate(self, d, b, L):
        c = self.sigma.numel()
        z = d.normal(b, c, L).mul_(torch.exp(0.5 * d.normal(c))[:, None])
        bias = 0.5 * d.normal(c)
        pre = d.normal(b, c, L) - 3.0 - bias[:, None]
        zs, ds = float(z.abs().max()) / 127, float(pre.abs().max()) / 127
        return q.Gate(z=_codes(z, zs), z_scale=zs, dt_q=_codes(pre, ds), dt_scale=ds, dt_bias=bias)

    def state(self, d, b):
        return d.normal(b, self.sigma.numel(), MAMBA1_STATES).mul_(0.1 * self.sigma[:, None])


def _mamba1_shape(channels, b, L):
    return q.Shape(batch=b, seqlen=L, nheads=1, headdim=channels, d_state=MAMBA1_STATES, ngroups=1, chunk=1,
                   n_head_clusters=1, n_chan_clusters=4, flags=0)


def _prepare_mamba1_scan(case, d):
    c, b, L = case["channels"], case["batch"], case["seqlen"]
    layer = _Mamba1(c, d)
    B, C = layer.bc_codes(d, b, L)
    gated = case["gated"]
    return dict(run=_run_mamba1_scan, shape=_mamba1_shape(c, b, L), layer=layer, x=layer.x(d, b, L), B=B, C=C,
                dt=None if gated else layer.dt(d, b, L), gate=layer.gate(d, b, L) if gated else None,
                init=layer.state(d, b) if case["resumed"] else None,
                y=torch.empty((b, c, L), dtype=torch.float16, device="cuda"),
                fin=torch.empty((b, c, MAMBA1_STATES), device="cuda"))


def _run_mamba1_scan(s):
    m = s["layer"]
    q.quamba_mamba1_scan(s["shape"], m.scales, s["x"], s["B"], s["C"], s["dt"], m.A, m.D, s["y"], init_state=s["init"],
                         final_state=s["fin"], gate=s["gate"])
    return s["y"], s["fin"]


def _prepare_mamba1_step(case, d):
    c, b = case["channels"], case["batch"]
    layer = _Mamba1(c, d)
    B, C = (v[:, :, 0].contiguous() for v in layer.bc_codes(d, b, 1))
    gate = None
    if case["gated"]:
        g = layer.gate(d, b, 1)
        gate = q.Gate(z=g.z[:, :, 0].contiguous(), z_scale=g.z_scale, dt_q=g.dt_q[:, :, 0].contiguous(),
                      dt_scale=g.dt_scale, dt_bias=g.dt_bias)
    return dict(run=_run_mamba1_step, shape=_mamba1_shape(c, b, 1), layer=layer, x=layer.x(d, b, 1)[:, :, 0].contiguous(),
                B=B, C=C, dt=None if gate else layer.dt(d, b, 1)[:, :, 0].contiguous(), gate=gate, state=layer.state(d, b),
                y=torch.empty((b, c), dtype=torch.float16, device="cuda"))


def _run_mamba1_step(s):
    m = s["layer"]
    q.quamba_mamba1_decode_step(s["shape"], m.scales, s["x"], s["B"], s["C"], s["dt"], m.A, m.D, s["state"], s["y"],
                                gate=s["gate"])
    return s["state"], s["y"]


_PREPARE = {"scan": _prepare_scan, "prompt": _prepare_prompt, "step": _prepare_step, "hadamard": _prepare_hadamard,
            "mamba1_scan": _prepare_mamba1_scan, "mamba1_step": _prepare_mamba1_step}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _Draw(seed))


def run(state):
    return state["run"](state)


# ---------------------------------------------------------------- what a pass cannot do without


def _gate_bytes(x_values, dt_values, gated, with_dt=True):
    """dt as fp32, or its codes; the gate's codes."""
    if not gated:
        return 4 * dt_values
    return x_values + (1 if with_dt else 4) * dt_values


def _scan_work(case):
    H, P, N, G, _, _, chunk = MODELS[case["model"]]
    tok = case["batch"] * case["seqlen"]
    qn = min(chunk, case["seqlen"])
    # chunked form: causal half of the scores and of their product with x, carried state, state update
    flops = 2 * tok * (H * ((qn + 1) / 2 * P + 2 * N * P) + G * (qn + 1) / 2 * N)
    # x, B, C codes in, fp16 y out
    return tok * (3 * H * P + 2 * G * N), flops


def _conv_work(model, tok):
    H, P, N, G = MODELS[model][:4]
    ct = H * P + 2 * G * N
    # int8 in and out, filter and bias; 4 multiply-adds, bias, SiLU and the rounding per value
    return 2 * tok * ct + 8 * ct, tok * ct * (8 + 8)


def work(case):
    kind = case["kind"]
    if kind == "hadamard":
        n, rows = case["width"], case["rows"]
        k = n & -n  # power-of-two part; the other factor (3 or 5, times 4) is summed over its blocks
        m = n // k * 4 if n != k else 1
        adds = math.log2(n / m) + (m - 1 if m > 1 else 0)
        return {"bytes": 3 * rows * n, "flops": rows * n * (adds + 2)}
    if kind in ("mamba1_scan", "mamba1_step"):
        c, b, N = case["channels"], case["batch"], MAMBA1_STATES
        L = case.get("seqlen", 1)
        by = b * c * L * 3 + _gate_bytes(b * c * L, b * c * L, case["gated"]) + 2 * b * N * L + 4 * c * (N + 1)
        states = 2 if kind == "mamba1_step" or case["resumed"] else 1
        return {"bytes": by + 4 * b * c * N * states, "flops": b * c * L * N * 7}
    H, P, N, G = MODELS[case["model"]][:4]
    if kind == "step":
        b, cell = case["batch"], 4 if case["cache"] == "fp32" else 1
        by, fl = _conv_work(case["model"], b)
        by += 6 * b * (H * P + 2 * G * N)                                  # conv state in and out
        by += 2 * cell * b * H * P * N                                     # cached state in and out
        by += _gate_bytes(b * H * P, b * H, case["gated"], cell == 4)
        by += b * H * P * (2 + 1)                                          # y and its transformed codes
        return {"bytes": by, "flops": fl + b * H * P * (N * (5 if cell == 4 else 9) + math.log2(H * P) + 2)}
    b, tok = case["batch"], case["batch"] * case["seqlen"]
    by, fl = _scan_work(case)
    if kind == "scan":
        return {"bytes": by + 4 * tok * H + (4 * b * H * P * N if case["final"] else 0), "flops": fl}
    cby, cfl = _conv_work(case["model"], tok)
    ct = H * P + 2 * G * N
    # x, B and C are outputs of the convolution and are counted there once
    by = cby + 2 * tok * H * P + _gate_bytes(tok * H * P, tok * H, case["gated"])
    by += 4 * b * H * P * N * (2 if case["resumed"] else 1) + 3 * b * ct * (2 if case["resumed"] else 1)
    return {"bytes": by, "flops": fl + cfl}


def tolerance(case):
    kind = case["kind"]
    if kind == "hadamard":
        return "exact"   # the order of the fp32 additions is part of the interface
    if kind in ("mamba1_scan", "mamba1_step"):
        # fp32 recurrence, y rounded to fp16 (2^-11 of a value)
        return {"rel": 5e-4, "max": 5e-3}
    if case["model"] == "tiny":
        return {"rel": 5e-4, "max": 5e-3}  # fp32 recurrence as well
    if kind == "step":
        # fp32 update and sum, y rounded to fp16.  The convolution's codes, its state and the 8-bit state are exact; a
        # value of y whose rounding flips moves a transformed value by less than a thousandth of a code.
        return {"rel": 5e-4, "max": 5e-3, "differ": 1e-3}
    # products of operands rounded to fp16 (2^-11 each), fp32 sums, y rounded to fp16; the convolution's codes are exact
    return {"rel": 2e-3, "max": 2e-2, "differ": 0.0}
