"""Workloads of the correlator library as a user's program runs them.

Each case is one pass through the public entry points of
`paper_1609_04205_amd`, at the array shapes of the library's own
configurations (48 antennas of one station, 288 antennas in 6 stations, 576 in
12; 64 channels; one second is 3051 spectra of 64 channels or 762 of 256) and
at odd sizes between them.

  listed()            the standing cases
  draw(rng)           one more case from the same ranges
  prepare(case, seed) inputs, plans, workspaces and output buffers on the GPU
  run(state)          one pass; returns its outputs
  work(case)          bytes and operations the pass cannot do without
  exact(case, seed)   the outputs in 64 bits, from plain torch
"""
import math
import random

import numpy as np
import torch

import paper_1609_04205_amd as afc

P, T, FINE = 64, 16, 256          # channels, taps, channels of the fine bank
NU0, SUBBAND_HZ, C_LIGHT = 60.0e6, 195312.5, 299792458.0
SIGMA_N, SIGMA_S = 32.0, 8.0      # receiver noise and sky source, per component
PACKET = 16                       # time samples per station packet
STATION = 48                      # antennas per station
DEV = "cuda"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # one station, one subband, a third of a second: the smallest whole
        # call, where launches and latency count
        {"name": "fx-48ant-1sb-i8", "op": "fx", "antennas": 48, "subbands": 1, "spectra": 1024, "dtype": "i8",
         "flagged": 2},
        # an array and integrations that fit no tile, float32 throughout,
        # every subband with its own integration length
        {"name": "fx-75ant-3sb-f32-ragged", "op": "fx", "antennas": 75, "subbands": 3, "spectra": 999, "dtype": "f32",
         "flagged": 3},
        # the 6-station array's channeliser, eight subbands of one second
        {"name": "channelise-288ant-8sb-i8", "op": "channelise", "antennas": 288, "subbands": 8, "spectra": 3051,
         "dtype": "i8"},
        # one subband of the 12-station array, as it arrives: half precision
        {"name": "channelise-576ant-1sb-f16", "op": "channelise", "antennas": 576, "subbands": 1, "spectra": 3051,
         "dtype": "f16"},
        # the 256-channel bank with delays and bandpass, 12 stations
        {"name": "fine-576ant-4sb-i8", "op": "fine", "antennas": 576, "subbands": 4, "spectra": 762, "dtype": "i8"},
        # the correlator on the whole step of the 12-station array
        {"name": "correlate-576ant-16sb-i8", "op": "correlate", "antennas": 576, "subbands": 16, "spectra": 3051,
         "dtype": "i8", "flagged": 0},
        # the same array in float32, the accuracy reference of the science case
        {"name": "correlate-576ant-2sb-f32", "op": "correlate", "antennas": 576, "subbands": 2, "spectra": 3051,
         "dtype": "f32", "flagged": 0},
        # batched form: ragged integrations, int8 and fp16 subbands, flags
        {"name": "plan-576ant-16sb-mixed", "op": "plan", "antennas": 576, "subbands": 16, "spectra": 3051, "mix": 4,
         "flagged": 29},
        # lost packets: masks, zeroing, weighting matrix, mean visibilities
        {"name": "lost-576ant-4sb-i8", "op": "lost", "antennas": 576, "subbands": 4, "spectra": 3051, "dtype": "i8"},
        # loss and gradient of the calibration, through autograd, on flagged data
        {"name": "calgrad-576ant-64ch", "op": "calgrad", "antennas": 576, "channels": 64, "weighted": True},
        # real-time flagging, then the gain solution of the 6-station array
        {"name": "calsolve-288ant-64ch", "op": "calsolve", "antennas": 288, "channels": 64, "iterations": 30},
        # snapshot image of the 12-station array from eight subbands
        {"name": "image-576ant-8sb-2048", "op": "image", "antennas": 576, "subbands": 8, "grid": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of one of the kinds above, its sizes spread over the logarithm
    of their range and bounded by the listed cases' cost."""
    op = rng.choice(["fx", "channelise", "fine", "correlate", "plan", "lost", "calgrad", "calsolve", "image"])
    na = _log_int(rng, 24, 576)
    if op in ("calgrad", "calsolve"):
        if op == "calsolve":
            return {"op": op, "antennas": min(na, 288), "channels": rng.choice([16, 32, 64]),
                    "iterations": rng.randint(10, 30)}
        return {"op": op, "antennas": na, "channels": rng.choice([16, 32, 64]), "weighted": rng.random() < 0.5}
    if op == "image":
        return {"op": op, "antennas": na, "subbands": rng.randint(1, 8), "grid": rng.choice([512, 1024, 2048])}
    s = _log_int(rng, 96, 762 if op == "fine" else 3051)
    cells = {"fx": 576 * 3051, "channelise": 8 * 288 * 3051, "fine": 4 * 576 * 762, "correlate": 8 * 576 * 3051,
             "plan": 8 * 576 * 3051, "lost": 4 * 576 * 3051}[op]       # antennas x spectra x subbands
    b = max(1, min(_log_int(rng, 1, 16), cells // (na * s)))
    case = {"op": op, "antennas": na, "subbands": b, "spectra": s}
    if op == "plan":
        case.update(mix=rng.randrange(1000), flagged=na // 20)
        return case
    case["dtype"] = rng.choice(["i8", "f16", "f32"])
    if op in ("fx", "correlate"):
        case["flagged"] = rng.choice([0, na // 20])
        if case["dtype"] == "f32":                                     # 16 times the matrix work of fp16
            case["subbands"] = max(1, min(b, 2 * 576 * 576 * 3051 // (na * na * s)))
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed, *more):
    g = torch.Generator(device=DEV)
    k = int(seed) & 0x7FFFFFFF
    for m in more:
        k = (k * 1000003 + int(m) + 1) & 0x7FFFFFFFFFFF
    g.manual_seed(k)
    return g


def _rnd(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype)


def _uni(g, *shape, dtype=torch.float64):
    return torch.rand(shape, generator=g, device=DEV, dtype=dtype)


def _positions(na, seed):
    """East and north of every antenna in metres: stations of 48 antennas in
    discs of 30 m, six on a ring of 150 m and six on one of 588 m."""
    g = _gen(seed, 11)
    k = torch.arange(na, device=DEV) // STATION
    ring = torch.where(k < 6, 150.0, 588.0).to(torch.float64)
    ang = 2.0 * math.pi * (k % 6) / 6.0 + torch.where(k < 6, 0.0, math.pi / 6.0)
    r, phi = 30.0 * torch.sqrt(_uni(g, na)), 2.0 * math.pi * _uni(g, na)
    return torch.stack([ring * torch.cos(ang) + r * torch.cos(phi), ring * torch.sin(ang) + r * torch.sin(phi)],
                       1).contiguous()


def _taps(channels):
    """Hann-windowed sinc, T taps per branch, in the order [tap][branch]."""
    m = np.arange(channels * T, dtype=np.float64)
    w = 0.5 - 0.5 * np.cos(2.0 * np.pi * m / (channels * T - 1))
    a = (m - (channels * T - 1) / 2.0) / channels
    return torch.from_numpy((w * np.sinc(a)).astype(np.float32)).to(DEV)


def _gain(taps, scale=1.0):
    sigma = math.hypot(SIGMA_N, SIGMA_S) * math.sqrt(float((taps.double() ** 2).sum())) * scale
    return float(np.float32(127.0 / (4.0 * sigma)))


def _voltages(b, rows, na, seed):
    """int16 [b][rows][na][2][2]: receiver noise and one source behind its
    geometric phases, rounded as the stations send it."""
    pos = _positions(na, seed)
    x = torch.empty((b, rows, na, 2, 2), dtype=torch.int16, device=DEV)
    step = max(1, (1 << 27) // (na * 4))
    for k in range(b):
        g = _gen(seed, 21, k)
        lm = 0.5 * _rnd(g, 2, dtype=torch.float64).clamp(-1, 1)
        ph = 2.0 * math.pi * (NU0 + k * SUBBAND_HZ) * (pos @ lm) / C_LIGHT
        c, s = torch.cos(ph).float()[None, :, None], torch.sin(ph).float()[None, :, None]
        for r in range(0, rows, step):
            n = min(rows, r + step) - r
            v = _rnd(g, n, na, 2, 2).mul_(SIGMA_N)
            q = _rnd(g, n, 1, 2, 2).mul_(SIGMA_S)
            v[..., 0] += q[..., 0] * c - q[..., 1] * s
            v[..., 1] += q[..., 0] * s + q[..., 1] * c
            x[k, r:r + n] = v.round_().clamp_(-32768, 32767).to(torch.int16)
    return x


_TORCH = {"i8": torch.int8, "f16": torch.float16, "f32": torch.float32}


def _samples(b, s, n, dtype, seed):
    """Channelised samples [b][P][Sb][n][8][2]: noise and a part that all
    receivers share, at the scale of the channeliser's output."""
    sb = -(-s // 8)
    z = torch.empty((b, P, sb, n, 8, 2), dtype=_TORCH[dtype], device=DEV)
    keep = (torch.arange(sb * 8, device=DEV).view(sb, 1, 8, 1) < s).float()
    scale = 31.75 if dtype != "f32" else 137.0
    for k in range(b):
        for c in range(0, P, 16):
            g = _gen(seed, 31, k, c)
            v = (_rnd(g, 16, sb, n, 8, 2) * 0.954 + _rnd(g, 16, sb, 1, 8, 2) * 0.3) * scale * keep
            z[k, c:c + 16] = v.round_().clamp_(-127, 127).to(torch.int8) if dtype == "i8" else v.to(z.dtype)
    return z


def _flags(b, na, flagged, seed):
    if not flagged:
        return None
    f = torch.zeros((b, na), dtype=torch.uint8, device=DEV)
    g = _gen(seed, 41)
    for k in range(b):
        f[k, torch.randperm(na, generator=g, device=DEV)[:flagged]] = 1
    return f


def _lengths(case):
    """Integration length of every subband."""
    b, s = case["subbands"], case["spectra"]
    r = random.Random(case.get("mix", 7) * 31 + 1)
    return [s] + [r.randint(max(1, s // 6), s) for _ in range(b - 1)]


def _mix(case):
    """Sample type of every subband of a plan, both in use."""
    r = random.Random(case["mix"] * 31 + 2)
    return [("i8", "f16")[k] if k < 2 else r.choice(("i8", "f16")) for k in range(case["subbands"])]


def _packets(b, rows, na, seed):
    """uint8 [b][packets][na]: bursts of lost packets of whole stations, about
    one packet in two hundred, and one station that sends nothing."""
    n_pk, n_st = -(-rows // PACKET), -(-na // STATION)
    g = _gen(seed, 51)
    start = (_uni(g, b, n_pk, n_st) < 6.0e-4).float()
    ok = (torch.nn.functional.max_pool1d(start.permute(0, 2, 1), 9, 1, 4) < 0.5).permute(0, 2, 1).to(torch.uint8)
    if n_st > 1:
        ok[b - 1, :, n_st - 1] = 0
    return ok[:, :, torch.arange(na, device=DEV) // STATION].contiguous()


def _pairs(na):
    t = torch.tril_indices(na, na, device=DEV)
    return t[0], t[1]


def _sky(na, channels, seed, nu0=NU0):
    """Model visibilities [channels][Nbl] complex128 of five point sources."""
    pos, g = _positions(na, seed), _gen(seed, 61)
    a, c = _pairs(na)
    lm = _uni(g, 5, 2) - 0.5
    flux = torch.exp(math.log(10.0) + math.log(100.0) * _uni(g, 5))
    m = torch.empty((channels, a.numel()), dtype=torch.complex128, device=DEV)
    for k in range(channels):
        off = k if k < channels // 2 else k - channels
        ph = 2.0 * math.pi * (nu0 + off * SUBBAND_HZ / channels) / C_LIGHT * (lm @ pos.T)
        e = torch.polar(flux.sqrt()[:, None].expand_as(ph).contiguous(), ph)
        m[k] = (e[:, a] * e[:, c].conj()).sum(0)
    return m


def _calibration(na, channels, seed, outliers=0.0):
    """V, M float32 [channels][Nbl][2][2][2] and unit gains: gains of 20 % in
    amplitude and any phase, noise of 5 %, some strong interference."""
    g = _gen(seed, 71)
    a, c = _pairs(na)
    sky = _sky(na, channels, seed)
    v = torch.empty((channels, a.numel(), 2, 2, 2), dtype=torch.float32, device=DEV)
    m = torch.zeros_like(v)
    amp, ph = 0.8 + 0.4 * _uni(g, channels, na, 2), 2.0 * math.pi * _uni(g, channels, na, 2)
    gain = torch.polar(amp, ph)
    auto = (a == c)
    for k in range(channels):
        level = 0.05 * sky[k].abs().mean().float()
        v[k] = _rnd(g, a.numel(), 2, 2, 2) * level
        if outliers:
            hit = _uni(g, a.numel()) < outliers
            v[k] += hit.float()[:, None, None, None] * 100.0 * level
        for p in range(2):
            s = gain[k, a, p] * sky[k] * gain[k, c, p].conj()
            v[k, :, p, p] += torch.view_as_real(s).float()
            v[k, :, p, p, 1].masked_fill_(auto, 0.0)
            m[k, :, p, p] = torch.view_as_real(sky[k]).float()
            m[k, :, p, p, 1].masked_fill_(auto, 0.0)
    unit = torch.zeros((channels, na, 2, 2), dtype=torch.float32, device=DEV)
    unit[..., 0] = 1.0
    return v, m, unit


def _n_bl(na):
    return na * (na + 1) // 2


# --------------------------------------------------------------------------
# the passes
# --------------------------------------------------------------------------
def prepare(case, seed):
    op, na = case["op"], case["antennas"]
    n = 2 * na
    st = {"op": op, "case": case}
    if op in ("fx", "channelise", "plan"):
        b, s = case["subbands"], case["spectra"]
        st["x"] = _voltages(b, (s + T - 1) * P, na, seed)
        st["taps"] = _taps(P)
        st["gain"] = _gain(st["taps"])
    if op in ("fx", "channelise", "fine"):
        st["z"] = torch.empty(afc.channelised_shape(case["subbands"], case["spectra"], n), dtype=_TORCH[case["dtype"]],
                              device=DEV)
    if op == "fine":
        b, s = case["subbands"], case["spectra"]
        g = _gen(seed, 81)
        st["x"] = _voltages(b, (s + T - 1) * FINE, na, seed)
        st["taps"] = _taps(FINE)
        st["delays"] = (6.0e-7 * _uni(g, na)).repeat_interleave(2) + 2.0e-9 * _uni(g, n)
        f = (torch.arange(FINE, device=DEV).double() / FINE + 0.5) % 1.0 - 0.5
        st["bandpass"] = (1.0 / ((1.0 - 1.2 * f * f) * (1.0 + 0.02 * torch.cos(14.0 * math.pi * f)))).float()
        st["center"] = [NU0 + k * SUBBAND_HZ for k in range(b)]
        st["gain"] = _gain(st["taps"], float((st["bandpass"].double() ** 2).view(P, 4).sum(1).max().sqrt()))
        st["ws"] = torch.empty(afc.fine_workspace_bytes(na, b, s), dtype=torch.uint8, device=DEV)
    if op == "correlate":
        st["z"] = _samples(case["subbands"], case["spectra"], n, case["dtype"], seed)
    if op in ("fx", "correlate"):
        b = case["subbands"]
        st["S"] = _lengths(case) if op == "fx" else None
        st["flags"] = _flags(b, na, case["flagged"], seed)
        st["vis"] = torch.empty(afc.visibility_shape(b, na), dtype=torch.int32 if case["dtype"] == "i8" else torch.float32,
                                device=DEV)
        st["weights"] = torch.empty((b, _n_bl(na)), dtype=torch.int32, device=DEV)
    if op == "plan":
        b = case["subbands"]
        st["plan"] = afc.Plan(na, _lengths(case), _mix(case), n_spectra=case["spectra"])
        st["ws"] = torch.empty(st["plan"].workspace_bytes, dtype=torch.uint8, device=DEV)
        st["flags"] = _flags(b, na, case["flagged"], seed)
        st["vis"] = torch.empty(afc.visibility_shape(b, na), dtype=torch.int32, device=DEV)
        st["weights"] = torch.empty((b, _n_bl(na)), dtype=torch.int32, device=DEV)
    if op == "lost":
        b, s = case["subbands"], case["spectra"]
        st["packets"] = _packets(b, (s + T - 1) * P, na, seed)
        st["z"] = _samples(b, s, n, case["dtype"], seed)
        st["spec"] = torch.empty(afc.validity_shape(b, s, na), dtype=torch.int32, device=DEV)
        st["weights"] = torch.empty((b, _n_bl(na)), dtype=torch.int32, device=DEV)
        g = _gen(seed, 91)
        v = _rnd(g, *afc.visibility_shape(b, na)).mul_(31.75 ** 2 * math.sqrt(s))
        st["vis"] = v.round_().to(torch.int32) if case["dtype"] == "i8" else v
        st["mean"] = torch.empty(afc.visibility_shape(b, na), dtype=torch.float32, device=DEV)
    if op == "calgrad":
        ch = case["channels"]
        st["V"], st["M"], g0 = _calibration(na, ch, seed)
        g = _gen(seed, 101)
        st["g"] = torch.view_as_complex(g0 + 0.1 * _rnd(g, *g0.shape)).contiguous().requires_grad_(True)
        st["flags"] = st["wt"] = None
        if case["weighted"]:
            st["flags"] = (_uni(g, ch, _n_bl(na), 2) < 0.01).to(torch.uint8)
            st["wt"] = (0.5 + 0.5 * _uni(g, ch, _n_bl(na), 2)).float()
    if op == "calsolve":
        st["V"], st["M"], st["g0"] = _calibration(na, case["channels"], seed, outliers=1e-3)
        st["g"] = torch.empty_like(st["g0"])
        st["flags"] = torch.empty((case["channels"], _n_bl(na), 2), dtype=torch.uint8, device=DEV)
    if op == "image":
        b = case["subbands"]
        st["imager"] = afc.Imager(_positions(na, seed), b, case["grid"])
        vis = torch.empty(afc.visibility_shape(b, na), dtype=torch.float32, device=DEV)
        for k in range(b):
            g = _gen(seed, 111, k)
            vis[k] = 20.0 * _rnd(g, *vis.shape[1:])
            sky = torch.view_as_real(_sky(na, P, seed, NU0 + k * SUBBAND_HZ)).float()
            vis[k, :, :, 0, 0] += sky
            vis[k, :, :, 1, 1] += sky
        st["vis"] = vis
        off = (torch.arange(P, device=DEV).double() + P // 2) % P - P // 2
        st["freq"] = torch.stack([NU0 + k * SUBBAND_HZ + off * SUBBAND_HZ / P for k in range(b)]).contiguous()
        st["weights"] = torch.randint(2500, 3052, (b, _n_bl(na)), generator=_gen(seed, 112), device=DEV).to(torch.int32)
        st["grid"] = torch.empty((case["grid"], case["grid"], 2), dtype=torch.float32, device=DEV)
        st["image"] = torch.empty((case["grid"], case["grid"]), dtype=torch.float32, device=DEV)
    return st


def run(st):
    op, case = st["op"], st["case"]
    if op == "channelise":
        return afc.channelise(st["x"], st["taps"], case["spectra"], case["dtype"], st["gain"], out=st["z"])
    if op == "fine":
        return afc.channelise_fine(st["x"], st["taps"], case["spectra"], st["delays"], st["bandpass"], st["center"],
                                   out_dtype=case["dtype"], gain=st["gain"], out=st["z"], workspace=st["ws"])
    if op in ("fx", "correlate"):
        if op == "fx":
            afc.channelise(st["x"], st["taps"], case["spectra"], case["dtype"], st["gain"], out=st["z"])
        return afc.correlate(st["z"], case["spectra"], st["S"], st["flags"], out=st["vis"], weights=st["weights"])
    if op == "plan":
        st["plan"].launch(st["x"], st["taps"], [st["gain"]] * case["subbands"], st["ws"], st["vis"], st["flags"],
                          st["weights"])
        vis = [st["vis"][k] if t == "i8" else st["vis"][k].view(torch.float32) for k, t in enumerate(_mix(case))]
        return vis, st["weights"]
    if op == "lost":
        s = case["spectra"]
        afc.validity(st["packets"], s, PACKET, P, out=st["spec"])
        afc.zero_invalid(st["z"], st["spec"], s)
        afc.validity_weights(st["spec"], s, out=st["weights"])
        afc.normalise_visibilities(st["vis"], st["weights"], out=st["mean"])
        return st["spec"], st["z"], st["weights"], st["mean"]
    if op == "calgrad":
        st["g"].grad = None
        loss = afc.cal_loss(st["V"], st["M"], st["g"], st["flags"], st["wt"])
        loss.sum().backward()
        return loss.detach(), st["g"].grad
    if op == "calsolve":
        afc.sigma_clip(st["V"], out=st["flags"])
        st["g"].copy_(st["g0"])
        loss = afc.calibrate_solve(st["V"], st["M"], st["g"], n_iter=case["iterations"], flags=st["flags"])
        return st["flags"], st["g"], loss
    if op == "image":
        st["imager"].grid(st["vis"], st["freq"], st["weights"], out=st["grid"])
        st["imager"].image(st["grid"], out=st["image"])
        return st["grid"], st["image"]
    raise ValueError(op)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    op, na = case["op"], case["antennas"]
    n, nbl = 2 * na, _n_bl(na)
    size = {"i8": 2, "f16": 4, "f32": 8}                       # bytes of a complex sample
    if op in ("calgrad", "calsolve"):
        ch = case["channels"]
        data = ch * nbl * 2 * 2 * 8                            # XX and YY of V and M
        if op == "calgrad":
            return {"bytes": data + ch * na * 2 * 8 * 2 + (ch * nbl * 2 * 5 if case["weighted"] else 0),
                    "flops": ch * nbl * 2 * 40}
        it = case["iterations"]
        return {"bytes": data + ch * nbl * 2 + ch * na * 2 * 8 * 2, "flops": ch * nbl * 2 * (40 * (it + 1) + 12)}
    b = case["subbands"]
    if op == "image":
        g = case["grid"]
        return {"bytes": b * P * nbl * 16 + b * nbl * 4 + g * g * (8 + 4),
                "flops": b * P * nbl * 60 + 10 * g * g * math.log2(g)}
    s = case["spectra"]
    if op == "lost":
        z = b * P * s * n * size[case["dtype"]] // 200         # the lost part
        return {"bytes": b * (s + T - 1) * P // PACKET * na + b * s * na // 8 + z + b * nbl * 4 + 2 * b * P * nbl * 32,
                "flops": b * P * nbl * 8 + b * nbl * s // 16}
    lengths = _lengths(case) if op in ("fx", "plan") else [s] * b
    types = _mix(case) if op == "plan" else [case["dtype"]] * b
    bytes_, flops = 0, 0
    for k, t in zip(lengths, types):
        if op == "fx":                                         # every subband is channelised in full
            bytes_ += (s + T - 1) * P * n * 4
            flops += 94 * s * P * n
        elif op in ("channelise", "plan"):
            bytes_ += (k + T - 1) * P * n * 4
            flops += 94 * k * P * n
        elif op == "fine":
            bytes_ += (k + T - 1) * FINE * n * 4
            flops += (64 + 40 + 8) * k * FINE * n
        if op in ("channelise", "fine", "correlate"):
            bytes_ += k * P * n * size[t]
        if op in ("fx", "correlate", "plan"):
            bytes_ += P * nbl * 32 + nbl * 4
            flops += 8 * P * k * (n * (n + 1) // 2)
    return {"bytes": bytes_, "flops": flops}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _dft(n):
    k = torch.arange(n, device=DEV, dtype=torch.float64)
    return torch.polar(torch.ones((n, n), dtype=torch.float64, device=DEV), -2.0 * math.pi * (torch.outer(k, k) % n) / n)


def _bank(x, taps, s, channels):
    """Filter bank of one subband: int16 [L][na][2][2] -> complex128 [s][n][channels]."""
    rows, n = x.shape[0], x.shape[1] * 2
    h = taps.double().view(T, channels)
    out = torch.empty((s, n, channels), dtype=torch.complex128, device=DEV)
    w = _dft(channels)
    step = max(1, (1 << 25) // (n * channels))
    for r in range(0, s, step):
        k = min(s, r + step) - r
        v = torch.view_as_complex(x[r * channels:(r + k + T - 1) * channels].double().view(k + T - 1, channels, n, 2))
        u = sum(h[t][None, :, None] * v[t:t + k] for t in range(T))
        out[r:r + k] = u.permute(0, 2, 1).contiguous() @ w
    return out


def _blocks(y):
    """complex [s][n][P] -> real [P][Sb][n][8][2]."""
    s, n, ch = y.shape
    sb = -(-s // 8)
    z = torch.zeros((sb * 8, n, ch), dtype=y.dtype, device=DEV)
    z[:s] = y
    return torch.view_as_real(z.view(sb, 8, n, ch).permute(3, 0, 2, 1).contiguous())


def _correlations(z, s, flags):
    """complex128 [P][s][n] -> float64 [P][Nbl][2][2][2]."""
    n = z.shape[2]
    na = n // 2
    a, c = _pairs(na)
    out = torch.empty((P, a.numel(), 2, 2), dtype=torch.complex128, device=DEV)
    for k in range(P):
        zt = z[k, :s].T.contiguous()
        v = zt @ zt.conj().resolve_conj().T.contiguous()
        v.diagonal().imag.zero_()
        out[k] = v.view(na, 2, na, 2).permute(0, 2, 1, 3)[a, c]
    if flags is not None:
        out[:, (flags[a] | flags[c]) != 0] = 0
    return torch.view_as_real(out)


def exact(case, seed):
    op, na = case["op"], case["antennas"]
    if case.get("dtype") == "i8" and op != "lost":
        return None                                            # whole numbers
    if op == "calgrad":
        return _exact_calgrad(case, seed)
    if op == "calsolve":
        return _exact_calsolve(case, seed)
    if op == "image":
        return _exact_image(case, seed)
    st = prepare(case, seed)
    s, b = case["spectra"], case["subbands"]
    if op == "channelise":
        return torch.stack([_blocks(_bank(st["x"][k], st["taps"], s, P)) for k in range(b)])
    if op == "fine":
        off = (torch.arange(FINE, device=DEV).double() + FINE // 2) % FINE - FINE // 2
        got = []
        for k in range(b):
            y = _bank(st["x"][k], st["taps"], s, FINE)
            turns = (st["center"][k] + off * SUBBAND_HZ / FINE)[None, :] * st["delays"][:, None]
            y *= torch.polar(st["bandpass"].double().expand_as(turns).contiguous(), 2.0 * math.pi * (turns - turns.floor()))
            got.append(_blocks(y.view(s, 2 * na, P, 4).sum(-1)))
        return torch.stack(got)
    if op == "fx":
        out = []
        for k in range(b):
            y = _bank(st["x"][k], st["taps"], s, P)
            if case["dtype"] == "f16":
                y = torch.view_as_complex(torch.view_as_real(y).half().double())
            out.append(_correlations(y.permute(2, 0, 1).contiguous(), st["S"][k],
                                     None if st["flags"] is None else st["flags"][k]))
        return torch.stack(out), None
    if op == "correlate":
        out = torch.empty(st["vis"].shape, dtype=torch.float64, device=DEV)
        for k in range(b):
            z = torch.view_as_complex(st["z"][k].permute(0, 1, 3, 2, 4).reshape(P, -1, 2 * na, 2).double())
            out[k] = _correlations(z, s, None if st["flags"] is None else st["flags"][k])
        return out, None
    if op == "plan":
        out = []
        for k, (t, length) in enumerate(zip(_mix(case), _lengths(case))):
            if t == "i8":
                out.append(None)
                continue
            y = _bank(st["x"][k], st["taps"], length, P)
            y = torch.view_as_complex(torch.view_as_real(y).half().double())
            out.append(_correlations(y.permute(2, 0, 1).contiguous(), length,
                                     None if st["flags"] is None else st["flags"][k]))
        return out, None
    if op == "lost":
        # valid spectra from the packets' arrival, then the mean per baseline
        a, c = _pairs(na)
        step = P // PACKET
        mean = torch.empty(st["vis"].shape, dtype=torch.float64, device=DEV)
        for k in range(b):
            lost = (st["packets"][k] == 0).float().view(s + T - 1, step, na).amax(1)        # per input spectrum
            bad = torch.nn.functional.max_pool1d(lost.T[None], T, 1)[0].T                   # [s][na]
            v = (bad < 0.5).double()
            w = (v.T.contiguous() @ v)[a, c]
            mean[k] = torch.where(w > 0, 1.0 / w.clamp(min=1.0), 0.0)[None, :, None, None, None] * st["vis"][k].double()
        return None, None, None, mean
    return None


def _square(t, na):
    """Lower triangle [Nbl] complex128 -> Hermitian [na][na]."""
    a, c = _pairs(na)
    f = torch.zeros((na, na), dtype=torch.complex128, device=DEV)
    f[c, a] = t.conj()
    f[a, c] = t
    return f


def _full(v, k, p, na):
    return _square(torch.view_as_complex(v[k, :, p, p].double()), na)


def _exact_calgrad(case, seed):
    na, ch = case["antennas"], case["channels"]
    st = prepare(case, seed)
    g = st["g"].detach().to(torch.complex128)
    loss = torch.empty((ch, 2), dtype=torch.float64, device=DEV)
    grad = torch.empty_like(g)
    for k in range(ch):
        for p in range(2):
            v, m = _full(st["V"], k, p, na), _full(st["M"], k, p, na)
            r = v - g[k, :, p, None] * m * g[k, None, :, p].conj()
            w = torch.ones((na, na), dtype=torch.float64, device=DEV)
            if case["weighted"]:
                w = _square(torch.where(st["flags"][k, :, p] != 0, 0.0, st["wt"][k, :, p].double()).to(torch.complex128),
                            na).real
            loss[k, p] = (w * (r.real ** 2 + r.imag ** 2)).sum()
            grad[k, :, p] = -4.0 * (w * r * m.conj()) @ g[k, :, p]
    return loss, torch.view_as_real(grad)


def _exact_calsolve(case, seed):
    na, ch, nbl = case["antennas"], case["channels"], _n_bl(case["antennas"])
    st = prepare(case, seed)
    a, c = _pairs(na)
    cross = (a != c)
    power = torch.stack([(st["V"][:, :, p, p].double() ** 2).sum(-1) for p in range(2)], -1)      # [ch][nbl][2]
    k2 = 25.0
    flag = (power > k2 * (power * cross[None, :, None]).sum(1, keepdim=True) / (nbl - na)) & cross[None, :, None]
    keep = (~flag).double()
    flag |= (power > k2 * (power * keep).sum(0, keepdim=True) / keep.sum(0, keepdim=True).clamp(min=1)) & cross[None, :, None]
    out = torch.empty((ch, na, 2), dtype=torch.complex128, device=DEV)
    loss = torch.empty((ch, 2), dtype=torch.float64, device=DEV)
    for k in range(ch):
        for p in range(2):
            w = _square((~flag[k, :, p]).to(torch.complex128), na).real
            v, m = _full(st["V"], k, p, na) * w, _full(st["M"], k, p, na) * w
            g = torch.ones(na, dtype=torch.complex128, device=DEV)
            m2 = m.real ** 2 + m.imag ** 2
            for i in range(1, case["iterations"] + 1):
                d = m2 @ (g.real ** 2 + g.imag ** 2)
                new = torch.where(d > 0, ((v * m.conj()) @ g) / torch.where(d > 0, d, 1.0), g)
                g = 0.5 * (new + g) if i % 2 == 0 else new
            g = g * (g[0].conj() / g[0].abs())
            out[k, :, p] = g
            r = v - g[:, None] * m * g[None, :].conj()
            loss[k, p] = (r.real ** 2 + r.imag ** 2).sum()
    return None, torch.view_as_real(out), loss


def _exact_image(case, seed):
    na, b, size = case["antennas"], case["subbands"], case["grid"]
    st = prepare(case, seed)
    pos = _positions(na, seed)
    a, c = _pairs(na)
    cross = a != c
    a, c = a[cross], c[cross]
    d = pos[a] - pos[c]
    re = torch.zeros(size * size, dtype=torch.float64, device=DEV)
    im = torch.zeros_like(re)
    norm = torch.zeros((), dtype=torch.float64, device=DEV)
    for k in range(b):
        w = st["weights"][k][cross].double()
        for f in range(P):
            v = st["vis"][k, f][cross].double()
            v = 0.5 * (v[:, 0, 0] + v[:, 1, 1])
            uv = d * st["freq"][k, f] / C_LIGHT * 2.0 + 0.5 * size
            lo = uv.floor()
            ok = ((lo >= 1) & (lo <= size - 2)).all(1)
            lo, fr, vv, ww = lo[ok].long(), (uv - lo)[ok], v[ok], w[ok]
            norm += 2.0 * ww.sum()
            for y in range(2):
                for x in range(2):
                    s = ww * (fr[:, 0] if x else 1.0 - fr[:, 0]) * (fr[:, 1] if y else 1.0 - fr[:, 1])
                    i, j = lo[:, 0] + x, lo[:, 1] + y
                    here, there = j * size + i, (size - j) * size + (size - i)
                    re.index_add_(0, here, s * vv[:, 0])
                    im.index_add_(0, here, s * vv[:, 1])
                    re.index_add_(0, there, s * vv[:, 0])
                    im.index_add_(0, there, -s * vv[:, 1])
    grid = torch.stack([re, im], 1).view(size, size, 2)
    g = np.fft.ifftshift(torch.view_as_complex(grid.contiguous()).cpu().numpy())
    image = np.fft.fftshift(np.fft.fft2(g)).real / float(norm)
    return grid, torch.from_numpy(np.ascontiguousarray(image)).to(DEV)
