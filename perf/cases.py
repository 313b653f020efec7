"""Workloads of the correlator library, for timing and for comparing results.

Each case is one piece of work that a program built on the package has it do,
through the public entry points of ``paper_2303_11557_amd``:

  step    one block of voltages through a plan: channelise, correlate, emit
  chan    data channelised elsewhere through the X-engine: load, correlate, emit
  beam    tied-array beams of a channelised block
  incoh   the incoherent beam of a channelised block
  post    occupancy weights and weighted channel averaging of visibilities
  batch   several uneven plans driven as one unit of device work

``listed`` holds named cases, ``draw`` makes others of the same ranges,
``prepare`` the inputs and plans a program has in hand, ``run`` one pass,
``work`` the bytes and operations the pass cannot do without, and ``exact`` its
results in 64 bits from plain torch.
"""
import math

import torch

from paper_2303_11557_amd import mwax
from paper_2303_11557_amd.mwax import Batch, Plan, make_config

F_S = 1.28e6                 # samples per second of a coarse channel
SKY_HZ = 121 * 1.28e6        # sky frequency of coarse channel 121
SUB_BLOCK = 64000            # samples of a 50 ms sub-block (lost packets zero whole sub-blocks)


# -- cases -------------------------------------------------------------------

def step(n_tiles, L, T, ints, prec, calls=1, order="tri", delays=False, average="no", F=1, weights=False):
    return {"kind": "step", "n_tiles": n_tiles, "L": L, "T": T, "ints": ints, "prec": prec, "calls": calls,
            "order": order, "delays": delays, "average": average, "F": F, "weights": weights}


def chan(n_tiles, L, T, ints, prec, order="tri"):
    return {"kind": "chan", "n_tiles": n_tiles, "L": L, "T": T, "ints": ints, "prec": prec, "order": order}


def beam(n_tiles, L, M, n_beams, prec):
    return {"kind": "beam", "n_tiles": n_tiles, "L": L, "M": M, "n_beams": n_beams, "prec": prec}


def incoh(n_tiles, L, M, t_avg, f_avg, prec):
    return {"kind": "incoh", "n_tiles": n_tiles, "L": L, "M": M, "t_avg": t_avg, "f_avg": f_avg, "prec": prec}


def post(n_tiles, L, F, ints, subs):
    return {"kind": "post", "n_tiles": n_tiles, "L": L, "F": F, "ints": ints, "subs": subs}


def batch(instances, samples, prec):
    """instances: "tiles/L/integrations, ..."; every instance takes `samples` samples per call."""
    return {"kind": "batch", "instances": instances, "samples": samples, "prec": prec}


def listed():
    return [
        # a handful of tiles for a moment: what an operator's check or a unit of a test does, where only
        # latency and the number of launches count (4 tiles, 5 ms of 10 kHz channels)
        {"name": "check_4t_int8", **step(4, 128, 50, 1, "int8")},
        # the plain FP32 path on a small array: 16 tiles, 0.1 s, one integration
        {"name": "small_16t_fp32", **step(16, 128, 1000, 1, "fp32")},
        # the FP32 path (the paper's precision) at 128 tiles: 1 s of 10 kHz channels, 0.5 s integrations
        {"name": "plain_128t_fp32", **step(128, 128, 5000, 2, "fp32")},
        # the headline: 256 tiles, 8 s of 10 kHz channels in one integration, INT8
        {"name": "headline_256t_int8", **step(256, 128, 80000, 1, "int8")},
        # binary16 at 256 tiles: 1 s calls and 2 s integrations, as a stream of blocks is processed
        {"name": "stream_256t_fp16", **step(256, 128, 20000, 1, "fp16", calls=2)},
        # the paper's fastest output mode: 6,400-point transform, 40 kHz by 250 ms, averaged in the X-engine
        {"name": "ultrafine_40khz_256t_int8", **step(256, 6400, 50, 4, "int8", average="xengine", F=200)},
        # an array with tiles out of service: 1.25 kHz channels, delays applied, 1 s integrations averaged by 8
        # at emission and divided by the occupancy weights
        {"name": "fine_93t_fp16", **step(93, 1024, 1250, 1, "fp16", delays=True, average="emission", F=8,
                                         weights=True)},
        # coarse channels of uneven arrays on one device, 0.5 s calls
        {"name": "batch_6_int8", **batch("64/32/1,128/128/2,256/1024/1,64/128/1,128/1024/1,256/32/2", 640000, "int8")},
        # an external channeliser's output ([time][channel][tile][pol]) correlated into the tile-baseline
        # order: 128 tiles, 1 s
        {"name": "loaded_128t_int8", **chan(128, 128, 10000, 1, "int8", order="tile_bl")},
        # tied-array beams: 256 tiles, 1 s, 32 beams
        {"name": "beams_256t_int8", **beam(256, 128, 10000, 32, "int8")},
        # the incoherent beam: 128 tiles, 1 s, binned by 10 spectra and 4 channels
        {"name": "incoherent_128t_fp16", **incoh(128, 128, 10000, 10, 4, "fp16")},
        # the output stage: occupancy of 8 s of 50 ms sub-blocks, 1.25 kHz channels averaged to 10 kHz
        {"name": "weights_average_256t", **post(256, 1024, 8, 1, 160)},
    ]


MOST_SAMPLES = 1 << 30       # samples of all inputs of a drawn case
MOST_CMAC = {"int8": 2e11, "fp16": 1e11, "fp32": 4e10}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "chan", "beam", "incoh", "post", "batch"))
    prec = rng.choice(("int8", "int8", "fp16", "fp32"))
    n_tiles = _log(rng, 3, 256)
    pairs = n_tiles * (2 * n_tiles + 1)
    if kind == "post":
        F = rng.choice((2, 3, 4, 5, 8, 10, 16, 25))
        most = max(2, min(1024, (1 << 30) // (8 * pairs)) // F)
        L = F * _log(rng, 2, max(3, most))
        ints = max(1, min(_log(rng, 1, 6), (1 << 30) // (8 * pairs * L)))
        return post(n_tiles, L, F, ints, rng.choice((5, 20, 40, 63, 160)))
    if kind == "batch":
        prec = rng.choice(("int8", "int8", "fp16"))
        samples = 16384 * _log(rng, 4, 24)
        n = rng.randint(2, 5)
        return batch(",".join("%d/%d/%d" % (_log(rng, 8, 128), rng.choice((32, 64, 128, 256, 512, 1024)),
                                            rng.choice((1, 1, 2))) for _ in range(n)), samples, prec)
    L = rng.choice((16, 32, 64, 128, 128, 256, 512, 1024, 6400))
    most = min(MOST_SAMPLES // (2 * n_tiles), MOST_CMAC[prec] / pairs)
    if kind in ("step", "chan") and L >= 1024:
        # short integrations of many channels: keep the output within a few GB
        most = min(most, 2.6e5) if n_tiles > 100 else most
    spectra = max(24, min(_log(rng, 40, max(41, most / L)), 200000))
    if kind == "beam":
        M = min(spectra, 1 + int(1.3e9 / (n_tiles * L * 16)))
        return beam(n_tiles, L, max(16, M), _log(rng, 1, 96), prec)
    if kind == "incoh":
        t_avg = rng.choice((1, 4, 10, 25, 100))
        M = t_avg * max(1, min(spectra, 1 + int(1.3e9 / (n_tiles * L * 16))) // t_avg)
        return incoh(n_tiles, L, M, t_avg, rng.choice((1, 2, 4, 8)), prec)
    vis = 8 * L * pairs
    ints = max(1, min(rng.choice((1, 1, 1, 2, 4)), int(3e9 // vis)))
    if kind == "chan":
        T = max(8, min(spectra, 1 + int(1.5e9 / (n_tiles * L * 16))) // ints)
        return chan(n_tiles, min(L, 1024), T, ints, prec, order=rng.choice(("tri", "tile_bl")))
    T = max(8, spectra // ints)
    average, F = "no", 1
    if L >= 512 and rng.random() < 0.7:
        average = "emission" if prec == "fp32" else rng.choice(("xengine", "xengine", "emission"))
        F = rng.choice((5, 50, 200)) if L == 6400 else rng.choice((4, 8, 16))
    calls = 1
    if rng.random() < 0.3:
        calls = 2
        T += T % 2
        ints = 1
    return step(n_tiles, L, T, ints, prec, calls=calls,
                order="tile_bl" if average == "no" and rng.random() < 0.25 else "tri",
                delays=rng.random() < 0.25, average=average, F=F, weights=average == "emission" and rng.random() < 0.5)


# -- inputs ------------------------------------------------------------------

def _gen(seed, k=0):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 64 + k)


def _volts(n_in, S, seed, k=0):
    """int8 [n_in][ld][2]: receiver noise of sigma 8, a common broad-band source with a phase per input, and
    1 % of the 50 ms sub-blocks zeroed (lost packets).  ld: S rounded up to 8 samples."""
    g = _gen(seed, k)
    ld = (S + 7) // 8 * 8
    out = torch.zeros((n_in, ld, 2), dtype=torch.int8, device="cuda")
    sky = torch.view_as_real(torch.randn((S,), generator=g, dtype=torch.complex64, device="cuda") * 3.0)
    ph = torch.rand((n_in,), generator=g, device="cuda") * (2 * math.pi)
    cs, sn = torch.cos(ph), torch.sin(ph)
    rows = max(1, min(n_in, (1 << 27) // max(1, S)))
    for n0 in range(0, n_in, rows):
        n1 = min(n_in, n0 + rows)
        x = torch.randn((n1 - n0, S, 2), generator=g, device="cuda").mul_(8.0)
        c, s = cs[n0:n1, None], sn[n0:n1, None]
        x[..., 0].addcmul_(sky[None, :, 0], c).addcmul_(sky[None, :, 1], s, value=-1.0)
        x[..., 1].addcmul_(sky[None, :, 1], c).addcmul_(sky[None, :, 0], s)
        out[n0:n1, :S] = x.round_().clamp_(-127, 127).to(torch.int8)
        del x
    blocks = S // SUB_BLOCK
    if blocks >= 2:
        lost = torch.rand((n_in, blocks), generator=g, device="cuda") < 0.01
        lost[:, 0] = False
        for n, b in lost.nonzero().tolist():
            out[n, b * SUB_BLOCK:(b + 1) * SUB_BLOCK] = 0
    return out[:, :S] if ld != S else out


def _channelised(n_in, L, M, prec, seed):
    """[M][L][n_in][2] in the element type of the precision: noise plus a common source."""
    g = _gen(seed)
    dt = {"int8": torch.int8, "fp16": torch.float16, "fp32": torch.float32}[prec]
    out = torch.empty((M, L, n_in, 2), dtype=dt, device="cuda")
    rows = max(1, (1 << 26) // (L * n_in))
    for m0 in range(0, M, rows):
        m1 = min(M, m0 + rows)
        x = torch.randn((m1 - m0, L, n_in, 2), generator=g, device="cuda")
        x += 0.3 * torch.randn((m1 - m0, L, 1, 2), generator=g, device="cuda")
        if prec == "int8":
            x = x.mul_(25.0).round_().clamp_(-127, 127)
        out[m0:m1] = x.mul_(8.0) if prec == "fp16" else (x.mul_(90.0) if prec == "fp32" else x)
    return out


def _delays(n_in, steps, seed):
    g = _gen(seed, 7)
    start = torch.rand((n_in, 1), generator=g, device="cuda") - 0.5
    rate = (torch.rand((n_in, 1), generator=g, device="cuda") - 0.5) * 1e-3
    return (start + rate * torch.arange(steps, device="cuda")).to(torch.float32).contiguous()


def _weights(ints, P, seed):
    g = _gen(seed, 9)
    return (torch.randint(120, 161, (ints, P), generator=g, device="cuda").to(torch.float32) / 160.0).contiguous()


def _scales(L, seed):
    r = torch.rand((L,), generator=torch.Generator().manual_seed(int(seed) + 3))
    return (0.5 + r).to(torch.float32).numpy()


def _beam_weights(L, n_beams, n_in, seed):
    ph = torch.rand((L, n_beams, n_in), generator=_gen(seed, 5), device="cuda") * (2 * math.pi)
    return torch.polar(torch.ones_like(ph), ph).contiguous()


def _step_samples(L):
    return L * max(1, 6400 // L)


def _instances(c):
    return [tuple(int(v) for v in w.split("/")) for w in c["instances"].split(",")]


def _batch_T(c, L, ints):
    return c["samples"] // L // ints


def prepare(c, seed):
    k = c["kind"]
    if k == "post":
        n_in, L, ints = 2 * c["n_tiles"], c["L"], c["ints"]
        P = n_in * (n_in + 1) // 2
        g = _gen(seed)
        vis = torch.randn((ints, L, P), generator=g, dtype=torch.complex64, device="cuda")
        flags = (torch.rand((n_in, ints * c["subs"]), generator=g, device="cuda") < 0.01).to(torch.uint8)
        return {"case": c, "vis": vis, "flags": flags}
    if k == "batch":
        inst = _instances(c)
        S = c["samples"]
        cfgs = [make_config(t, L=L, T=_batch_T(c, L, i), xprec=c["prec"], max_samples=_batch_T(c, L, i) * i * L)
                for t, L, i in inst]
        volts = [_volts(2 * t, _batch_T(c, L, i) * i * L, seed, n) for n, (t, L, i) in enumerate(inst)]
        return {"case": c, "batch": Batch(cfgs), "volts": volts, "ints": [i for _, _, i in inst], "S": S}
    n_in, L = 2 * c["n_tiles"], c["L"]
    if k in ("beam", "incoh"):
        M = c["M"]
        p = Plan(make_config(c["n_tiles"], L=L, T=M, xprec=c["prec"], max_samples=M * L))
        if c["prec"] == "int8":
            p.set_scales(_scales(L, seed))
        p.load_channelised(_channelised(n_in, L, M, c["prec"], seed))
        w = _beam_weights(L, c["n_beams"], n_in, seed) if k == "beam" else None
        return {"case": c, "plan": p, "w": w}
    T, ints = c["T"], c["ints"]
    if k == "chan":
        p = Plan(make_config(c["n_tiles"], L=L, T=T, xprec=c["prec"], max_samples=T * ints * L))
        return {"case": c, "plan": p, "x": _channelised(n_in, L, T * ints, c["prec"], seed)}
    S = T * ints * L
    p = Plan(make_config(c["n_tiles"], L=L, T=T, xprec=c["prec"], max_samples=S // c["calls"]))
    s = {"case": c, "plan": p, "volts": _volts(n_in, S, seed)}
    if c["average"] == "xengine":
        p.set_averaging(c["F"])
    if c["delays"]:
        st = _step_samples(L)
        s["delays"] = _delays(n_in, (S + st - 1) // st, seed)
    if c["weights"]:
        s["weights"] = _weights(ints, p.P, seed)
    return s


def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "post":
        w = mwax.vis_weights(s["flags"], c["subs"])
        return [w, mwax.fscrunch(s["vis"], c["F"], weights=w)]
    if k == "batch":
        b = s["batch"]
        b.run(s["volts"])
        return [p.integrate(i) for p, i in zip(b.plans, s["ints"])]
    p = s["plan"]
    if k == "beam":
        return p.beamform(s["w"])
    if k == "incoh":
        return p.beamform_incoherent(c["t_avg"], c["f_avg"])
    if k == "chan":
        p.load_channelised(s["x"])
        p.correlate()
        return p.integrate(c["ints"], order=c["order"])
    if c["delays"]:
        # the table belongs to this observation: it starts at the plan's current position
        p.set_delays(s["delays"], step_samples=_step_samples(c["L"]), sky_freq_hz=SKY_HZ)
    v = s["volts"]
    n = v.shape[1] // c["calls"]
    for q in range(c["calls"]):
        p.channelise(v[:, q * n:(q + 1) * n])
        p.correlate()
    if c["average"] == "emission":
        return p.integrate_averaged(c["F"], c["ints"], weights=s.get("weights"))
    return p.integrate(c["ints"], order=c["order"])


# -- what a pass cannot do without --------------------------------------------

ELEM = {"int8": 2, "fp16": 4, "fp32": 8}     # bytes of a channelised complex sample


def _fft_flops(samples, L):
    return 5.0 * samples * math.log2(L) if L > 1 else 0.0


def work(c):
    k = c["kind"]
    if k == "batch":
        got = {"bytes": 0.0, "flops": 0.0}
        for t, L, i in _instances(c):
            w = work(step(t, L, _batch_T(c, L, i), i, c["prec"]))
            got = {q: got[q] + w[q] for q in got}
        return got
    n_in, L = 2 * c["n_tiles"], c["L"]
    P = n_in * (n_in + 1) // 2
    if k == "post":
        vis = 8.0 * c["ints"] * L * P
        return {"bytes": vis + vis / c["F"] + 4.0 * c["ints"] * P + n_in * c["ints"] * c["subs"],
                "flops": 2.0 * c["ints"] * L * P}
    if k == "beam":
        x = float(n_in) * L * c["M"]
        return {"bytes": x * ELEM[c["prec"]] + 8.0 * L * c["n_beams"] * (n_in + c["M"]), "flops": 8.0 * x * c["n_beams"]}
    if k == "incoh":
        x = float(n_in) * L * c["M"]
        return {"bytes": x * ELEM[c["prec"]] + 8.0 * L * c["M"] / (c["t_avg"] * c["f_avg"]), "flops": 4.0 * x}
    S = float(c["T"] * c["ints"] * L)
    out = 8.0 * c["ints"] * P * L
    if k == "chan":
        return {"bytes": n_in * S * ELEM[c["prec"]] + out, "flops": 8.0 * P * S}
    if c["average"] != "no":
        out /= c["F"]
    return {"bytes": 2.0 * n_in * S + out, "flops": 8.0 * P * S + _fft_flops(n_in * S, L)}


# -- results in 64 bits -------------------------------------------------------

def _spectra(v, L, m0, m1, delays=None, dsteps=0):
    """Frames m0 .. m1 - 1 of voltages [n][S][2] -> complex128 [n][m1 - m0][L], DC at channel L/2."""
    x = torch.view_as_complex(v[:, m0 * L:m1 * L].to(torch.float64).contiguous()).reshape(v.shape[0], m1 - m0, L)
    x = torch.fft.fftshift(torch.fft.fft(x, dim=2), dim=2) if L > 1 else x
    if delays is not None:
        frames = torch.arange(m0, m1, device="cuda") * L // dsteps
        d = delays[:, frames].to(torch.float64)                                  # [n][m]
        f = (torch.arange(L, device="cuda", dtype=torch.float64) - L // 2) / L + SKY_HZ / F_S
        turns = d[:, :, None] * f[None, None, :]
        x = x * torch.polar(torch.ones_like(turns), -2 * math.pi * (turns - turns.round()))
    return x


def _herk(x):
    """sum over m of x_i conj(x_j), [c][n][m] complex128 -> [c][n][n]."""
    r, i = x.real.contiguous(), x.imag.contiguous()
    rt, it = r.transpose(1, 2).contiguous(), i.transpose(1, 2).contiguous()
    return torch.complex(torch.bmm(r, rt) + torch.bmm(i, it), torch.bmm(i, rt) - torch.bmm(r, it))


def _average(v, F):
    """Channel averaging of [L][P] (see mwax_fscrunch) in 64 bits."""
    L = v.shape[0]
    if F == 1:
        return v
    N, half = L // F, F // 2
    out = torch.zeros((N, v.shape[1]), dtype=v.dtype, device=v.device)
    base = L // 2 + (torch.arange(N, device=v.device) - N // 2) * F
    for d in range(-half, half + 1):
        w = torch.full((N, 1), 0.5 if F % 2 == 0 and abs(d) == half else 1.0, dtype=torch.float64, device=v.device)
        if d == 0:
            w[N // 2] = 0.0
        out += w * v[(base + d) % L]
    div = torch.full((N, 1), float(F), dtype=torch.float64, device=v.device)
    div[N // 2] = F - 1
    return out / div


def _tile_bl(full):
    """[L][n][n] -> [n_baselines][L][4] (XX, XY, YX, YY of tiles a >= b)."""
    n = full.shape[1]
    a, b = torch.tril_indices(n // 2, n // 2, device="cuda")
    return torch.stack([full[:, 2 * a + p, 2 * b + q].t() for p in (0, 1) for q in (0, 1)], 2)


def _visibilities(spectra_of, n_in, L, T, j, order, F, weights):
    """Integration j in 64 bits; spectra_of(m0, m1) -> complex128 [n][m][L]."""
    full = torch.zeros((L, n_in, n_in), dtype=torch.complex128, device="cuda")
    chunk = max(1, min(T, int(2.0e8 // (n_in * L)) or 1))
    for m in range(0, T, chunk):
        x = spectra_of(j * T + m, j * T + min(T, m + chunk)).permute(2, 0, 1)      # [c][n][m]
        for c0 in range(0, L, 256):
            full[c0:c0 + 256] += _herk(x[c0:c0 + 256])
    if order == "tile_bl":
        return _tile_bl(full)
    i1, i2 = torch.tril_indices(n_in, n_in, device="cuda")
    v = torch.empty((L, i1.numel()), dtype=torch.complex128, device="cuda")
    for c0 in range(0, L, 256):
        v[c0:c0 + 256] = full[c0:c0 + 256, i1, i2]
    v = _average(v, F)
    return v if weights is None else v / weights[j].to(torch.float64)


def _exact_step(c, seed, k=0):
    n_in, L, T = 2 * c["n_tiles"], c["L"], c["T"]
    if 16.0 * L * n_in * n_in > 4e10:
        return None
    S = T * c["ints"] * L
    v = _volts(n_in, S, seed, k)
    st = _step_samples(L)
    d = _delays(n_in, (S + st - 1) // st, seed) if c["delays"] else None
    w = _weights(c["ints"], n_in * (n_in + 1) // 2, seed) if c["weights"] else None
    return torch.stack([_visibilities(lambda a, b: _spectra(v, L, a, b, d, st), n_in, L, T, j, c["order"], c["F"], w)
                        for j in range(c["ints"])])


def _post_scale(L, prec):
    """What a loaded binary16 value is multiplied by: spectra were stored times 2^-e."""
    lg = max(0, (L - 1).bit_length())
    return 2.0 ** ((lg + 1) // 2) if prec == "fp16" else 1.0


def exact(c, seed):
    k = c["kind"]
    if k == "batch":
        return [_exact_step(step(t, L, _batch_T(c, L, i), i, c["prec"]), seed, n)
                for n, (t, L, i) in enumerate(_instances(c))]
    n_in, L = 2 * c["n_tiles"], c["L"]
    if k == "step":
        return _exact_step(c, seed)
    if k == "post":
        s = prepare(c, seed)
        ok = 1.0 - s["flags"].to(torch.float64).reshape(n_in, c["ints"], c["subs"])
        a = ok.permute(1, 0, 2).contiguous()
        i1, i2 = torch.tril_indices(n_in, n_in, device="cuda")
        w = (torch.bmm(a, a.transpose(1, 2).contiguous()) / c["subs"])[:, i1, i2]
        out = []
        for j in range(c["ints"]):
            v = _average(s["vis"][j].to(torch.complex128), c["F"])
            out.append(v / torch.where(w[j] > 0, w[j], torch.ones_like(w[j])))
        return [w, torch.stack(out)]
    post_scale = _post_scale(L, c["prec"])
    if k == "chan":
        T, ints = c["T"], c["ints"]
        if 16.0 * L * n_in * n_in > 4e10:
            return None
        x = _channelised(n_in, L, T * ints, c["prec"], seed)

        def spectra_of(a, b):
            return torch.view_as_complex(x[a:b].to(torch.float64)).permute(2, 0, 1) * post_scale

        return torch.stack([_visibilities(spectra_of, n_in, L, T, j, c["order"], 1, None) for j in range(ints)])
    M = c["M"]
    x = _channelised(n_in, L, M, c["prec"], seed)
    sc = torch.full((L,), post_scale, dtype=torch.float64, device="cuda")
    if c["prec"] == "int8":
        sc = torch.from_numpy(_scales(L, seed)).cuda().to(torch.float64)
    rows = max(1, int(1e8 // (L * n_in)))
    if k == "incoh":
        rows = max(1, rows // c["t_avg"]) * c["t_avg"]
        out = []
        for m in range(0, M, rows):
            y = x[m:m + rows].to(torch.float64)
            pw = (y * y).sum(3).reshape(y.shape[0], L, n_in // 2, 2).sum(2) * (sc * sc)[None, :, None]
            out.append(pw.reshape(-1, c["t_avg"], L // c["f_avg"], c["f_avg"], 2).sum((1, 3)))
        return torch.cat(out)
    w = _beam_weights(L, c["n_beams"], n_in, seed).to(torch.complex128).permute(0, 2, 1).contiguous()   # [L][n][b]
    wr, wi = w.real.contiguous(), w.imag.contiguous()
    out = torch.empty((M, L, c["n_beams"]), dtype=torch.complex128, device="cuda")
    for m in range(0, M, rows):
        y = x[m:m + rows].to(torch.float64) * sc[None, :, None, None]
        yr, yi = y[..., 0].permute(1, 0, 2).contiguous(), y[..., 1].permute(1, 0, 2).contiguous()        # [L][m][n]
        b = torch.complex(torch.bmm(yr, wr) - torch.bmm(yi, wi), torch.bmm(yr, wi) + torch.bmm(yi, wr))
        out[m:m + rows] = b.permute(1, 0, 2)
    return out
