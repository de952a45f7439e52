"""Performance cases of the X-engine: the work a node's program has it do.

Every case is one pass through the public entry points on data that is
already on the GPU (samples arrive there from the network), with the
correlator, the beam set or the prepared batch that such a program keeps
between passes.  Integrations end with the export that resets the slot, so
each pass starts from cleared accumulators and returns whole visibilities.

Samples are CHIME-shaped (receiver noise, a weak common sky signal with a
geometric phase per input and a few narrow-band tones, scaled by 3, rounded
and clipped to [-7, 7]); the flagged case adds carriers and impulsive bursts
in whole (block, input) cells.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2005_09481_amd import xeng

FRAME = 256          # samples per streaming frame
CHUNK = 4096         # samples generated or contracted at a time


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one channel of a small array, alone: latency and launch count
        {"name": "channel_n64", "kind": "channel", "n": 64, "t": 4096, "re_low": False},
        # one channel of a pathfinder-sized array
        {"name": "channel_n512", "kind": "channel", "n": 512, "t": 8192, "re_low": False},
        # one CHIME channel, 84 ms of samples: the headline workload
        {"name": "channel_n2048", "kind": "channel", "n": 2048, "t": 32768, "re_low": False},
        # an array whose inputs are no multiple of 16, real part in the low nibble
        {"name": "channel_n1000", "kind": "channel", "n": 1000, "t": 32768, "re_low": True},
        # the channels one GPU serves, uneven integrations, one batched call and one batched export
        {"name": "channels16", "kind": "batch", "mix": "channels", "jobs": 16, "n": 2048, "t": 16384, "salt": 3},
        # independent sub-arrays of uneven size and length in one batched call
        {"name": "subarrays64", "kind": "batch", "mix": "subarrays", "jobs": 64, "n": 2048, "t": 16384, "salt": 4},
        # every channel of a small array in one prepared launch, then their exports
        {"name": "narrow1024", "kind": "prepared", "jobs": 1024, "n": 64, "t": 4096},
        # continuous batching: each launch integrates the few frames that arrived, the exports follow
        {"name": "stream32", "kind": "stream", "jobs": 32, "n": 2048, "frames": 4, "launches": 4},
        # RFI excision, then flag-aware correlation with sample counts
        {"name": "flagged_n2048", "kind": "flagged", "n": 2048, "t": 32768, "block": 256},
        # the unsigned form with pre-sums
        {"name": "presum_n2048", "kind": "presum", "n": 2048, "t": 32768},
        # the ten pulsar beams of a CHIME channel, exact sums
        {"name": "beams10_exact", "kind": "beams", "n": 2048, "t": 32768, "beams": 10, "shift": -1},
        # beams of an array of odd size, 8 + 8-bit export
        {"name": "beams16_8bit", "kind": "beams", "n": 1000, "t": 16384, "beams": 16, "shift": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cap_t(n, t, cmacs):
    """The longest integration up to t whose correlation stays below `cmacs`."""
    return max(64, min(t, int(cmacs // (n * (n + 1) // 2))))


def draw(rng):
    kind = rng.choice(["channel", "channel", "channel", "batch", "prepared", "stream", "flagged", "presum", "beams"])
    if kind == "channel":
        n = _log(rng, 16, 4096)
        if rng.random() < 0.6:
            n = max(16, n // 16 * 16)
        return {"kind": kind, "n": n, "t": _cap_t(n, _log(rng, 256, 65536), 1.2e11), "re_low": rng.random() < 0.3}
    if kind == "batch":
        return {"kind": kind, "mix": rng.choice(["channels", "subarrays"]), "jobs": rng.randint(2, 16),
                "n": 16 * _log(rng, 8, 128), "t": _log(rng, 1024, 12000), "salt": rng.randrange(1 << 20)}
    if kind == "prepared":
        return {"kind": kind, "jobs": _log(rng, 8, 768), "n": rng.choice([16, 32, 48, 64]), "t": _log(rng, 256, 4096)}
    if kind == "stream":
        return {"kind": kind, "jobs": rng.randint(2, 16), "n": 16 * _log(rng, 16, 128), "frames": rng.randint(1, 8),
                "launches": rng.randint(1, 4)}
    if kind == "flagged":
        n = _log(rng, 64, 2048)
        if rng.random() < 0.7:
            n = max(64, n // 16 * 16)
        return {"kind": kind, "n": n, "t": _log(rng, 1024, 32768), "block": rng.choice([64, 100, 256, 512])}
    if kind == "presum":
        n = _log(rng, 96, 2048)
        if rng.random() < 0.7:
            n = n // 16 * 16
        return {"kind": kind, "n": n, "t": _log(rng, 512, 32768)}
    n = _log(rng, 64, 4096)
    if rng.random() < 0.6:
        n = max(64, n // 16 * 16)
    return {"kind": "beams", "n": n, "t": _log(rng, 256, 32768), "beams": rng.randint(1, 16),
            "shift": rng.choice([-1, 6, 10])}


def _jobs(case):
    """(N, T) of every job of a batched case."""
    kind = case["kind"]
    if kind == "prepared":
        return [(case["n"], case["t"])] * case["jobs"]
    if kind == "stream":
        return [(case["n"], case["frames"] * case["launches"] * FRAME)] * case["jobs"]
    if kind != "batch":
        return [(case["n"], case["t"])]
    rng = random.Random(case["salt"])
    out = []
    for _ in range(case["jobs"]):
        if case["mix"] == "channels":
            out.append((case["n"], rng.randint(max(1, case["t"] // 8), case["t"])))
        else:
            out.append((max(16, case["n"] >> rng.randint(0, 3)), max(64, case["t"] >> rng.randint(0, 2))))
    return out


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _generator(seed):
    return torch.Generator(device=_device()).manual_seed(int(seed) & 0x7FFFFFFF)


def _pack(re, im, re_low):
    re, im = (re + 8).to(torch.uint8), (im + 8).to(torch.uint8)
    return (im << 4) | re if re_low else (re << 4) | im


def _samples(gen, n, t, re_low=False):
    """uint8 [t, n]: CHIME-shaped 4+4-bit samples."""
    dev = _device()
    out = torch.empty((t, n), dtype=torch.uint8, device=dev)
    phase = 2 * math.pi * 0.01 * (torch.arange(n, device=dev) % 256).float()
    gr, gi = torch.cos(phase), torch.sin(phase)
    theta = 2 * math.pi * torch.rand((3, n), generator=gen, device=dev)
    for t0 in range(0, t, CHUNK):
        tc = min(CHUNK, t - t0)
        re = torch.randn((tc, n), generator=gen, device=dev) * math.sqrt(0.5)
        im = torch.randn((tc, n), generator=gen, device=dev) * math.sqrt(0.5)
        s = torch.randn((2, tc, 1), generator=gen, device=dev) * math.sqrt(0.05)
        re += s[0] * gr - s[1] * gi
        im += s[0] * gi + s[1] * gr
        time = torch.arange(t0, t0 + tc, device=dev, dtype=torch.float64)
        for k, f in enumerate((0.0625, 0.19, 0.3125)):
            turn = (2 * math.pi * ((f * time) % 1.0)).float()[:, None] + theta[k]
            re += 0.3 * torch.cos(turn)
            im += 0.3 * torch.sin(turn)
        re = torch.clamp(torch.round(3.0 * re), -7, 7)
        im = torch.clamp(torch.round(3.0 * im), -7, 7)
        out[t0:t0 + tc] = _pack(re, im, re_low)
    return out


def _interference(gen, x, block):
    """Carriers in 3 % of the (block, input) cells, impulsive bursts in 2 %."""
    t, n = x.shape
    dev = x.device
    nb = -(-t // block)
    kind = torch.rand((nb, n), generator=gen, device=dev).repeat_interleave(block, dim=0)[:t]
    turn = torch.arange(t, device=dev) % 4
    carrier = _pack(torch.tensor([6.0, 0.0, -6.0, 0.0], device=dev), torch.tensor([0.0, 6.0, 0.0, -6.0], device=dev),
                    False)[turn]
    spike = torch.rand((t, n), generator=gen, device=dev) < 4.0 / block
    burst = torch.where(spike, torch.full_like(x, 0x11), torch.full_like(x, 0x88))
    x = torch.where(kind < 0.03, carrier[:, None], x)
    return torch.where(kind > 0.98, burst, x)


def _weights(case, seed):
    """int8 [B][N][2]: a phase ramp per beam."""
    rng = random.Random(int(seed))
    n, beams = case["n"], case["beams"]
    i = torch.arange(n, dtype=torch.float64)
    w = torch.empty((beams, n, 2), dtype=torch.int8)
    for b in range(beams):
        ph = -2 * math.pi * (b + 1) * 0.37 * i / n + rng.uniform(0, 2 * math.pi)
        w[b, :, 0] = torch.round(127 * torch.cos(ph)).to(torch.int8)
        w[b, :, 1] = torch.round(127 * torch.sin(ph)).to(torch.int8)
    return w


def _inputs(case, seed):
    """The sample arrays of a case, one per job."""
    gen = _generator(seed)
    if case["kind"] == "prepared":
        # one array holds the channels side by side; each job takes its own
        n, t = case["n"], case["t"]
        x = _samples(gen, n, t * case["jobs"])
        return [x[k * t:(k + 1) * t] for k in range(case["jobs"])]
    if case["kind"] == "flagged":
        return [_interference(gen, _samples(gen, case["n"], case["t"]), case["block"])]
    return [_samples(gen, n, t, case.get("re_low", False)) for n, t in _jobs(case)]


# ---------------------------------------------------------------------------
# What a program has in hand, and one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    xs = _inputs(case, seed)
    st = {"case": case, "xs": xs}
    if kind == "beams":
        st["beams"] = xeng.Beams(_weights(case, seed).numpy(), device=torch.cuda.current_device())
        dtype = torch.int32 if case["shift"] < 0 else torch.int8
        st["out"] = torch.empty((case["t"], case["beams"], 2), dtype=dtype, device="cuda")
        return st
    if kind in ("channel", "presum", "flagged"):
        n = case["n"]
        st["corr"] = xeng.Correlator(n, 1, re_low=case.get("re_low", False), counts=kind == "flagged")
        st["out"] = torch.empty((xeng.tri(n), 2), dtype=torch.int32, device="cuda")
        if kind == "flagged":
            st["flags"] = torch.empty((-(-case["t"] // case["block"]), n), dtype=torch.uint8, device="cuda")
            st["counts"] = torch.empty(xeng.tri(n), dtype=torch.int32, device="cuda")
        return st
    if kind == "batch":
        corrs = [xeng.Correlator(n, 1) for n, _ in _jobs(case)]
        slots = [(c, 0) for c in corrs]
    else:
        c = xeng.Correlator(case["n"], case["jobs"])
        slots = [(c, k) for k in range(case["jobs"])]
    if kind == "prepared":
        # one export buffer for all channels
        st["out"] = torch.empty((case["jobs"], xeng.tri(case["n"]), 2), dtype=torch.int32, device="cuda")
        outs = list(st["out"])
    else:
        outs = [torch.empty((xeng.tri(c.n_inputs), 2), dtype=torch.int32, device="cuda") for c, _ in slots]
    st["dumps"] = [(c, s, o, True) for (c, s), o in zip(slots, outs)]
    if kind == "prepared":
        st["batch"] = xeng.Batch([(c, s, x) for (c, s), x in zip(slots, xs)])
    elif kind == "stream":
        rows = case["frames"] * FRAME
        st["calls"] = [[(c, s, x[k * rows:(k + 1) * rows]) for (c, s), x in zip(slots, xs)]
                       for k in range(case["launches"])]
    else:
        st["calls"] = [[(c, s, x) for (c, s), x in zip(slots, xs)]]
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "beams":
        return state["beams"].form(state["xs"][0], shift=case["shift"], out=state["out"])
    if kind == "channel":
        state["corr"].correlate(0, state["xs"][0])
        return state["corr"].dump(0, out=state["out"])
    if kind == "presum":
        state["corr"].correlate_presum(0, state["xs"][0])
        return state["corr"].dump(0, out=state["out"])
    if kind == "flagged":
        x, corr = state["xs"][0], state["corr"]
        flags = xeng.rfi_flags(x, block_len=case["block"], out=state["flags"])
        corr.correlate_flagged(0, x, flags, case["block"])
        counts = corr.dump_counts(0, out=state["counts"])
        return [flags, counts, corr.dump(0, out=state["out"])]
    if kind == "prepared":
        state["batch"].launch()
        xeng.dump_batch(state["dumps"])
        return state["out"]
    for jobs in state["calls"]:
        xeng.correlate_batch(jobs)
    return xeng.dump_batch(state["dumps"])


def work(case):
    if case["kind"] == "beams":
        n, t, b = case["n"], case["t"], case["beams"]
        return {"bytes": n * t + 2 * n * b + t * b * 2 * (4 if case["shift"] < 0 else 1), "flops": 8 * n * t * b}
    nbytes = flops = 0
    for n, t in _jobs(case):
        pairs = n * (n + 1) // 2
        nbytes += n * t + 8 * pairs
        flops += 8 * t * pairs
        if case["kind"] == "flagged":
            nbytes += 4 * pairs + n * -(-t // case["block"])
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------
def _parts(x, re_low):
    hi, lo = (x >> 4).double() - 8, (x & 15).double() - 8
    return (lo, hi) if re_low else (hi, lo)


def _visibilities(x, re_low=False, keep=None):
    """int64 [N(N+1)/2, 2]: sum over time of x_i conj(x_j), i <= j, row by row."""
    t, n = x.shape
    re = torch.zeros((n, n), dtype=torch.float64, device=x.device)
    im = torch.zeros_like(re)
    for t0 in range(0, t, CHUNK):
        a, b = _parts(x[t0:t0 + CHUNK], re_low)
        if keep is not None:
            a, b = a * keep[t0:t0 + CHUNK], b * keep[t0:t0 + CHUNK]
        at, bt = a.t().contiguous(), b.t().contiguous()
        re += at @ a + bt @ b
        im += bt @ a - at @ b
    i = torch.triu_indices(n, n, device=x.device)
    return torch.stack([re[i[0], i[1]], im[i[0], i[1]]], dim=1).round().to(torch.int64)


def _sk_flags(x, block):
    """Spectral kurtosis outside [0.625, 1.375], or no power, per (block, input)."""
    t, n = x.shape
    out = []
    for t0 in range(0, t, block):
        a, b = _parts(x[t0:t0 + block], False)
        p = (a * a + b * b).to(torch.int64)
        m, s1, s2 = p.shape[0], p.sum(0), (p * p).sum(0)
        num = 1000 * (m + 1) * (m * s2 - s1 * s1)
        den = (m - 1) * s1 * s1
        bad = (num < 625 * den) | (num > 1375 * den) | (s1 == 0)
        out.append(bad if m > 1 else torch.zeros_like(bad))
    return torch.stack(out).to(torch.uint8)


def exact(case, seed):
    xs = _inputs(case, seed)
    if case["kind"] == "beams":
        w = _weights(case, seed).double().to(xs[0].device)
        wr, wi = w[:, :, 0].t().contiguous(), w[:, :, 1].t().contiguous()
        a, b = _parts(xs[0], False)
        y = torch.stack([a @ wr - b @ wi, a @ wi + b @ wr], dim=2)
        if case["shift"] >= 0:
            y = torch.clamp(torch.round(y / 2.0 ** case["shift"]), -127, 127)
        return y.round().to(torch.int64)
    if case["kind"] == "flagged":
        x, block, n = xs[0], case["block"], case["n"]
        flags = _sk_flags(x, block)
        keep = (flags == 0).double().repeat_interleave(block, dim=0)[:case["t"]]
        i = torch.triu_indices(n, n, device=x.device)
        counts = (keep.t().contiguous() @ keep)[i[0], i[1]].round().to(torch.int64)
        return [flags.to(torch.int64), counts, _visibilities(x, keep=keep)]
    if case["kind"] in ("channel", "presum"):
        return _visibilities(xs[0], case.get("re_low", False))
    if case["kind"] == "prepared":
        return torch.stack([_visibilities(x) for x in xs])
    return [_visibilities(x) for x in xs]
