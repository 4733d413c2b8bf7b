"""The work that programs of this framework ask of it, through its public entry
points: rendering (a few sounds, one batch, the ragged corpus batch), the
render's adjoint, the spectral loss and features, the proposal network
(training step, inference on a few sounds), the distance between two sets of
sounds and a nebula-search trial, the resonant filter and the FM voice.

listed() names one case of each, at the sizes of the framework's own
workloads; draw() gives more of the same ranges.  prepare() makes the inputs on
the GPU from the seed alone, run() is one pass, work() the bytes and operations
that a pass cannot do without, and exact() the same outputs in float64 by plain
torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

F32, F64, I64 = torch.float32, torch.float64, torch.int64
SR, RC, Q = 44100.0, 441.0, 100
DEV = "cuda"
CYCLES = {"1-2-4": (1, 2, 4), "1-2-3-4": (1, 2, 3, 4)}
MR_SIZES = (512, 1024, 2048)


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a handful of 1 s sounds: what an interactive program renders, bound by launches
        {"name": "render_8x1s", "kind": "render", "voices": 8, "samples": 44100},
        # the plain batch of 128 sounds of 4 s
        {"name": "render_128x4s", "kind": "render", "voices": 128, "samples": 176400},
        # the ragged corpus batch: draw and render 16384 sounds of 1, 2 and 4 s
        {"name": "render_ragged_16384", "kind": "render_ragged", "voices": 16384, "unit": 44100,
         "cycle": "1-2-4"},
        # gradient sound matching, one step's parts: the render's adjoint ...
        {"name": "render_backward_256x4s", "kind": "adjoint", "voices": 256, "samples": 176400},
        # ... and the multi-resolution loss with its gradient against a fixed target
        {"name": "mrstft_grad_256x4s", "kind": "mrstft", "voices": 256, "samples": 176400,
         "cached": True, "grad": True},
        # features of one training batch of 1-4 s sounds
        {"name": "logmel_4096_1-4s", "kind": "logmel", "voices": 4096, "unit": 44100,
         "cycle": "1-2-3-4"},
        # one training step of the proposal network
        {"name": "mlp_train_4096", "kind": "mlp_train", "batch": 4096},
        # the proposal asked about a few sounds: forward of a small batch
        {"name": "mlp_forward_16", "kind": "mlp_forward", "batch": 16},
        # distance between two sets of 1000 sounds (8192 log-mel features each)
        {"name": "mmd_1000x1000", "kind": "mmd", "n": 1000, "m": 1000, "dim": 8192},
        # one nebula-search trial: draw, render, embed 256 sounds and score them
        {"name": "nebula_trial_256x4s", "kind": "nebula", "sounds": 256, "samples": 176400,
         "target": 256, "pool": 512},
        # the resonant filter on rendered sounds of mixed length, forward and backward
        {"name": "vcf_fwd_bwd_4096", "kind": "vcf", "voices": 4096, "unit": 44100,
         "cycle": "1-2-4"},
        # the FM voice on the ragged corpus batch
        {"name": "fm_ragged_16384", "kind": "fm", "voices": 16384, "unit": 44100,
         "cycle": "1-2-4"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("render", "render_ragged", "adjoint", "mrstft", "logmel", "mlp_train",
                       "mlp_forward", "mmd", "nebula", "vcf", "fm"))
    if kind == "render":
        return {"kind": kind, "voices": _log(rng, 2, 512), "samples": _log(rng, 4410, 176400)}
    if kind in ("render_ragged", "fm"):
        return {"kind": kind, "voices": _log(rng, 512, 16384), "unit": _log(rng, 8821, 44100),
                "cycle": "1-2-4"}
    if kind == "adjoint":
        return {"kind": kind, "voices": _log(rng, 8, 256), "samples": _log(rng, 22050, 176400)}
    if kind == "mrstft":
        return {"kind": kind, "voices": _log(rng, 8, 256), "samples": _log(rng, 11025, 176400),
                "cached": rng.random() < 0.6, "grad": rng.random() < 0.7}
    if kind == "logmel":
        return {"kind": kind, "voices": _log(rng, 16, 4096), "unit": _log(rng, 11025, 44100),
                "cycle": "1-2-3-4"}
    if kind == "mlp_train":
        return {"kind": kind, "batch": _log(rng, 256, 4096)}
    if kind == "mlp_forward":
        return {"kind": kind, "batch": _log(rng, 1, 1024)}
    if kind == "mmd":
        return {"kind": kind, "n": _log(rng, 128, 1000), "m": _log(rng, 128, 1000), "dim": 8192}
    if kind == "nebula":
        t = _log(rng, 64, 256)
        return {"kind": kind, "sounds": _log(rng, 64, 256), "samples": _log(rng, 44100, 176400),
                "target": t, "pool": t + rng.randrange(0, 257)}
    return {"kind": kind, "voices": _log(rng, 64, 4096), "unit": _log(rng, 8821, 44100),
            "cycle": "1-2-4"}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def voice_table():
    """The default Voice nebula: (min, max, curve, symmetric) of 78 parameters."""
    lo, hi, sym = [0.0] * 78, [1.0] * 78, [0.0] * 78
    lo[0], hi[0], hi[1] = 24.0, 84.0, 4.0
    for b in range(2, 32, 5):
        hi[b:b + 5] = (2.0, 2.0, 1.0, 2.0, 6.0)
        lo[b + 4] = 0.1
    for b in (32, 40):
        lo[b:b + 3], hi[b:b + 3] = (0.0, -10.0, -math.pi), (20.0, 20.0, math.pi)
    lo[68:71], hi[68:71] = (-24.0, -12.0, -math.pi), (24.0, 12.0, math.pi)
    lo[71:75], hi[71:75] = (-24.0, -12.0, -math.pi, 0.0), (24.0, 12.0, math.pi, 1.0)
    for p in (68, 69, 71, 72):
        sym[p] = 1.0
    return np.stack([lo, hi, [1.0] * 78, sym], axis=1)


def fm_table():
    """The default FM nebula (44 parameters)."""
    lo, hi, cv, sym = [0.0] * 44, [1.0] * 44, [1.0] * 44, [0.0] * 44
    lo[0], hi[0], lo[1], hi[1] = 24.0, 84.0, 0.1, 4.0
    for b in (2, 10, 18, 26):
        lo[b:b + 8] = (0.5, -50.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.1)
        hi[b:b + 8] = (8.0, 50.0, 1.0, 2.0, 2.0, 1.0, 2.0, 6.0)
        cv[b], sym[b + 1] = 2.0, 1.0
    hi[34:40], cv[34:40] = [2.0] * 6, [2.0] * 6
    return np.stack([lo, hi, cv, sym], axis=1)


def lengths(case):
    c = np.array(CYCLES[case["cycle"]], dtype=np.int64)
    return c[np.arange(case["voices"]) % len(c)] * case["unit"]


def ragged(case):
    """(lengths, offsets, longest-first order) of a ragged case's voices."""
    n = lengths(case)
    off = np.concatenate([[0], np.cumsum(n)])
    order = np.argsort(-n, kind="stable").astype(np.int32)
    return n, torch.from_numpy(off).to(DEV), torch.from_numpy(order).to(DEV)


def gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & (2**62 - 1))


def sounds(voices, samples, g, out=None):
    """[voices, samples] float32 sounds: decaying harmonics and noise that end
    in exact silence, as synthesised notes do."""
    out = torch.empty(voices, samples, dtype=F32, device=DEV) if out is None else out
    step = max(1, (1 << 25) // max(1, samples))
    t = torch.arange(samples, device=DEV, dtype=F32) / SR
    for a in range(0, voices, step):
        b = min(voices, a + step)
        r = torch.rand(b - a, 8, generator=g, device=DEV)
        f = 40.0 * 2.0 ** (5.0 * r[:, 0:1])
        ph = (f * t) % 1.0
        y = torch.zeros(b - a, samples, dtype=F32, device=DEV)
        for k in range(1, 6):
            y += torch.sin(2.0 * math.pi * ((k * ph) % 1.0)) * (0.5 ** (k * r[:, 1:2] * 2.0))
        y *= torch.exp(-t * (0.2 + 4.0 * r[:, 2:3]))
        y += (0.3 * r[:, 3:4] ** 2) * (torch.rand(b - a, samples, generator=g, device=DEV) * 2 - 1)
        end = (0.3 + 3.0 * r[:, 4:5]) * max(1.0, samples / SR) / 2.0
        y *= torch.clamp((end - t) * 20.0, 0.0, 1.0) * torch.clamp(t * 200.0, 0.0, 1.0)
        out[a:b] = y * (0.2 + 0.8 * r[:, 5:6])
    return out


def packed_sounds(n, g):
    """The packed buffer of ragged voices of lengths n."""
    total, top, off = int(n.sum()), int(n.max()), 0
    out = torch.empty(total, dtype=F32, device=DEV)
    step = max(1, (1 << 25) // top)
    for a in range(0, len(n), step):
        part = sounds(len(n[a:a + step]), top, g)
        for i, k in enumerate(n[a:a + step]):
            out[off:off + k] = part[i, :k]
            off += int(k)
    return out


def features(rows, dim, g):
    """[rows, dim] log-mel-like features: a spectral slope, smooth differences
    between sounds, noise, and the floor log(1e-6) where a sound is silent."""
    k = torch.arange(dim, device=DEV, dtype=F32) / dim
    r = torch.rand(rows, 4, generator=g, device=DEV)
    y = 4.0 - 10.0 * r[:, 0:1] * k + 3.0 * torch.sin(6.0 * (k + r[:, 1:2]) * (1.0 + r[:, 2:3]))
    y = y + 2.0 * torch.randn(rows, dim, generator=g, device=DEV)
    silent = (torch.arange(dim, device=DEV) % 64).float() / 64.0 > 0.3 + r[:, 3:4]
    floor = torch.full((), math.log(1e-6), dtype=F32, device=DEV)
    return torch.where(silent, floor, torch.clamp(y, min=float(floor)))


def mlp_weights(g):
    def w(o, i, s):
        return (torch.randn(o, i, generator=g, device=DEV) * math.sqrt(s / i)).cpu().numpy()
    return {"w1t": w(1024, 8192, 2.0), "b1": np.zeros(1024, np.float32),
            "w2t": w(1024, 1024, 2.0), "b2": np.zeros(1024, np.float32),
            "w3t": w(78, 1024, 1.0), "b3": np.zeros(78, np.float32)}


def mlp_batch(batch, g):
    x = torch.randn(batch, 8192, generator=g, device=DEV).to(torch.bfloat16)
    return x, torch.rand(batch, 78, generator=g, device=DEV)


def vcf_controls(voices, periods, g):
    walk = torch.cumsum(torch.randn(voices, periods, generator=g, device=DEV) * 0.03, 1)
    env = (0.5 + 0.5 * torch.sin(walk + 3.0 * torch.rand(voices, 1, generator=g, device=DEV)))
    r = torch.rand(voices, 3, generator=g, device=DEV)
    p = torch.stack([30.0 + 70.0 * r[:, 0], -24.0 + 72.0 * r[:, 1], 0.5 + 14.5 * r[:, 2] ** 2], 1)
    return env.contiguous(), p.contiguous()


def corpus_first(seed):
    """First voice index of a seed's batch."""
    return (int(seed) % 1000003) * 16384


def nebula_curves(seed):
    return np.random.default_rng(int(seed)).uniform(-1.0, 1.0, 4)


NEBULA_PARAMS = (0, 2, 3, 77)          # pitch, attack, decay, noise level


def prepare(case, seed):
    import paper_2104_12922_amd as S
    from paper_2104_12922_amd import fm, learned, nebula, vcf
    g, kind, s = gen(seed), case["kind"], dict(case)
    s["seed"] = int(seed)
    if kind == "render":
        s.update(S=S, table=voice_table(), first=corpus_first(seed))
    elif kind == "render_ragged":
        n, off, order = ragged(case)
        table = voice_table()
        table[1, 0] = 0.1
        s.update(S=S, table=table, first=corpus_first(seed), off=off, order=order,
                 longest=int(n.max()),
                 u=torch.empty(case["voices"], 78, dtype=F32, device=DEV),
                 audio=torch.empty(int(n.sum()), dtype=F32, device=DEV))
    elif kind == "adjoint":
        u = torch.rand(case["voices"], 78, generator=g, device=DEV)
        gy = torch.randn(case["voices"], case["samples"], generator=g, device=DEV) * 1e-4
        s.update(S=S, table=voice_table(), u=u, gy=gy,
                 ws=S.synth_render_backward_workspace(voice_table(), *gy.shape))
    elif kind == "mrstft":
        x = sounds(case["voices"], case["samples"], g)
        y = sounds(case["voices"], case["samples"], g)
        ws = S.synth_mrstft_workspace(*x.shape, grad=case["grad"])
        s.update(S=S, x=x, ws=ws, y=S.synth_mrstft_target(y) if case["cached"] else y)
    elif kind == "logmel":
        n, off, _ = ragged(case)
        s.update(lm=learned.LogMel(), audio=packed_sounds(n, g), off=off)
    elif kind in ("mlp_train", "mlp_forward"):
        net = learned.MLP(mlp_weights(g))
        x, t = mlp_batch(case["batch"], g)
        s.update(net=net, x=x, t=t)
    elif kind == "mmd":
        s.update(N=nebula, X=features(case["n"], case["dim"], g),
                 Y=features(case["m"], case["dim"], g) * 0.9)
    elif kind == "nebula":
        sets = nebula.SoundSets(case["sounds"], case["samples"], seed=30)
        s.update(z=nebula_curves(seed), k=int(seed) % 4096,
                 search=nebula.NebulaSearch(voice_table(), features(case["pool"], 8192, g),
                                            NEBULA_PARAMS, sets, target_per_trial=case["target"],
                                            seed=1))
    elif kind == "vcf":
        n, off, order = ragged(case)
        env, p = vcf_controls(case["voices"], -(-int(n.max()) // Q), g)
        s.update(V=vcf, x=packed_sounds(n, g), env=env, p=p, off=off, order=order,
                 longest=int(n.max()),
                 gy=torch.randn(int(n.sum()), generator=g, device=DEV) * 1e-3)
    elif kind == "fm":
        n, off, order = ragged(case)
        s.update(FM=fm, table=fm_table(), first=corpus_first(seed), off=off, order=order,
                 audio=torch.empty(int(n.sum()), dtype=F32, device=DEV))
    else:
        raise ValueError(kind)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "render":
        u = s["S"].synth_sample_params(0, s["first"], s["voices"])
        y = s["S"].synth_render(u, s["table"], n_samples=s["samples"], first_g=s["first"])
        return {"u": u, "audio": y}
    if kind == "render_ragged":
        s["S"].synth_sample_params(0, s["first"], s["voices"], out=s["u"])
        y = s["S"].synth_render_plan(s["u"], s["table"], 4, 1, offsets=s["off"],
                                     first_g=s["first"], order=s["order"],
                                     max_samples=s["longest"], out=s["audio"])
        return {"u": s["u"], "audio": y}
    if kind == "adjoint":
        return s["S"].synth_render_backward(s["u"], s["gy"], s["table"], workspace=s["ws"])
    if kind == "mrstft":
        return s["S"].synth_mrstft_loss(s["x"], s["y"], grad=s["grad"], workspace=s["ws"])
    if kind == "logmel":
        return s["lm"](s["audio"], offsets=s["off"])
    if kind == "mlp_train":
        loss = s["net"].train_step(s["x"], s["t"])
        return {"loss": loss, "g": s["net"].g, "w": s["net"].w}
    if kind == "mlp_forward":
        return s["net"].forward(s["x"])
    if kind == "mmd":
        return s["N"].mmd_l1(s["X"], s["Y"]).tolist()      # numbers, as a search reads them
    if kind == "nebula":
        return s["search"].score(s["z"], s["k"])
    if kind == "vcf":
        kw = dict(offsets=s["off"], max_samples=s["longest"], order=s["order"])
        y, st = s["V"].lowpass(s["x"], s["env"], s["p"], keep_states=True, **kw)
        gx, gp, ge = s["V"].lowpass_backward(s["x"], s["gy"], s["env"], s["p"], st, **kw)
        return {"y": y, "gx": gx, "gp": gp, "ge": ge}
    u = s["FM"].fm_sample_params(0, s["first"], s["voices"])
    y = s["FM"].fm_render(u, s["table"], offsets=s["off"], order=s["order"], out=s["audio"])
    return {"u": u, "audio": y}


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: of the
    definitions, a transcendental counted as one."""
    kind = case["kind"]
    B = case.get("voices", 0)
    if kind == "render":
        N = B * case["samples"]
        return {"bytes": 4 * N + 4 * 78 * B, "flops": 45 * N}
    if kind in ("render_ragged", "fm"):
        N = int(lengths(case).sum())
        return {"bytes": 4 * N + 4 * 78 * B, "flops": (45 if kind != "fm" else 32) * N}
    if kind == "adjoint":
        N = B * case["samples"]
        return {"bytes": 4 * N + 8 * 78 * B, "flops": 150 * N}
    if kind == "mrstft":
        N = B * case["samples"]
        fft = sum(4.0 * 2.5 * math.log2(n) for n in MR_SIZES)   # one real transform, hop n/4
        passes = 1 + (0 if case["cached"] else 1) + (1 if case["grad"] else 0)
        read = 4 + (24 if case["cached"] else 4)
        return {"bytes": (read + (4 if case["grad"] else 0)) * N + 8 * B, "flops": passes * fft * N}
    if kind == "logmel":
        n = lengths(case)
        used = np.minimum(n, 63 * 2756 + 2048)
        frames = np.minimum(64, -(-n // 2756)).sum()
        read = float(np.minimum(used, frames / B * 2048).sum())
        return {"bytes": 4 * read + 4 * 8192 * B, "flops": float(frames) * (2.5 * 2048 * 11 + 8000)}
    if kind in ("mlp_train", "mlp_forward"):
        b, w = case["batch"], 8192 * 1024 + 1024 * 1024 + 1024 * 78
        if kind == "mlp_forward":
            return {"bytes": 2 * w + 2 * 8192 * b + 4 * 78 * b, "flops": 2.0 * w * b}
        # weights and moments read and written, bf16 copies read and written, gradients written
        return {"bytes": (6 * 4 + 4 + 2 * 2) * w + 2 * 8192 * b + 2 * 4 * 78 * b,
                "flops": (4.0 * w + 2.0 * (w - 8192 * 1024)) * b}
    if kind == "mmd":
        rows = case["n"] + case["m"]
        return {"bytes": 4 * case["dim"] * rows + 32,
                "flops": 3.0 * case["dim"] * rows * math.log2(rows)}
    if kind == "nebula":
        n, rows = case["sounds"], case["sounds"] + case["target"]
        return {"bytes": 2 * 4 * n * case["samples"] + 2 * 4 * 8192 * rows,
                "flops": 45.0 * n * case["samples"] + n * 64 * (2.5 * 2048 * 11 + 8000)
                + 3.0 * 8192 * rows * math.log2(rows)}
    n = lengths(case)
    env = 4 * B * -(-int(n.max()) // Q)
    return {"bytes": (8 + 12) * int(n.sum()) + 3 * env, "flops": 40 * int(n.sum())}


# ---------------------------------------------------------------------------
# The same in float64
# ---------------------------------------------------------------------------
def philox(c0, c1, c2, c3, key):
    """Philox4x32-10 on int64 tensors of 32-bit words; key: a 64-bit number."""
    m = 0xFFFFFFFF
    k0, k1 = key & m, (key >> 32) & m
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & m) ^ c1 ^ k0, p1 & m, ((p0 >> 32) & m) ^ c3 ^ k1, p0 & m)
    return c0, c1, c2, c3


def exact_draw(first, count, params, tag, key=0):
    g = first + torch.arange(count, dtype=I64, device=DEV)[:, None]
    blk = torch.arange(-(-params // 4), dtype=I64, device=DEV)[None, :]
    z = torch.zeros_like(g + blk)
    w = torch.stack(philox((g & 0xFFFFFFFF) + z, (g >> 32) + z, blk + z, z + tag, key), -1)
    return (w.reshape(count, -1)[:, :params] >> 8).to(F64) * 2.0 ** -24


def exact_noise(g, N, key):
    n = torch.arange(N, dtype=I64, device=DEV)
    blk = torch.arange(-(-N // 8), dtype=I64, device=DEV)[None, :]
    g = g[:, None]
    z = torch.zeros_like(g + blk)
    w = torch.stack(philox((g & 0xFFFFFFFF) + z, (g >> 32) + z, blk + z, z + 1, key), -1)
    w = w.reshape(g.shape[0], -1)[:, n >> 1]
    h = (w >> ((n & 1) * 16)) & 0xFFFF
    return (h.to(F64) + 0.5) / 32768.0 - 1.0


def pow01(x, e):
    pos = x > 0
    return torch.where(pos, torch.where(pos, x, torch.ones_like(x)) ** e, torch.zeros_like(x))


def exact_map(u, table):
    lo, hi, c, sym = (torch.from_numpy(np.ascontiguousarray(table[:, k])).to(DEV) for k in range(4))
    d = 2.0 * u - 1.0
    plain = torch.where(c == 1.0, u, pow01(u, 1.0 / c))
    about = torch.where(c == 1.0, d.abs(), pow01(d.abs(), 1.0 / c))
    return torch.where(sym > 0.5, lo + (hi - lo) * (1.0 + torch.sign(d) * about) / 2.0,
                       lo + (hi - lo) * plain)


def exact_adsr(j, v, b, off):
    """Envelope of the five parameters from column b, at control samples j."""
    def ramp(start, length):
        pos = length > 0
        x = torch.clamp((j - start) / torch.where(pos, length, torch.ones_like(length)), 0.0, 1.0)
        return torch.where(pos, x, (j >= start).to(F64))
    A, D, S, R, e = (v[:, b + k:b + k + 1] for k in range(5))
    A, D, R = A * RC, D * RC, R * RC
    return pow01(ramp(0.0 * A, A), e) * (S + (1.0 - S) * pow01(1.0 - ramp(A, D), e)) \
        * pow01(1.0 - ramp(off * RC, R), e)


def before(x):
    """Exclusive cumulative sum along the last axis."""
    return torch.cumsum(x, -1) - x if not x.requires_grad else torch.cat(
        [torch.zeros_like(x[..., :1]), torch.cumsum(x, -1)[..., :-1]], -1)


def up(y, N):
    """Control to audio rate: linear, the last value held."""
    n = torch.arange(N, device=DEV)
    j, t = n // Q, (n % Q).to(F64) / Q
    return (1.0 - t) * y[..., j] + t * y[..., torch.clamp(j + 1, max=y.shape[-1] - 1)]


def exact_voice(u, g, N, table, key=0):
    """The Voice's audio [B, N] in float64 (u float64, voice indices g)."""
    v = exact_map(u, table)
    c = [v[:, k:k + 1] for k in range(78)]
    J = -(-N // Q)
    j = torch.arange(J, dtype=F64, device=DEV)[None, :]
    env = [exact_adsr(j, v, 2 + 5 * k, c[1]) for k in range(6)]
    x = [env[0], env[1]]
    for i, b in enumerate((32, 40)):
        f = torch.clamp(c[b] + c[b + 1] * env[2 + 2 * i], min=0.0)
        th = c[b + 2] / (2 * math.pi) + before(f / RC)
        ph = th - torch.floor(th)
        shapes = ((1.0 + torch.sin(2 * math.pi * ph)) / 2.0, 1.0 - (2.0 * ph - 1.0).abs(), ph,
                  1.0 - ph, (ph < 0.5).to(F64))
        w = v[:, b + 3:b + 8].sum(-1, keepdim=True)
        num = sum(shapes[k] * c[b + 3 + k] for k in range(5))
        raw = torch.where(w > 0, num / torch.where(w > 0, w, torch.ones_like(w)), 0.0 * num)
        x.append(raw * env[3 + 2 * i])
    y = []
    for o in range(5):
        G = [c[48 + 4 * o + i] for i in range(4)]
        y.append(sum(G[i] * x[i] for i in range(4)) / torch.clamp(sum(G), min=1.0))

    def phase(b, a):
        m = c[0] + c[b] + c[b + 1] * a
        f = torch.clamp(440.0 * torch.pow(2.0, (m - 69.0) / 12.0), max=SR / 2.0)
        th = c[b + 2] / (2 * math.pi) + before(f / SR)
        return 2 * math.pi * (th - torch.floor(th))
    p1, p2 = phase(68, up(y[0], N)), phase(71, up(y[2], N))
    m = torch.clamp(c[0] + c[71] + torch.clamp(c[72], min=0.0), min=0.0)
    top = torch.clamp(440.0 * torch.pow(2.0, (m - 69.0) / 12.0), max=SR / 2.0)
    K = 12000.0 / (top * torch.log10(top))
    square = (1.0 - c[74] / 2.0) * torch.tanh(K * torch.sin(p2)) * (1.0 + c[74] * torch.cos(p2))
    return c[75] * torch.sin(p1) * up(y[1], N) + c[76] * square * up(y[3], N) \
        + c[77] * exact_noise(g, N, key) * up(y[4], N)


def exact_fm(u, N, table):
    v = exact_map(u, table)
    J = -(-N // Q)
    j = torch.arange(J, dtype=F64, device=DEV)[None, :]
    n = torch.arange(N, dtype=F64, device=DEV)[None, :]
    pairs = ((0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3))
    o = [None] * 4
    for i in (3, 2, 1, 0):
        b = 2 + 8 * i
        f = 440.0 * torch.pow(2.0, (v[:, 0:1] - 69.0) / 12.0) * v[:, b:b + 1] \
            * torch.pow(2.0, v[:, b + 1:b + 2] / 1200.0)
        th = n * torch.clamp(f, max=SR / 2.0) / SR
        for k, (a, d) in enumerate(pairs):
            if a == i:
                th = th + v[:, 34 + k:35 + k] * o[d]
        th = th - torch.floor(th)
        a = up(exact_adsr(j, v, b + 3, v[:, 1:2]), N)
        o[i] = v[:, b + 2:b + 3] * a * torch.sin(2 * math.pi * th)
    w = v[:, 40:44]
    return sum(w[:, i:i + 1] * o[i] for i in range(4)) / torch.clamp(w.sum(-1, keepdim=True), min=1.0)


def by_length(case, render, most=1 << 23):
    """The packed float64 buffer of a ragged case, voices of one length at a
    time: render(indices, length) gives [len(indices), length]."""
    n = lengths(case)
    off = np.concatenate([[0], np.cumsum(n)])
    out = torch.empty(int(n.sum()), dtype=F64, device=DEV)
    for N in np.unique(n):
        idx = np.nonzero(n == N)[0]
        step = max(1, most // int(N))
        for a in range(0, len(idx), step):
            part = idx[a:a + step]
            y = render(torch.from_numpy(part).to(DEV), int(N))
            for r, i in enumerate(part):
                out[off[i]:off[i + 1]] = y[r]
    return out


def hann(n):
    return 0.5 - 0.5 * torch.cos(2.0 * math.pi * torch.arange(n, dtype=F64, device=DEV) / n)


def exact_mrstft(x, y):
    """Per-voice loss of float64 [B, N] sounds."""
    total = torch.zeros(x.shape[0], dtype=F64, device=DEV)
    for n in MR_SIZES:
        if x.shape[1] >= n:
            X, Y = (torch.fft.rfft(v.unfold(1, n, n // 4) * hann(n)).abs() for v in (x, y))
            total = total + (torch.log(X + 1e-5) - torch.log(Y + 1e-5)).abs().mean((-2, -1))
    return total


def exact_logmel(x):
    """[B, 8192] features of float64 [B, N] sounds, samples past the end 0."""
    need = 63 * 2756 + 2048
    x = torch.nn.functional.pad(x, (0, max(0, need - x.shape[1])))[:, :need]
    P = torch.fft.rfft(x.unfold(1, 2048, 2756) * hann(2048)).abs() ** 2
    top = 2595.0 * math.log10(1.0 + SR / 2.0 / 700.0)
    e = 700.0 * (10.0 ** (np.linspace(0.0, top, 130) / 2595.0) - 1.0)
    f = np.arange(1025) * SR / 2048
    M = np.stack([np.maximum(0.0, np.minimum((f - e[b]) / (e[b + 1] - e[b]),
                                             (e[b + 2] - f) / (e[b + 2] - e[b + 1])))
                  for b in range(128)])
    mel = P.reshape(-1, 1025) @ torch.from_numpy(M).to(DEV).T.contiguous()
    return torch.log(mel.reshape(x.shape[0], 64, 128).transpose(1, 2) + 1e-6).reshape(x.shape[0], -1)


def exact_mmd(X, Y):
    X, Y = X.to(F64), Y.to(F64)

    def pairs(A, B):
        return sum(float((B - a).abs().sum()) for a in A)
    n, m = len(X), len(Y)
    xy, xx, yy = pairs(X, Y), pairs(X, X), pairs(Y, Y)
    return torch.tensor([2 * xy / (n * m) - xx / (n * n) - yy / (m * m), xy, xx, yy], dtype=F64)


def gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def exact_mlp(init, x):
    w = {k: torch.from_numpy(a).to(DEV) for k, a in init.items()}
    w = {k: (a.to(torch.bfloat16) if k.startswith("w") else a).to(F64) for k, a in w.items()}
    for a in w.values():
        a.requires_grad_(True)
    h = gelu(x.to(F64) @ w["w1t"].T + w["b1"])
    h = gelu(h @ w["w2t"].T + w["b2"])
    return w, torch.sigmoid(h @ w["w3t"].T + w["b3"])


def exact_vcf(x, env, p, gy):
    """(y, dL/dx, dL/dp, dL/denv) of float64 [B, N] sounds: every control
    period is run from a zero state and from the two unit states, all periods
    at once, then the periods' true entry states follow one after another."""
    B, N = x.shape
    J = -(-N // Q)
    x, env, p = (t.detach().clone().requires_grad_(True) for t in (x, env[:, :J], p))
    m = p[:, 0:1] + p[:, 1:2] * env
    f = torch.clamp(440.0 * torch.pow(2.0, (m - 69.0) / 12.0), 10.0, 0.45 * SR)
    w = 2.0 * math.pi * f / SR
    c, al = torch.cos(w), torch.sin(w) / (2.0 * p[:, 2:3])
    b0, b1 = (1.0 - c) / 2.0 / (1.0 + al), (1.0 - c) / (1.0 + al)
    a1, a2 = -2.0 * c / (1.0 + al), (1.0 - al) / (1.0 + al)
    xp = torch.nn.functional.pad(x, (2, J * Q - N))
    drive = [b0 * xp[:, k + 2:k + 2 + J * Q:Q] + b1 * xp[:, k + 1:k + 1 + J * Q:Q]
             + b0 * xp[:, k:k + J * Q:Q] for k in range(Q)]
    zero, one = torch.zeros_like(f), torch.ones_like(f)

    def sweep(y1, y2, u):
        out = []
        for k in range(Q):
            y = (u[k] if u is not None else 0.0) - a1 * y1 - a2 * y2
            y1, y2 = y, y1
            out.append(y)
        return out
    z, e1, e2 = sweep(zero, zero, drive), sweep(one, zero, None), sweep(zero, one, None)
    s1, s2 = torch.zeros_like(f[:, 0]), torch.zeros_like(f[:, 0])
    S1, S2 = [], []
    last = [[t.unbind(1) for t in (v[-1], v[-2])] for v in (z, e1, e2)]
    for j in range(J):
        S1.append(s1)
        S2.append(s2)
        s1, s2 = (last[0][0][j] + last[1][0][j] * s1 + last[2][0][j] * s2,
                  last[0][1][j] + last[1][1][j] * s1 + last[2][1][j] * s2)
    S1, S2 = torch.stack(S1, 1), torch.stack(S2, 1)
    y = torch.stack([z[k] + e1[k] * S1 + e2[k] * S2 for k in range(Q)], -1).reshape(B, -1)[:, :N]
    gx, ge, gp = torch.autograd.grad(y, (x, env, p), gy)
    return y.detach(), gx, gp, ge


def exact(case, seed):
    g, kind = gen(seed), case["kind"]
    B = case.get("voices", 0)
    if kind in ("render", "render_ragged", "fm"):
        first, fm = corpus_first(seed), kind == "fm"
        u = exact_draw(first, B, 44 if fm else 78, 1 if fm else 0)
        ids = first + torch.arange(B, dtype=I64, device=DEV)
        if kind == "render":
            step = max(1, (1 << 22) // case["samples"])
            y = torch.cat([exact_voice(u[a:a + step], ids[a:a + step], case["samples"], voice_table())
                           for a in range(0, B, step)])
        elif fm:
            y = by_length(case, lambda i, N: exact_fm(u[i], N, fm_table()))
        else:
            table = voice_table()
            table[1, 0] = 0.1
            y = by_length(case, lambda i, N: exact_voice(u[i], ids[i], N, table))
        return {"u": u, "audio": y}
    if kind == "adjoint":
        u = torch.rand(B, 78, generator=g, device=DEV)
        gy = torch.randn(B, case["samples"], generator=g, device=DEV) * 1e-4
        ids, step, out = torch.arange(B, dtype=I64, device=DEV), max(1, (1 << 22) // case["samples"]), []
        for a in range(0, B, step):
            v = u[a:a + step].to(F64).requires_grad_(True)
            y = exact_voice(v, ids[a:a + step], case["samples"], voice_table())
            out.append(torch.autograd.grad(y, v, gy[a:a + step].to(F64))[0])
        return torch.cat(out)
    if kind == "mrstft":
        x = sounds(B, case["samples"], g)
        y = sounds(B, case["samples"], g)
        step, loss, grad = max(1, (1 << 22) // case["samples"]), [], []
        for a in range(0, B, step):
            v = x[a:a + step].to(F64).requires_grad_(case["grad"])
            r = exact_mrstft(v, y[a:a + step].to(F64))
            loss.append(r.detach())
            if case["grad"]:
                grad.append(torch.autograd.grad(r.sum(), v)[0])
        return (torch.cat(loss), torch.cat(grad)) if case["grad"] else torch.cat(loss)
    if kind == "logmel":
        n = lengths(case)
        audio, off = packed_sounds(n, g), np.concatenate([[0], np.cumsum(n)])
        out = torch.empty(B, 8192, dtype=F64, device=DEV)
        for a in range(0, B, 32):
            x = torch.zeros(min(32, B - a), 4 * case["unit"], dtype=F64, device=DEV)
            for i in range(x.shape[0]):
                x[i, :n[a + i]] = audio[off[a + i]:off[a + i + 1]]
            out[a:a + 32] = exact_logmel(x)
        return out
    if kind == "mlp_forward":
        init = mlp_weights(g)
        return exact_mlp(init, mlp_batch(case["batch"], g)[0])[1].detach()
    if kind == "mlp_train":
        init = mlp_weights(g)
        x, t = mlp_batch(case["batch"], g)
        w, out = exact_mlp(init, x)
        loss = ((out - t.to(F64)) ** 2).mean()
        loss.backward()
        # Adam's first step: m / (1 - b1) = g, sqrt(v / (1 - b2)) = |g|
        new = {k: torch.from_numpy(init[k]).to(DEV).to(F64)
               - 3e-4 * w[k].grad / (w[k].grad.abs() + 1e-8) for k in w}
        return {"loss": loss.detach(), "g": {k: w[k].grad for k in w}, "w": new}
    if kind == "mmd":
        return exact_mmd(features(case["n"], case["dim"], g),
                         features(case["m"], case["dim"], g) * 0.9).tolist()
    if kind == "nebula":
        k = int(seed) % 4096
        table = voice_table()
        table[list(NEBULA_PARAMS), 2] = 10.0 ** nebula_curves(seed)
        first, n = k << 20, case["sounds"]
        u = exact_draw(first, n, 78, 0, key=30)
        ids = first + torch.arange(n, dtype=I64, device=DEV)
        step = max(1, (1 << 22) // case["samples"])
        X = torch.cat([exact_logmel(exact_voice(u[a:a + step], ids[a:a + step], case["samples"],
                                                table, key=30)) for a in range(0, n, step)])
        Y = features(case["pool"], 8192, g)
        if case["target"] < case["pool"]:
            r = torch.Generator().manual_seed(1000003 + k)
            Y = Y[torch.randperm(case["pool"], generator=r)[:case["target"]].to(DEV)]
        return float(exact_mmd(X, Y)[0])
    n = lengths(case)
    off = np.concatenate([[0], np.cumsum(n)])
    J = -(-int(n.max()) // Q)
    env, p = vcf_controls(B, J, g)
    x, gy = packed_sounds(n, g), torch.randn(int(n.sum()), generator=g, device=DEV) * 1e-3
    out = {"y": torch.empty(int(n.sum()), dtype=F64, device=DEV), "gp": torch.empty(B, 3, dtype=F64, device=DEV),
           "gx": torch.empty(int(n.sum()), dtype=F64, device=DEV), "ge": torch.zeros(B, J, dtype=F64, device=DEV)}
    for N in np.unique(n):
        idx = np.nonzero(n == N)[0]
        step = max(1, (1 << 26) // int(N))
        for a in range(0, len(idx), step):
            part = idx[a:a + step]
            i = torch.from_numpy(part).to(DEV)
            xs, gs = (torch.stack([t[off[k]:off[k + 1]] for k in part]).to(F64) for t in (x, gy))
            y, gx, gp, ge = exact_vcf(xs, env[i].to(F64), p[i].to(F64), gs)
            out["gp"][i] = gp
            out["ge"][i, :ge.shape[1]] = ge
            for r, k in enumerate(part):
                out["y"][off[k]:off[k + 1]] = y[r]
                out["gx"][off[k]:off[k + 1]] = gx[r]
    return out
