"""Timed cases of the one-spike convolutional SNN path, on the GPU.

Each case is one pass through the public entry points as a program calls them:
whole steps of a :class:`Chain` (batch training, single-image inference, the
natural-image layer), online plasticity (:class:`OnlineTrainer`), and single
layers and operators (encoder, conv + fire, kWTA + STDP, pointwise inhibition
and pooling of potentials).

Kinds and the ranges they are drawn from:

* ``chain``: the 3-layer network (conv 6->30 k5, pool 2, conv 30->250 k3, pool 3,
  conv 250->200 k5 with the infinite threshold) on H x W images, a batch of B,
  learning (``learn``) or forward only, in the full form (every call writes all
  its outputs), the compact form (first-spike maps between layers) or the fused
  form (conv and pool in one launch), with or without local normalisation.
* ``online``: N images one at a time, each learnt from before the next, in HIP
  graphs of ``group`` steps.
* ``natural``: 4 Gabor orientations, pool 7/6, conv 4->20 k17, kWTA and STDP on
  photograph-sized images.
* ``encode``: the rank-order encoder alone, all its outputs, on larger images.
* ``conv``: one conv + fire call from a wave or from a first-spike map, finite
  threshold or Eq.5, stride 1 or 2, with or without spike pooling behind it.
* ``learn``: kWTA and STDP of one layer from its first-spike map and potentials.
* ``inhibit``: pointwise inhibition (with its wave and masked potentials), then
  pooling of the potentials.

Chains, online runs and ``learn`` use weights on a binary grid on which every
partial sum is exact in float32, so that winners (a discontinuous function of
the potentials) are the same for every correct implementation; the ``conv``
cases take plain float weights, where rounding shows in the potentials.
"""
import math
from types import SimpleNamespace

import torch

import paper_1903_02440_amd as spk
from paper_1903_02440_amd.pipeline import Chain, OnlineTrainer

DEV = "cuda"
U8, F32, F64, I32 = torch.uint8, torch.float32, torch.float64, torch.int32


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a serving program classifies one 28x28 image: every launch is latency
        {"name": "infer_b1", "kind": "chain", "B": 1, "H": 28, "W": 28, "T": 15, "form": "compact", "learn": False,
         "norm": 0},
        # the tutorial's training loop: one image per step, 32 images
        {"name": "online_32", "kind": "online", "N": 32, "H": 28, "W": 28, "T": 15, "group": 16},
        # an ordinary training batch in the form that moves least, an odd size
        {"name": "train_fused_b97", "kind": "chain", "B": 97, "H": 28, "W": 28, "T": 15, "form": "fused", "learn": True,
         "norm": 0},
        # the benchmark's training step: 1000 images, every call writes its full outputs
        {"name": "train_full_b1000", "kind": "chain", "B": 1000, "H": 28, "W": 28, "T": 15, "form": "full",
         "learn": True, "norm": 0},
        # one training step of the natural-image layer
        {"name": "natural_b64", "kind": "natural", "B": 64, "H": 160, "W": 250, "T": 30},
        # encoding photographs: DoG bank, odd sides
        {"name": "encode_b7_241x321", "kind": "encode", "B": 7, "H": 241, "W": 321, "T": 20, "bank": "dog"},
        # a layer given its input's spike wave (the forward stress layer), pooled on spikes
        {"name": "conv_wave_b256", "kind": "conv", "B": 256, "Cin": 30, "H": 14, "W": 14, "Cout": 250, "K": 3, "pad": 1,
         "stride": 1, "T": 15, "wave": True, "inf": False, "pool": 3, "geometric": False},
        # the largest layer: 64 maps of 256x256, 64 steps
        {"name": "conv_large", "kind": "conv", "B": 1, "Cin": 64, "H": 256, "W": 256, "Cout": 256, "K": 5, "pad": 2,
         "stride": 1, "T": 64, "wave": False, "inf": False, "pool": 0, "geometric": True},
        # the classifying layer with the infinite threshold, an odd batch
        {"name": "conv_eq5_b301", "kind": "conv", "B": 301, "Cin": 250, "H": 4, "W": 4, "Cout": 200, "K": 5, "pad": 2,
         "stride": 1, "T": 15, "wave": False, "inf": True, "pool": 0, "geometric": False},
        # a strided layer with ragged sizes
        {"name": "conv_stride2_ragged", "kind": "conv", "B": 31, "Cin": 13, "H": 65, "W": 43, "Cout": 70, "K": 7,
         "pad": 3, "stride": 2, "T": 21, "wave": False, "inf": False, "pool": 0, "geometric": False},
        # winners and plasticity of the largest layer, 4 images
        {"name": "learn_large_b4", "kind": "learn", "B": 4, "Cin": 64, "Cout": 256, "H": 256, "W": 256, "K": 5,
         "pad": 2, "T": 64, "k": 32, "r": 4},
        # the inhibition and potential pooling between two layers, 200 images
        {"name": "inhibit_b200", "kind": "inhibit", "B": 200, "C": 250, "H": 14, "W": 14, "T": 15, "pool": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _images(C, KF, H, W):
    """The fewest images drawn of this size.  The filter works on bands of as many
    rows as fit 64 KiB; where a batch has fewer than 128 such bands, the code that
    these cases were first measured on cuts them thinner and, at some heights, then
    runs past its buffers, so drawn batches (and drawn chains with local
    normalisation, which filter separately) have at least 128."""
    rows = (65536 - 16 * C - 8 * C * KF * KF) // (8 * (W + KF + 2)) - KF + 1
    return -(-128 // -(-H // rows))


def draw(rng):
    kind = rng.choice(["chain", "chain", "online", "natural", "encode", "conv", "conv", "conv", "learn", "inhibit"])
    if kind == "chain":
        H, W = rng.randint(24, 36), rng.randint(24, 36)
        T = rng.randint(10, 20)
        B = min(_log(rng, 1, 1000), 784000 * 15 // (H * W * T))
        return {"kind": kind, "B": B, "H": H, "W": W, "T": T,
                "form": rng.choice(["full", "compact", "fused"]), "learn": rng.random() < 0.6,
                "norm": rng.choice([0, 0, 3, 8]) if B >= 128 else 0}
    if kind == "online":
        return {"kind": kind, "N": rng.randint(16, 48), "H": rng.randint(24, 32), "W": rng.randint(24, 32),
                "T": rng.randint(10, 20), "group": rng.choice([8, 16, 32])}
    if kind == "natural":
        H, W = rng.randint(110, 240), rng.randint(110, 320)
        B = max(_images(4, 5, H, W), min(_log(rng, 1, 64), 64 * 40000 // (H * W)))
        return {"kind": kind, "B": B, "H": H, "W": W, "T": rng.randint(10, 30)}
    if kind == "encode":
        H, W, bank = _log(rng, 40, 340), _log(rng, 40, 340), rng.choice(["dog", "gabor"])
        least = _images(6, 13, H, W) if bank == "dog" else _images(4, 5, H, W)
        return {"kind": kind, "B": max(least, min(_log(rng, 1, 64), 1600000 // (H * W))), "H": H, "W": W,
                "T": rng.randint(10, 30), "bank": bank}
    if kind == "conv":
        while True:
            K = rng.choice([3, 5, 7])
            c = {"kind": kind, "B": 1, "Cin": _log(rng, 4, 250), "H": _log(rng, 4, 64), "W": _log(rng, 4, 64),
                 "Cout": _log(rng, 16, 256), "K": K, "pad": rng.randint(0, K // 2), "stride": rng.choice([1, 1, 1, 2]),
                 "T": rng.randint(8, 32), "wave": rng.random() < 0.4, "inf": rng.random() < 0.3, "pool": 0,
                 "geometric": rng.random() < 0.3}
            Ho, Wo = _out(c)
            taps = c["Cin"] * K * K
            if Ho < 2 or Wo < 2 or taps > 7000 or (c["W"] + 2 * c["pad"]) * (c["Cin"] + 7) > 32768:
                continue
            outs = c["T"] * c["Cout"] * Ho * Wo
            c["B"] = max(1, min(1000, int(_log(rng, 2e5, 2e8) / outs), int(8e12 / (2.0 * outs * taps))))
            c["pool"] = rng.choice([0, 2]) if not c["inf"] and min(Ho, Wo) >= 2 else 0
            return c
    if kind == "learn":
        H, W = _log(rng, 12, 256), _log(rng, 12, 256)
        Cout, K = _log(rng, 20, 256), rng.choice([3, 5])
        return {"kind": kind, "B": min(_log(rng, 1, 500), max(1, (1 << 25) // (Cout * H * W))),
                "Cin": _log(rng, 4, 64), "Cout": Cout, "H": H, "W": W, "K": K, "pad": K // 2,
                "T": rng.randint(10, 64), "k": rng.randint(1, 32), "r": rng.randint(0, 4)}
    C, H, W, T = _log(rng, 8, 256), _log(rng, 8, 64), _log(rng, 8, 64), rng.randint(8, 30)
    return {"kind": kind, "B": max(1, min(500, int(_log(rng, 1e6, 3e8) / (C * H * W * T)))), "C": C, "H": H, "W": W,
            "T": T, "pool": rng.choice([2, 2, 3])}


# ------------------------------------------------------------------ sizes
def _out(c):
    return ((c["H"] + 2 * c["pad"] - c["K"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["K"]) // c["stride"] + 1)


def _conv(cin, cout, K, pad, thr, k, r, learn, a_plus=0.004, a_minus=-0.003, stabilizer=True):
    return SimpleNamespace(cin=cin, cout=cout, K=K, pad=pad, thr=thr, k=k, r=r, learn=learn, a_plus=a_plus,
                           a_minus=a_minus, lb=0.0, ub=1.0, stabilizer=stabilizer)


def _stages(c):
    """The stages of a chain case."""
    if c["kind"] == "natural":
        return [SimpleNamespace(P=7, R=6, D=0), _conv(4, 20, 17, 0, 36.0, 1, 5, "stdp")]
    # online: rates on the weights' grid and no stabilizer, so that the sums stay exact from image to image
    kw = dict(a_plus=2.0 ** -8, a_minus=-3 * 2.0 ** -10, stabilizer=False) if c["kind"] == "online" else {}
    return [_conv(6, 30, 5, 2, 15.0, 5, 3, "stdp", **kw), SimpleNamespace(P=2, R=2, D=0),
            _conv(30, 250, 3, 1, 10.0, 8, 1, "stdp", **kw), SimpleNamespace(P=3, R=3, D=0),
            _conv(250, 200, 5, 2, math.inf, 1, 0, "rstdp", **kw)]


def _threshold(c):
    """5 % of the sum of all weights, as the workloads' layers have it (Eq.5: infinite)."""
    return math.inf if c["inf"] else 0.04 * c["Cin"] * c["K"] ** 2


# ------------------------------------------------------------------ seeded inputs
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 64 + stream)
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=F32)


def _strokes(g, B, H, W):
    """Digit-like images: three line strokes of width 1 to 3, 255 on black."""
    yy = torch.arange(H, device=DEV, dtype=F32).view(1, H, 1)
    xx = torch.arange(W, device=DEV, dtype=F32).view(1, 1, W)
    on = torch.zeros((B, H, W), dtype=torch.bool, device=DEV)
    for _ in range(3):
        p = _rand(g, B, 4)
        y0, x0, y1, x1 = [(3 + p[:, j] * ((H if j % 2 == 0 else W) - 7)).view(B, 1, 1) for j in range(4)]
        w = torch.randint(1, 4, (B, 1, 1), generator=g, device=DEV).float()
        dy, dx = y1 - y0, x1 - x0
        s = (((yy - y0) * dy + (xx - x0) * dx) / (dy * dy + dx * dx).clamp_min(1e-6)).clamp(0, 1)
        on |= (yy - (y0 + s * dy)) ** 2 + (xx - (x0 + s * dx)) ** 2 <= (w / 2) ** 2 + 0.25
    return on.to(U8) * 255


def _pink(g, B, H, W):
    """Photograph-like images: 1/f noise scaled to 0..255."""
    fy, fx = torch.fft.fftfreq(H, device=DEV)[:, None], torch.fft.rfftfreq(W, device=DEV)[None, :]
    f = torch.sqrt(fy * fy + fx * fx)
    f[0, 0] = 1
    spec = torch.fft.rfft2(torch.randn((B, H, W), generator=g, device=DEV)) / f
    spec[:, 0, 0] = 0
    im = torch.fft.irfft2(spec, s=(H, W))
    lo, hi = im.amin((1, 2), keepdim=True), im.amax((1, 2), keepdim=True)
    return torch.round(255 * (im - lo) / (hi - lo).clamp_min(1e-12)).to(U8)


def _quantise(k):
    """Zero mean, largest 1, multiples of 2^-8 with sum 0."""
    k = k - k.mean()
    q = torch.round(k / k.abs().max() * 256)
    n = k.shape[0] // 2
    q[n, n] -= q.sum()
    return q / 256


def _bank(name):
    """The filter banks of the two image workloads, f32 [C, KF, KF]."""
    def grid(n):
        r = torch.arange(n, dtype=F64) - (n - 1) / 2
        return torch.meshgrid(r, r, indexing="ij")
    out = []
    if name == "dog":
        for n in (3, 7, 13):
            yy, xx = grid(n)
            d2 = yy * yy + xx * xx
            a, b = [torch.exp(-d2 / (2 * s * s)) / (2 * math.pi * s * s) for s in (n / 9, 2 * n / 9)]
            k = torch.nn.functional.pad(_quantise(a - b), [(13 - n) // 2] * 4)
            out += [k, -k]
    else:
        for th in (0, 45, 90, 135):
            yy, xx = grid(5)
            t = math.radians(th)
            u, v = xx * math.cos(t) + yy * math.sin(t), -xx * math.sin(t) + yy * math.cos(t)
            out.append(_quantise(torch.exp(-(u * u + 0.25 * v * v) / (2 * 2.8 ** 2)) * torch.cos(2 * math.pi * u / 5)))
    return torch.stack(out).float()


def _weights(g, shape, mean, std, bits):
    """Normal weights clipped to [0, 1]; with bits, rounded to multiples of 2^-bits."""
    w = (mean + std * torch.randn(shape, generator=g, device=DEV)).clamp(0, 1)
    return torch.round(w * 2 ** bits) / 2 ** bits if bits else w


def _grid_weights(c, seed, g0=10):
    """One weight tensor per conv stage, on a grid on which sums of all taps are exact."""
    out = []
    for st in _stages(c):
        if hasattr(st, "cout"):
            taps = st.cin * st.K * st.K
            bits = 11 if c["kind"] == "online" else min(16, 24 - math.ceil(math.log2(taps + 1)))
            out.append(_weights(_gen(seed, g0 + len(out)), (st.cout, st.cin, st.K, st.K), 0.8, 0.05, bits))
    return out


def _times(c, g, shape):
    """First-spike times: geometric (p = 0.05), or silent (60 %) and else uniform."""
    if c["geometric"]:
        t = torch.floor(torch.log(_rand(g, *shape).clamp_min(1e-9)) / math.log(0.95))
        return t.clamp_max(c["T"]).to(U8)
    t = torch.randint(0, c["T"], shape, generator=g, device=DEV)
    t[_rand(g, *shape) < 0.6] = c["T"]
    return t.to(U8)


def _wave(t, T):
    """Eq.1: 1 from the first-spike step on."""
    steps = torch.arange(T, device=DEV, dtype=U8).view((1, T) + (1,) * (t.dim() - 1))
    return (steps >= t.unsqueeze(1)).to(U8)


def _layer_maps(c, seed):
    """First-spike map and potential at the first spike of a layer whose features
    see the same input: a location's potential is shared but for a small part."""
    g = _gen(seed, 3)
    B, C, H, W, T = c["B"], c.get("Cout", c.get("C")), c["H"], c["W"], c["T"]
    base = torch.randn((B, 1, H, W), generator=g, device=DEV) * 4 + 40
    noise = torch.randn((B, C, H, W), generator=g, device=DEV)
    p0 = base + noise
    late = torch.randint(1, max(2, T // 3), (B, 1, H, W), generator=g, device=DEV)
    silent = _rand(g, B, 1, H, W) < 0.1
    first = p0 >= 40
    tf = torch.where(first, torch.zeros_like(late), late).masked_fill_(silent, T).to(U8)
    vf = torch.where(first, p0, p0 + 20).masked_fill_(silent.expand_as(p0), 0.0)
    return tf.contiguous(), vf.contiguous()


def _inputs(case, seed):
    """Everything a case's pass reads, by name."""
    c, k = case, case["kind"]
    if k in ("chain", "online"):
        n = c["B"] if k == "chain" else c["N"]
        return {"image": _strokes(_gen(seed, 0), n, c["H"], c["W"]), "bank": _bank("dog").to(DEV),
                "labels": torch.randint(0, 10, (n,), generator=_gen(seed, 1), device=DEV).to(I32),
                "weights": _grid_weights(c, seed)}
    if k == "natural":
        return {"image": _pink(_gen(seed, 0), c["B"], c["H"], c["W"]), "bank": _bank("gabor").to(DEV),
                "labels": torch.zeros((c["B"],), dtype=I32, device=DEV), "weights": _grid_weights(c, seed)}
    if k == "encode":
        return {"image": _pink(_gen(seed, 0), c["B"], c["H"], c["W"]), "bank": _bank(c["bank"]).to(DEV)}
    if k == "conv":
        t = _times(c, _gen(seed, 0), (c["B"], c["Cin"], c["H"], c["W"]))
        return {"t": t, "w": _weights(_gen(seed, 10), (c["Cout"], c["Cin"], c["K"], c["K"]), 0.8, 0.05, 0)}
    if k == "learn":
        tf, vf = _layer_maps(c, seed)
        t = _times(dict(c, geometric=True), _gen(seed, 0), (c["B"], c["Cin"], c["H"], c["W"]))
        return {"tf": tf, "vf": vf, "pre": t,
                "w": _weights(_gen(seed, 10), (c["Cout"], c["Cin"], c["K"], c["K"]), 0.5, 0.1, 0)}
    tf, vf = _layer_maps(c, seed)
    B, C, H, W, T = c["B"], c["C"], c["H"], c["W"], c["T"]
    steps = torch.arange(T, device=DEV).view(1, T, 1, 1, 1)
    late = (steps - tf.unsqueeze(1).long()).float()
    P = torch.where(late >= 0, vf.unsqueeze(1) + late, vf.unsqueeze(1) * 0.9 + late).clamp_min_(0)
    return {"tf": tf, "vf": vf, "P": P.contiguous()}


# ------------------------------------------------------------------ state and pass
def prepare(case, seed):
    c, k, x = case, case["kind"], _inputs(case, seed)
    s = {"case": c, **x}
    if k in ("chain", "natural"):
        full = k == "natural" or c["form"] == "full"
        bank = x["bank"]
        s["chain"] = Chain(_stages(c), c["B"], c["T"], c["H"], c["W"], 1, source="image", filter_bank=bank,
                           device=DEV, want_potentials=full, want_spikes=full, want_waves=full,
                           fused=k == "chain" and c["form"] == "fused",
                           local_norm=(c["norm"], 1e-12) if c.get("norm") else None)
        s["chain"].set_weights(x["weights"])
    elif k == "online":
        s["trainer"] = OnlineTrainer(_stages(c), c["T"], c["H"], c["W"], 1, x["bank"], device=DEV,
                                     steps_per_graph=c["group"])
        s["trainer"].set_weights(x["weights"])
        n = min(c["group"], c["N"])
        s["trainer"].run(x["image"][:n], x["labels"][:n])  # captures its graph
    elif k == "encode":
        B, H, W, T, C = c["B"], c["H"], c["W"], c["T"], x["bank"].shape[0]
        s["wave"] = torch.empty((B, T, C, H, W), dtype=U8, device=DEV)
        s["ws"] = torch.empty(max(256, spk.spk_encode_latency_workspace_size(B, C, H, W, T)), dtype=U8, device=DEV)
    elif k == "conv":
        B, T, F, (Ho, Wo) = c["B"], c["T"], c["Cout"], _out(c)
        if c["wave"]:
            s["wave"] = _wave(x["t"], T)
        s["out"] = dict(potentials=torch.empty((B, T, F, Ho, Wo), dtype=F32, device=DEV),
                        spikes=torch.empty((B, T, F, Ho, Wo), dtype=U8, device=DEV),
                        t_first=torch.empty((B, F, Ho, Wo), dtype=U8, device=DEV),
                        v_first=torch.empty((B, F, Ho, Wo), dtype=F32, device=DEV),
                        workspace=torch.empty(max(256, spk.spk_conv_fire_strided_workspace_size(
                            B, T, c["Cin"], c["H"], c["W"], F, c["K"], c["stride"], c["pad"])), dtype=U8, device=DEV))
    elif k == "learn":
        s["wave"] = _wave(x["pre"], c["T"])
        s["weight"] = x["w"].clone()
        s["ws_k"] = torch.empty(max(256, spk.spk_kwta_workspace_size(c["B"], c["Cout"], c["H"], c["W"])), dtype=U8,
                                device=DEV)
        s["ws_s"] = torch.empty(max(256, spk.spk_stdp_workspace_size(c["Cout"], c["Cin"], c["K"], c["B"], c["k"])),
                                dtype=U8, device=DEV)
    return s


def run(s):
    c = s["case"]
    k = c["kind"]
    if k in ("chain", "natural"):
        ch = s["chain"]
        ch.set_input(image=s["image"], labels=s["labels"])  # the program's next batch
        if k == "chain" and not c["learn"]:
            ch.forward()
        else:
            ch.set_weights(s["weights"])  # every pass learns from the same weights
            ch.step()
        out = {"weights": ch.weights(), "decision": ch.decision if k == "chain" else None}
        for i in ch.conv_stages():
            b = ch.bufs[i]
            out["stage%d" % i] = {n: b[n] for n in ("P", "S", "tf", "vf", "win", "nw") if b[n] is not False}
        return out
    if k == "online":
        tr = s["trainer"]
        tr.set_weights(s["weights"])
        tr.run(s["image"], s["labels"])
        last = tr.chain.bufs[-1]
        return {"weights": tr.weights(), "vf": last["vf"], "win": last["win"], "decision": tr.chain.decision}
    if k == "encode":
        return spk.spk_encode_latency(s["image"], s["bank"], c["T"], wave=s["wave"], intensities=None,
                                      workspace=s["ws"])
    if k == "conv":
        thr = _threshold(c)
        if c["wave"] and c["stride"] == 1:
            out = spk.spk_conv_fire(s["wave"], s["w"], c["pad"], thr, **s["out"])
        elif c["wave"]:
            out = spk.spk_conv_fire_strided(s["wave"], s["w"], c["stride"], c["pad"], thr, **s["out"])
        elif c["stride"] == 1:
            out = spk.spk_conv_fire_first_spike(s["t"], c["T"], s["w"], c["pad"], thr, **s["out"])
        else:
            out = spk.spk_conv_fire_first_spike_strided(s["t"], c["T"], s["w"], c["stride"], c["pad"], thr, **s["out"])
        out = dict(zip(("P", "S", "tf", "vf"), out))
        if c["pool"]:
            out["pooled"], out["pooled_tf"] = spk.spk_pool(out["S"], c["pool"], out_t_first=None)
        return out
    if k == "learn":
        s["weight"].copy_(s["w"])  # every pass learns from the same weights
        win, nw = spk.spk_kwta(s["tf"], s["vf"], c["T"], c["k"], c["r"], workspace=s["ws_k"])
        spk.spk_stdp(s["weight"], c["pad"], s["wave"], win, nw, 0.004, -0.003, workspace=s["ws_s"])
        return {"win": win, "nw": nw, "weight": s["weight"]}
    tf, vf, wave = spk.spk_pointwise_inhibition(s["tf"], s["vf"], c["T"], out_wave=None, potentials=s["P"])
    return {"tf": tf, "vf": vf, "wave": wave, "P": s["P"], "pooled": spk.spk_pool_potentials(s["P"], c["pool"])}


# ------------------------------------------------------------------ what a pass cannot do without
def _conv_work(B, T, cin, h, w, cout, K, ho, wo, per_step, inf, wave=False):
    """Bytes and operations of one conv + fire: the input and the weights once, the
    first-spike time and potential, per-step potentials and spikes where wanted; one
    addition per tap (a neuron's potential grows by a tap's weight when it spikes)
    and per step (Eq.5 has one step)."""
    neurons = B * cout * ho * wo
    byt = (T if wave else 1) * B * cin * h * w + 4 * cout * cin * K * K + 5 * neurons + 5 * T * neurons * per_step
    return byt, neurons * (cin * K * K + (0 if inf else T))


def work(case):
    c, k = case, case["kind"]
    byt = ops = 0
    if k in ("chain", "online", "natural"):
        full = k == "natural" or c.get("form") == "full"
        learn = k != "chain" or c["learn"]
        B, T, h, w, ch = c.get("B", 1), c["T"], c["H"], c["W"], 4 if k == "natural" else 6
        taps = 100 if k == "natural" else 2 * (9 + 49 + 169)
        byt, ops = B * h * w + B * ch * h * w * (1 + T * full), 2 * B * h * w * taps
        for st in _stages(c):
            if hasattr(st, "cout"):
                ho, wo = h + 2 * st.pad - st.K + 1, w + 2 * st.pad - st.K + 1
                b, o = _conv_work(B, T, ch, h, w, st.cout, st.K, ho, wo, full, math.isinf(st.thr))
                byt, ops = byt + b + 5 * B * st.cout * ho * wo + 16 * B * st.k, ops + o
                if learn:
                    byt += 8 * st.cout * st.cin * st.K ** 2 + B * st.k * st.cin * st.K ** 2
                ch, h, w = st.cout, ho, wo
            else:
                ho, wo = (h - st.P) // st.R + 1, (w - st.P) // st.R + 1
                byt += B * ch * (h * w + ho * wo * (1 + T * full))
                h, w = ho, wo
        n = c["N"] if k == "online" else 1
        return {"bytes": n * byt, "flops": n * ops}
    if k == "encode":
        n = c["B"] * c["H"] * c["W"]
        C, taps = (6, 2 * (9 + 49 + 169)) if c["bank"] == "dog" else (4, 100)
        return {"bytes": n * (1 + C * (5 + c["T"])), "flops": 2 * n * taps}
    if k == "conv":
        Ho, Wo = _out(c)
        byt, ops = _conv_work(c["B"], c["T"], c["Cin"], c["H"], c["W"], c["Cout"], c["K"], Ho, Wo, True, c["inf"],
                              c["wave"])
        if c["pool"]:
            p = c["pool"]
            byt += c["B"] * c["Cout"] * (c["T"] * Ho * Wo + (c["T"] + 1) * (Ho // p) * (Wo // p))
        return {"bytes": byt, "flops": ops}
    if k == "learn":
        n, taps = c["B"] * c["Cout"] * c["H"] * c["W"], c["Cin"] * c["K"] ** 2
        return {"bytes": 5 * n + 16 * c["B"] * c["k"] + 8 * c["Cout"] * taps + c["B"] * c["k"] * taps,
                "flops": 2 * n + 5 * c["B"] * c["k"] * taps}
    n, p = c["B"] * c["C"] * c["H"] * c["W"], c["pool"]
    m = c["B"] * c["C"] * (c["H"] // p) * (c["W"] // p)
    # the potentials are masked in place: all written, the winners' read, and read again to be pooled
    return {"bytes": 10 * n + c["T"] * (n + 8 * n + 4 * m), "flops": n + c["T"] * (n + m * p * p)}


def tolerance(case):
    k = case["kind"]
    if k in ("chain", "online", "natural", "learn"):
        # sums are exact, winners the same; an update chain is rounded to float once per update
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if k == "encode":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}  # double sums rounded once
    if k == "conv" and case["inf"]:
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}  # 32-bit sums in another order
    if k == "conv":
        # ... and a potential within rounding of the threshold may spike a step earlier or later,
        # which moves its first-spike time and potential: against 64 bits 0 to 10 of 1.7e7 neurons
        # and 0 to 3 of 1.3e7 were seen, a relative 5e-4 in v_first; four in the smallest layers
        Ho, Wo = _out(case)
        n = case["B"] * case["Cout"] * Ho * Wo
        flips = max(4.0, 2.5e-6 * n)
        return {"rel": min(0.03, max(2e-3, math.sqrt(flips / n))), "max": 0.99,
                "differ": min(0.01, flips * max(1, case["pool"] ** 2) / n)}
    return "exact"  # selection only


# ------------------------------------------------------------------ the same in 64 bits
def _exact_filter(image, bank):
    B, H, W = image.shape
    C, KF, _ = bank.shape
    p = KF // 2
    x = torch.nn.functional.pad(image.to(F64), [p] * 4)
    out = torch.zeros((B, C, H, W), dtype=F64, device=DEV)
    for ky in range(KF):
        for kx in range(KF):
            for ch in range(C):
                tap = float(bank[ch, ky, kx])
                if tap:
                    out[:, ch] += tap * x[:, ky:ky + H, kx:kx + W]
    return out.clamp_min_(0)


def _exact_rank(I, T):
    """First-spike times: the n positive entries ranked descending, equal ones by index."""
    B = I.shape[0]
    v = I.float().reshape(B, -1)
    order = torch.argsort(v, dim=1, descending=True, stable=True)
    n = (v > 0).sum(1, keepdim=True)
    rank = torch.arange(v.shape[1], device=DEV).unsqueeze(0).expand_as(v)
    t = torch.where(rank < n, rank * T // n.clamp_min(1), T).to(U8)
    return torch.empty_like(t).scatter_(1, order, t).reshape(I.shape)


def _exact_conv(t, w, T, pad, stride, thr):
    """(P, tf, vf) in 64 bits from first-spike times."""
    B, Cin, H, W = t.shape
    F, _, K, _ = w.shape
    Ho, Wo = (H + 2 * pad - K) // stride + 1, (W + 2 * pad - K) // stride + 1
    w2 = w.double().reshape(F, -1).t().contiguous()
    P = torch.zeros((B, T, F, Ho, Wo), dtype=F64, device=DEV)
    step = max(1, min(B, int(2e8 / (Ho * Wo * Cin * K * K))))
    for b in range(0, B, step):
        x = torch.nn.functional.pad(t[b:b + step], [pad] * 4, value=T)
        win = x.unfold(2, K, stride).unfold(3, K, stride).permute(0, 2, 3, 1, 4, 5).reshape(-1, Cin * K * K)
        for s in range(T - 1 if math.isinf(thr) else 0, T):
            p = (win <= s).double() @ w2
            P[b:b + step, s] = p.reshape(-1, Ho, Wo, F).permute(0, 3, 1, 2)
    on = P > 0 if math.isinf(thr) else P >= thr
    tf = T - on.sum(1)
    vf = torch.gather(P, 1, tf.clamp_max(T - 1).unsqueeze(1)).squeeze(1).masked_fill_(tf == T, 0)
    return P, tf.to(U8), vf


def _exact_kwta(tf, vf, T, k, r):
    """Winners [B,k,4] and their numbers: earliest, then largest potential, then lowest index."""
    B, C, H, W = tf.shape
    N = H * W
    t = tf.long().reshape(B, C, N).clone()
    v = vf.reshape(B, C, N)
    yy, xx = torch.arange(N, device=DEV) // W, torch.arange(N, device=DEV) % W
    idx = torch.arange(C * N, device=DEV).reshape(1, C, N)
    win = torch.full((B, k, 4), -1, dtype=torch.long, device=DEV)
    for j in range(k):
        first = t.reshape(B, -1).min(1).values.view(B, 1, 1)
        cand = t == first
        top = torch.where(cand, v, -math.inf).reshape(B, -1).max(1).values.view(B, 1, 1)
        at = torch.where(cand & (v == top), idx, C * N).reshape(B, -1).min(1).values
        f, n = at // N, at % N
        row = torch.stack([f, first.view(B), yy[n], xx[n]], 1)
        ok = (first.view(B) < T)
        win[:, j] = torch.where(ok[:, None], row, win[:, j])
        near = ((yy[None] - yy[n][:, None]).abs() <= r) & ((xx[None] - xx[n][:, None]).abs() <= r)
        gone = near.unsqueeze(1) | (torch.arange(C, device=DEV).view(1, C, 1) == f.view(B, 1, 1))
        t.masked_fill_(gone & ok.view(B, 1, 1), T)
    return win, (win[:, :, 0] >= 0).sum(1)


def _exact_stdp(w, pre, pad, win, sign, st):
    """Eq.4 image by image (pre: first-spike times; sign: +1, -1 or 0 per image)."""
    w = w.double().clone()
    K = w.shape[2]
    x = torch.nn.functional.pad(pre, [pad] * 4, value=255)
    host, signs = win.cpu().tolist(), sign.cpu().tolist()
    ltp, ltd = torch.tensor([st.a_plus, st.a_minus], dtype=F32, device=DEV).double()  # rates are floats
    for b, rows in enumerate(host):
        rows = [q for q in rows if q[0] >= 0]
        if not rows or not signs[b]:
            continue
        f = torch.tensor([q[0] for q in rows], device=DEV)
        pre_t = torch.stack([x[b, :, q[2]:q[2] + K, q[3]:q[3] + K] for q in rows])
        on = pre_t <= torch.tensor([q[1] for q in rows], device=DEV).view(-1, 1, 1, 1)
        a = torch.where(on, ltp, ltd) * signs[b]
        v = w[f]
        u = a * (v - st.lb) * (st.ub - v) if st.stabilizer else a
        w[f] = (v + u).clamp(st.lb, st.ub).float().double()
    return w


def _exact_network(c, x, weights):
    """One step of a chain's network on its images: per stage outputs, updated weights."""
    T = c["T"]
    I = _exact_filter(x["image"], x["bank"])
    t = _exact_rank(I, T)
    outs, convs, wi = {}, [], 0
    for i, st in enumerate(_stages(c)):
        if hasattr(st, "cout"):
            P, tf, vf = _exact_conv(t, weights[wi], T, st.pad, 1, st.thr)
            win, nw = _exact_kwta(tf, vf, T, st.k, st.r)
            outs["stage%d" % i] = {"P": P, "vf": vf, "win": win}
            convs.append((st, t, win))
            t, wi = tf, wi + 1
        else:
            t = t.unfold(2, st.P, st.R).unfold(3, st.P, st.R).amin((4, 5)).contiguous()
    f = convs[-1][2][:, 0, 0]
    reward = torch.where(f < 0, 0, torch.where(f % 10 == x["labels"], 1, -1))
    new = []
    for (st, pre, win), w in zip(convs, weights):
        sign = reward if st.learn == "rstdp" else torch.ones_like(reward)
        new.append(_exact_stdp(w, pre, st.pad, win, sign, st))
    return outs, new


def exact(case, seed):
    c, k, x = case, case["kind"], _inputs(case, seed)
    if k in ("chain", "natural"):
        if c.get("norm"):
            return None  # ranks of quotients: ties fall by their rounding, and every later stage with them
        outs, new = _exact_network(c, x, x["weights"])
        full = k == "natural" or c["form"] == "full"
        learn = k == "natural" or c["learn"]
        res = {"weights": new if learn else [w.double() for w in x["weights"]], "decision": None}
        for n, o in outs.items():
            res[n] = {"P": o["P"], "vf": o["vf"]} if full else {"vf": o["vf"]}
        return res
    if k == "online":
        w = [v.clone() for v in x["weights"]]
        for i in range(c["N"]):
            one = {"image": x["image"][i:i + 1], "bank": x["bank"], "labels": x["labels"][i:i + 1]}
            outs, w = _exact_network(dict(c, B=1), one, w)
        return {"weights": w, "vf": outs["stage4"]["vf"], "win": None, "decision": None}
    if k == "encode":
        return None, None, _exact_filter(x["image"], x["bank"])
    if k == "conv":
        P, _, vf = _exact_conv(x["t"], x["w"], c["T"], c["pad"], c["stride"], _threshold(c))
        if c["inf"]:
            return {"P": P, "S": None, "tf": None, "vf": vf}
        return {"P": P, "S": None, "tf": None, "vf": None}  # vf jumps where a potential is at the threshold
    if k == "learn":
        win, _ = _exact_kwta(x["tf"], x["vf"], c["T"], c["k"], c["r"])
        st = _conv(c["Cin"], c["Cout"], c["K"], c["pad"], 0.0, c["k"], c["r"], "stdp")
        sign = torch.ones((c["B"],), dtype=torch.long, device=DEV)
        return {"win": None, "nw": None, "weight": _exact_stdp(x["w"], x["pre"], c["pad"], win, sign, st)}
    t, v = x["tf"], x["vf"]
    win, n = _exact_first(t, v, c["T"])
    keep = (torch.arange(c["C"], device=DEV).view(1, -1, 1, 1) == win) & n
    P = x["P"].double() * keep.unsqueeze(1)
    p = c["pool"]
    pooled = torch.nn.functional.max_pool2d(P.reshape(-1, 1, c["H"], c["W"]), p, p).reshape(
        P.shape[:3] + (c["H"] // p, c["W"] // p))
    return {"tf": None, "vf": v.double() * keep, "wave": None, "P": P, "pooled": pooled}


def _exact_first(t, v, T):
    """Per location the winning feature [B,1,H,W] and whether any feature spikes."""
    first = t.amin(1, keepdim=True)
    cand = t == first
    top = torch.where(cand, v, -math.inf).amax(1, keepdim=True)
    idx = torch.arange(t.shape[1], device=DEV).view(1, -1, 1, 1)
    return torch.where(cand & (v == top), idx, t.shape[1]).amin(1, keepdim=True), first < T
