"""Stage-isolated parity: every libspyke call against the oracle on the same
seeded inputs, at sizes spanning several tiles with ragged tails, plus the
edge cases of each call.  Runs through the C ABI on the GPU."""
import functools
import math

import numpy as np
import pytest
import torch

import oracle as orc
import synth
import weights
from parity import assert_close, assert_equal, compare_conv_fire

spk = pytest.importorskip("paper_1903_02440_amd")

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    return t.cpu().numpy()


def dev_shifted(a, shift=1):
    """A device copy of `a` that starts `shift` elements into its allocation,
    so that its address is not aligned to the element group the kernels'
    wide loads use."""
    a = np.ascontiguousarray(a)
    flat = torch.empty(a.size + shift, dtype=torch.from_numpy(a[:0].reshape(-1)).dtype, device="cuda")
    view = flat[shift:].view(a.shape)
    view.copy_(torch.from_numpy(a))
    return view


def sync():
    torch.cuda.synchronize()


def wave_of(tf, T):
    """Eq.1 written directly with numpy (input preparation only)."""
    return (np.arange(T, dtype=np.int32)[None, :, None, None, None] >= tf[:, None].astype(np.int32)).astype(np.uint8)


# ---------------------------------------------------------------- conv + fire
def gpu_conv(wave, W, pad, thr):
    out = spk.spk_conv_fire(dev(wave), dev(W), pad, thr)
    sync()
    return tuple(host(x) for x in out)


def test_conv_toy_t1(golden):
    g = golden("t1_conv_fire.txt")
    T = int(g["T"][0])
    wave = g["wave_in"].astype(np.uint8)
    W = g["weight"].astype(np.float32)
    for thr, key in ((1.875, "a"), (2.0, "b"), (3.0, "c")):
        P, S, tf, vf = gpu_conv(wave, W, 0, thr)
        assert_equal(P, g["potentials"].astype(np.float32), "P")
        assert_equal(tf, g["t_first_" + key].astype(np.uint8), "t_first")
    P, S, tf, vf = gpu_conv(wave, W, 0, 1.875)
    assert_equal(S, g["spikes_a"].astype(np.uint8), "spikes")
    assert vf.item() == np.float32(1.875)
    P, S, tf, vf = gpu_conv(wave, W, 0, math.inf)
    assert_equal(P, g["potentials_inf"].astype(np.float32), "P inf")
    assert_equal(S, g["spikes_inf"].astype(np.uint8), "S inf")
    assert tf.item() == 2 and vf.item() == np.float32(2.625)
    P, S, tf, vf = gpu_conv(wave, W, 1, 100.0)
    assert_equal(P[0, :, 0, 0, 0], g["potentials_pad1_00"].astype(np.float32), "P pad")


CONV_CASES = [
    # name, B, T, Cin, H, W, Cout, K, pad, thr, p_silent
    ("mnist-S1", 3, 15, 6, 28, 28, 30, 5, 2, 15.0, 0.5),
    ("mnist-S2", 2, 15, 30, 14, 14, 250, 3, 1, 10.0, 0.6),
    ("mnist-S3-inf", 5, 15, 250, 4, 4, 200, 5, 2, math.inf, 0.7),
    ("natural-S2", 2, 30, 4, 26, 41, 20, 17, 0, 36.0, 0.5),
    ("T64-ragged", 2, 64, 8, 12, 11, 40, 5, 2, 12.0, 0.4),
    ("odd-sizes", 3, 7, 3, 5, 9, 17, 3, 0, 1.0, 0.5),
    ("tiny", 1, 1, 1, 1, 1, 1, 1, 0, 0.5, 0.3),
    ("inf-small", 3, 4, 2, 6, 6, 5, 3, 1, math.inf, 0.5),
    ("K1", 2, 5, 7, 3, 5, 33, 1, 0, 2.0, 0.3),
    # 9, 10, 13 and 14 position tiles per image, enough of them for whole-image
    # tasks (8 feature pairs): the feature halves of the last tile (9, 13) or of
    # the last two tiles (10, 14) go to two waves each
    ("tiles9-split", 57, 9, 12, 12, 12, 256, 3, 1, 4.0, 0.4),
    ("tiles10-split", 52, 9, 12, 12, 13, 256, 3, 1, 4.0, 0.4),
    ("tiles13-split", 40, 15, 16, 14, 14, 256, 3, 1, 6.0, 0.5),
    ("tiles14-split", 37, 15, 16, 16, 14, 256, 3, 1, 6.0, 0.5),
    # Eq.5 on few tasks: the K chunks split over workgroups, two chunks per part
    ("inf-ksplit", 112, 15, 64, 12, 12, 8, 5, 2, math.inf, 0.6),
]


# Layers whose weight fragments are streamed (a feature pair's past LDS): every feature group size and
# number of wave groups, chunks that end inside an image and maps of 1 to 3 positions (a quad of
# positions then spans images), K-steps that are no whole chunk, steps that are no whole block
STREAM_CASES = [
    # name, B, T, Cin, H, W, Cout, K, pad, stride, thr, p_silent
    ("groups-of-64", 64, 4, 64, 16, 16, 256, 3, 1, 1, 30.0, 0.6),
    ("groups-of-64-words-from-L2", 8, 2, 160, 46, 46, 256, 3, 1, 1, 60.0, 0.6),
    ("one-wave-group", 24, 3, 13, 65, 43, 70, 7, 3, 2, 20.0, 0.6),
    ("two-wave-groups", 90, 7, 4, 26, 41, 20, 17, 0, 1, 36.0, 0.5),
    ("two-wave-groups-words-from-L2", 2, 5, 160, 26, 25, 40, 5, 2, 1, 60.0, 0.6),
    ("four-wave-groups", 3, 17, 4, 26, 41, 20, 17, 0, 1, 36.0, 0.5),
    ("one-position", 37, 5, 140, 3, 3, 33, 3, 0, 1, 60.0, 0.5),
    ("three-positions", 70, 13, 150, 3, 5, 17, 3, 0, 1, 60.0, 0.5),
    ("two-by-one", 9, 1, 160, 4, 3, 65, 3, 0, 1, 10.0, 0.3),
    ("T-255", 1, 255, 200, 5, 6, 20, 3, 1, 1, 60.0, 0.2),
]


@pytest.mark.parametrize("case", STREAM_CASES, ids=[c[0] for c in STREAM_CASES])
@pytest.mark.parametrize("kind", ["normal", "dyadic", "bf16"])
def test_conv_fire_streamed_weights(case, kind, near_log):
    name, B, T, Cin, H, W, Cout, K, pad, stride, thr, ps = case
    g = synth.rng(190 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, ps)
    shape = (Cout, Cin, K, K)
    if kind == "normal":
        Wt = synth.normal_weights(g, shape, 0.8, 0.05)
    else:  # exactly summable
        Wt = synth.dyadic_weights(g, shape, Cin * K * K) if kind == "dyadic" else weights.wide_range_dyadic(
            g, shape, Cin * K * K)
    # (the oracle takes the first and the last image of the larger cases)
    Ho, Wo = (H + 2 * pad - K) // stride + 1, (W + 2 * pad - K) // stride + 1
    pick = sorted({0, B - 1}) if B * Ho * Wo * Cout * Cin * K * K > 5e8 else list(range(B))
    ref = orc.conv_fire(wave_of(tf[pick], T), Wt, pad, thr, stride)
    got = spk.spk_conv_fire_first_spike_strided(dev(tf), T, dev(Wt), stride, pad, thr)
    lone = spk.spk_conv_fire_first_spike_strided(dev(tf), T, dev(Wt), stride, pad, thr, potentials=False, spikes=False)
    odd = [dev_shifted(np.zeros(tuple(x.shape), r.dtype)) for x, r in zip(got, ref)]
    spk.spk_conv_fire_first_spike_strided(dev(tf), T, dev(Wt), stride, pad, thr, *odd)
    sync()
    near_log(f"conv streamed {name}/{kind}",
             compare_conv_fire(tuple(host(x)[pick] for x in got), ref, thr, exact_potentials=kind != "normal"),
             ref[2].size)
    if kind != "normal":
        for x, r, what in zip(got, ref, ("P", "S", "t_first", "v_first")):
            assert_equal(host(x)[pick], r, what)
    assert torch.equal(lone[2], got[2]) and torch.equal(lone[3], got[3])
    for x, o in zip(got, odd):
        assert torch.equal(x, o), "unaligned outputs"


def fin_task_form(B, Cout, Ho, Wo):
    """How the finite-threshold conv call cuts its work (a restatement of the
    host plan): ("image", split) when each task is one whole image, split being
    whether the last tile's feature halves go to two waves; ("chunks", False)
    for chunks of the flattened position space."""
    mt = -(-Ho * Wo // 16)
    n_pairs = -(-(-(-Cout // 16)) // 2)
    ct = 16 if (Ho * Wo) % 4 == 0 else 8
    while ct > 4 and n_pairs * B * mt // ct < 256:
        ct //= 2
    if mt > ct:
        return ("chunks", False)
    return ("image", (mt & 3) in (1, 2) and mt > 8 and ct == 16)


# The steps a wave takes at a time: 3, 4 or 5 by T, with two or four groups of waves
STREAM_STEP_CASES = [
    ("two-groups-of-5-steps", 90, 10, 4, 26, 41, 20, 17, 0, 1, 36.0, 0.5),
    ("two-groups-of-5-steps-words-from-L2", 14, 9, 160, 26, 25, 33, 5, 2, 1, 60.0, 0.6),
    ("two-groups-of-4-steps-words-from-L2", 14, 8, 160, 26, 25, 33, 5, 2, 1, 60.0, 0.6),
    ("four-groups-of-3-steps", 3, 11, 4, 26, 41, 20, 17, 0, 1, 36.0, 0.5),
    ("four-groups-of-3-steps-words-from-L2", 1, 9, 160, 26, 25, 33, 5, 2, 1, 60.0, 0.6),
    ("four-groups-of-5-steps-words-from-L2", 1, 18, 160, 26, 25, 33, 5, 2, 1, 60.0, 0.6),
]


def test_conv_fire_streamed_more_positions_than_a_launch_has_threads():
    # 8200 maps of 256x256 are more than 2^29 positions, in groups of 64 by 512 threads each more
    # threads than a launch may have: 41 distinct images, repeated
    n, reps, T, K = 41, 200, 4, 17
    g = synth.rng(192, 0)
    tf = synth.times_uniform_or_silent(g, (n, 1, 256, 256), T, 0.6)
    Wt = synth.dyadic_weights(g, (1, 1, K, K), K * K)
    _, _, gt, gv = spk.spk_conv_fire_first_spike(dev(tf).repeat(reps, 1, 1, 1), T, dev(Wt), 8, 20.0,
                                                 potentials=False, spikes=False)
    sync()
    _, _, rt, rv = orc.conv_fire(wave_of(tf[:3], T), Wt, 8, 20.0)
    assert_equal(host(gt[:3]), rt, "t_first")
    assert_equal(host(gv[:3]), rv, "v_first")
    for r in range(1, reps):
        assert torch.equal(gt[r * n:(r + 1) * n], gt[:n]) and torch.equal(gv[r * n:(r + 1) * n], gv[:n]), r


@pytest.mark.parametrize("case", STREAM_STEP_CASES, ids=[c[0] for c in STREAM_STEP_CASES])
@pytest.mark.parametrize("kind", ["normal", "dyadic"])
def test_conv_fire_streamed_steps(case, kind, near_log):
    test_conv_fire_streamed_weights(case, kind, near_log)


def test_split_cases_take_the_whole_image_split():
    for name in ("tiles9-split", "tiles10-split", "tiles13-split", "tiles14-split"):
        _, B, T, Cin, H, W, Cout, K, pad, thr, ps = next(c for c in CONV_CASES if c[0] == name)
        assert fin_task_form(B, Cout, H + 2 * pad - K + 1, W + 2 * pad - K + 1) == ("image", True), name


@pytest.mark.parametrize("case", CONV_CASES, ids=[c[0] for c in CONV_CASES])
@pytest.mark.parametrize("kind", ["normal", "dyadic"])
def test_conv_fire_parity(case, kind, near_log):
    name, B, T, Cin, H, W, Cout, K, pad, thr, ps = case
    g = synth.rng(100 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, ps)
    wave = wave_of(tf, T)
    if kind == "dyadic":
        Wt = synth.dyadic_weights(g, (Cout, Cin, K, K), Cin * K * K)
    else:
        Wt = synth.normal_weights(g, (Cout, Cin, K, K), 0.8, 0.05)
    gpu = gpu_conv(wave, Wt, pad, thr)
    ref = orc.conv_fire(wave, Wt, pad, thr)
    near_log(f"conv {name}/{kind}", compare_conv_fire(gpu, ref, thr, exact_potentials=(kind == "dyadic")),
             ref[2].size)
    if kind == "dyadic" and not math.isinf(thr):
        # exact arithmetic leaves nothing near threshold unresolved
        assert_equal(gpu[1], ref[1], "spikes (exact)")


@pytest.mark.parametrize("case", CONV_CASES, ids=[c[0] for c in CONV_CASES])
def test_conv_fire_first_spike_input(case, near_log):
    # the first-spike-map entry on the map of an Eq.1 wave: oracle parity on the wave, and
    # bitwise the same outputs as the wave entry
    name, B, T, Cin, H, W, Cout, K, pad, thr, ps = case
    g = synth.rng(150 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, ps)
    wave = wave_of(tf, T)
    Wt = synth.normal_weights(g, (Cout, Cin, K, K), 0.8, 0.05)
    got = spk.spk_conv_fire_first_spike(dev(tf), T, dev(Wt), pad, thr)
    via_wave = spk.spk_conv_fire(dev(wave), dev(Wt), pad, thr)
    sync()
    for a, b in zip(got, via_wave):
        assert torch.equal(a, b)
    ref = orc.conv_fire(wave, Wt, pad, thr)
    near_log(f"conv first-spike input {name}", compare_conv_fire(tuple(host(x) for x in got), ref, thr), ref[2].size)


@pytest.mark.parametrize("case", [c for c in CONV_CASES if not math.isinf(c[9])], ids=lambda c: c[0])
@pytest.mark.parametrize("kind", ["normal", "dyadic", "loguniform"])
def test_conv_fire_f32mfma_parity(case, kind, near_log):
    # the dense fp32 form of the contraction: the oracle's potentials within 1e-5 (exactly
    # summable weights: bit-exact), spikes and first-spike times under the parity rules
    name, B, T, Cin, H, W, Cout, K, pad, thr, ps = case
    g = synth.rng(160 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, ps)
    if kind == "dyadic":
        Wt = synth.dyadic_weights(g, (Cout, Cin, K, K), Cin * K * K)
    elif kind == "loguniform":
        Wt = synth.loguniform_weights(g, (Cout, Cin, K, K), 12.0, 0.1)
        thr = 0.37
    else:
        Wt = synth.normal_weights(g, (Cout, Cin, K, K), 0.8, 0.05)
    got = spk.spk_conv_fire_first_spike_f32mfma(dev(tf), T, dev(Wt), pad, thr)
    sync()
    ref = orc.conv_fire(wave_of(tf, T), Wt, pad, thr)
    near_log(f"conv f32mfma {name}/{kind}",
             compare_conv_fire(tuple(host(x) for x in got), ref, thr, exact_potentials=(kind == "dyadic")),
             ref[2].size)


# Weight ranges that the 16-bit terms of the contraction must carry: the
# layer shapes of the workloads (finite threshold and Eq.5), the natural
# layer whose fragments are read from the workspace, and a ragged small case.
RANGE_SHAPES = [
    # name, B, T, Cin, H, W, Cout, K, pad, thr
    ("S1", 3, 15, 6, 28, 28, 30, 5, 2, 1.37),
    ("S2", 2, 15, 30, 14, 14, 250, 3, 1, 1.43),
    ("S3-inf", 5, 15, 250, 4, 4, 200, 5, 2, math.inf),
    ("natural", 2, 30, 4, 26, 41, 20, 17, 0, 2.71),
    ("ragged", 3, 7, 3, 5, 9, 17, 3, 0, 0.37),
]
# (thresholds away from integers: plasticity leaves weights just below 1, so
# potentials sit near whole numbers)
RANGE_KINDS = ["loguniform", "tiny-feature", "subnormal-feature", "learned", "learned-long"]


@functools.lru_cache(maxsize=None)
def _range_weights(kind, shape_name):
    name, B, T, Cin, H, W, Cout, K, pad, thr = next(c for c in RANGE_SHAPES if c[0] == shape_name)
    return weights.range_weights(kind, (Cout, Cin, K, K), 40 + len(name), T, H, W, pad)


@pytest.mark.parametrize("case", RANGE_SHAPES, ids=[c[0] for c in RANGE_SHAPES])
@pytest.mark.parametrize("kind", RANGE_KINDS)
def test_conv_fire_weight_range(case, kind, near_log):
    # potentials within 1e-5 relative of the oracle's (exact zeros exactly) for
    # weights spread over 12 decades, features far below the layer's largest
    # weight, subnormal weights and weights shaped by plasticity
    name, B, T, Cin, H, W, Cout, K, pad, thr = case
    if kind == "learned-long" and Cin * K * K > 1000:
        pytest.skip("the oracle's plasticity run takes minutes at this size; the smaller layers cover it")
    g = synth.rng(170 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5)
    wave = wave_of(tf, T)
    Wt = _range_weights(kind, name)
    gpu = gpu_conv(wave, Wt, pad, thr)
    ref = orc.conv_fire(wave, Wt, pad, thr)
    n_near = compare_conv_fire(gpu, ref, thr)
    near_log(f"conv weight-range {name}/{kind}", n_near, ref[2].size)
    assert n_near <= ref[2].size // 100, "the case leaves too many neurons near the threshold to test spikes"


@pytest.mark.parametrize("case", RANGE_SHAPES, ids=[c[0] for c in RANGE_SHAPES])
def test_conv_fire_bf16_split_exact(case):
    # exactly summable weights of at most 17 significant bits whose range takes
    # the bf16 split: bit-exact
    name, B, T, Cin, H, W, Cout, K, pad, thr = case
    g = synth.rng(180 + len(name), 1)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5)
    wave = wave_of(tf, T)
    Wt = weights.wide_range_dyadic(g, (Cout, Cin, K, K), Cin * K * K)
    thr = math.inf if math.isinf(thr) else float(np.float32(0.37 * Cin * K * K))
    gpu = gpu_conv(wave, Wt, pad, thr)
    ref = orc.conv_fire(wave, Wt, pad, thr)
    for x, r, what in zip(gpu, ref, ("P", "S", "t_first", "v_first")):
        assert_equal(x, r, what)


def test_conv_fire_deterministic_and_optional_outputs():
    B, T, Cin, H, W, Cout, K, pad = 2, 15, 30, 14, 14, 250, 3, 1
    g = synth.rng(7, 1)
    wave = dev(wave_of(synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5), T))
    Wt = dev(synth.normal_weights(g, (Cout, Cin, K, K), 0.8, 0.05))
    a = spk.spk_conv_fire(wave, Wt, pad, 10.0)
    b = spk.spk_conv_fire(wave, Wt, pad, 10.0)
    _, _, tf, vf = spk.spk_conv_fire(wave, Wt, pad, 10.0, potentials=False, spikes=False)
    sync()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert torch.equal(tf, a[2]) and torch.equal(vf, a[3])


def test_conv_fire_unaligned_wave():
    B, T, Cin, H, W, Cout, K, pad = 2, 15, 6, 28, 28, 30, 5, 2
    g = synth.rng(8, 1)
    wave = wave_of(synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5), T)
    Wt = synth.dyadic_weights(g, (Cout, Cin, K, K), Cin * K * K)
    out = spk.spk_conv_fire(dev_shifted(wave), dev(Wt), pad, 15.0)
    sync()
    ref = orc.conv_fire(wave, Wt, pad, 15.0)
    for x, r, name in zip(out, ref, ("P", "S", "t_first", "v_first")):
        assert_equal(host(x), r, name)


# ---------------------------------------------------------------- synaptic events
@pytest.mark.parametrize("case", [(3, 15, 6, 28, 28, 30, 5, 2), (5, 15, 30, 14, 14, 250, 3, 1),
                                  (7, 15, 250, 4, 4, 200, 5, 2), (2, 30, 4, 26, 41, 20, 17, 0),
                                  (3, 7, 3, 5, 9, 17, 3, 1), (1, 4, 2, 3, 3, 1, 3, 0), (13, 9, 5, 7, 7, 11, 3, 2)])
def test_count_events_parity(case):
    # batch * output positions not a multiple of 64 in the last cases (the reduction's tail), padding in most
    B, T, Cin, H, W, Cout, K, pad = case
    g = synth.rng(140 + H + Cin, 0)
    tf = synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.6)
    count = spk.spk_count_events(dev(wave_of(tf, T)), Cout, K, pad)
    sync()
    assert int(count.item()) == orc.count_events(tf, T, Cout, K, pad)


# ---------------------------------------------------------------- pool
# (B, T, C, H, W, P, R, D).  First-spike pooling stages whole planes in LDS
# (blocks of channels) when C*Ho*Wo is a multiple of 4 and a plane holds at
# most 16 KB: the first two (a partial last block), (4x4 window with padding)
# and (odd 5x5 output planes); the 160x250 planes and the rest take the
# direct paths.
POOL_CASES = [(3, 15, 30, 28, 28, 2, 2, 0), (2, 15, 250, 14, 14, 3, 3, 0), (2, 30, 4, 160, 250, 7, 6, 0),
              (2, 7, 3, 9, 10, 3, 2, 1), (1, 5, 2, 5, 5, 5, 1, 2), (2, 3, 1, 1, 1, 1, 1, 0),
              (2, 9, 8, 12, 12, 4, 2, 1), (2, 5, 12, 10, 10, 2, 2, 0),
              # batches of a few hundred images
              (256, 15, 30, 8, 8, 2, 2, 0), (260, 15, 25, 9, 9, 3, 3, 0),
              # waves through LDS: blocks of maps that end in the last bytes and outputs of no whole
              # quad, one map a block, more outputs than inputs; a map past LDS; T > 127
              (2, 15, 37, 13, 11, 3, 3, 0), (1, 4, 3, 127, 129, 5, 4, 2), (2, 200, 5, 6, 7, 2, 1, 1),
              (1, 3, 2, 130, 130, 3, 3, 0), (3, 15, 130, 3, 5, 2, 2, 0), (1, 3, 2, 60, 60, 2, 1, 0)]


@pytest.mark.parametrize("case", POOL_CASES)
def test_pool_parity(case):
    B, T, C, H, W, P, R, D = case
    g = synth.rng(200 + H, 0)
    tf = synth.times_uniform_or_silent(g, (B, C, H, W), T, 0.7)
    wave = wave_of(tf, T)
    out, otf = spk.spk_pool(dev(wave), P, R, D, out_t_first=None)
    sync()
    ref = orc.pool(wave, P, R, D)
    assert_equal(host(out), ref, "pooled wave")
    assert_equal(host(otf), orc.first_spike(ref), "pooled t_first")
    so, _ = spk.spk_pool(dev_shifted(wave), P, R, D, out_wave=dev_shifted(np.zeros_like(ref)))
    sync()
    assert_equal(host(so), ref, "pooled wave, unaligned")


# Batches from which waves go through LDS (192 workgroups of 2x2 or 3x3 windows, 512 of others, 640 from 6x6
# on) and the ones just below: a map a workgroup or all maps of an image, ragged quads, maps that end
# in the last bytes, padding, more outputs than inputs, T > 127
@pytest.mark.parametrize("case", [(191, 3, 37, 13, 11, 3, 3, 0), (192, 3, 37, 13, 11, 3, 3, 0),
                                  (192, 3, 130, 3, 5, 2, 2, 0), (97, 5, 30, 28, 28, 2, 2, 0),
                                  (171, 3, 3, 127, 129, 5, 4, 2), (170, 3, 3, 127, 129, 5, 4, 2),
                                  (512, 200, 2, 6, 7, 2, 1, 1), (511, 3, 5, 6, 7, 2, 1, 1),
                                  (512, 3, 8, 12, 12, 4, 2, 1), (640, 2, 5, 19, 21, 7, 6, 0)])
def test_pool_parity_batches(case):
    test_pool_parity(case)


@pytest.mark.parametrize("case", POOL_CASES)
def test_pool_first_spike_parity(case):
    B, T, C, H, W, P, R, D = case
    g = synth.rng(250 + H, 0)
    tf = synth.times_uniform_or_silent(g, (B, C, H, W), T, 0.7)
    out, otf = spk.spk_pool_first_spike(dev(tf), T, P, R, D)
    sync()
    ref = orc.pool(wave_of(tf, T), P, R, D)
    assert_equal(host(out), ref, "pooled wave")
    assert_equal(host(otf), orc.first_spike(ref), "pooled t_first")


def test_pool_toy_t2(golden):
    g = golden("t2_pool.txt")
    T = int(g["T"][0])
    out, otf = spk.spk_pool(dev(wave_of(g["t_first_in"].astype(np.uint8), T)), 2, 2, 0, out_t_first=None)
    sync()
    assert_equal(host(otf), g["t_first_out"].astype(np.uint8), "T2")


# ---------------------------------------------------------------- pointwise inhibition, potentials pooling
@pytest.mark.parametrize("case", [(3, 15, 30, 28, 28), (2, 15, 250, 14, 14), (2, 9, 7, 5, 3), (1, 4, 1, 2, 2),
                                  (2, 15, 200, 4, 4)])
def test_pointwise_inhibition_parity(case):
    B, T, C, H, W = case
    g = synth.rng(700 + C + H, 0)
    tf = synth.times_uniform_or_silent(g, (B, C, H, W), T, 0.5)
    vf = (g.integers(0, 6, (B, C, H, W)) * 0.5).astype(np.float32)  # ties decided by the feature index
    vf[tf >= T] = 0
    pot = g.normal(0, 3, (B, T, C, H, W)).astype(np.float32)
    rt, rv, rp = orc.pointwise_inhibition(tf, vf, T, pot)
    gp = dev(pot)
    ot, ov, ow = spk.spk_pointwise_inhibition(dev(tf), dev(vf), T, out_wave=None, potentials=gp)
    sync()
    assert_equal(host(ot), rt, "t_first")
    assert_equal(host(ov), rv, "v_first")
    assert_equal(host(ow), orc.expand_wave(rt, T), "wave")
    assert_equal(host(gp), rp, "masked potentials")
    # in place, without the optional outputs
    it, iv = dev(tf), dev(vf)
    spk.spk_pointwise_inhibition(it, iv, T, out_t_first=it, out_v_first=iv)
    sync()
    assert_equal(host(it), rt, "t_first in place")
    assert_equal(host(iv), rv, "v_first in place")


# Runs of up to 1024 locations: ragged quads, a run of the last few, one location, T > 127, many
# parts per run; unaligned tensors; potentials that are no numbers or infinite
@pytest.mark.parametrize("case", [(1, 6, 9, 40, 41), (2, 130, 3, 33, 32), (3, 15, 1, 1, 1), (1, 20, 260, 32, 32),
                                  (2, 7, 5, 27, 38)])
@pytest.mark.parametrize("put", [dev, dev_shifted])
def test_pointwise_inhibition_runs(case, put):
    B, T, C, H, W = case
    g = synth.rng(720 + C + H, 0)
    tf = synth.times_uniform_or_silent(g, (B, C, H, W), T, 0.5)
    tf[:, :, 0] = g.integers(0, 2, (B, C, W))  # equal times: the potentials decide
    vf = (g.integers(0, 6, (B, C, H, W)) * 0.5).astype(np.float32)
    vf[g.random(vf.shape) < 0.2] = np.nan
    vf[g.random(vf.shape) < 0.1] = -np.inf
    vf[g.random(vf.shape) < 0.05] = np.inf
    vf[tf >= T] = 0
    pot = g.normal(0, 3, (B, T, C, H, W)).astype(np.float32)
    rt, rv, rp = orc.pointwise_inhibition(tf, vf, T, pot)
    gp, it, iv = put(pot), put(tf), put(vf)
    ot, ov, ow = spk.spk_pointwise_inhibition(it, iv, T, out_wave=None, potentials=gp)
    spk.spk_pointwise_inhibition(it, iv, T, out_t_first=it, out_v_first=iv)
    sync()
    for what, t, v in (("", ot, ov), (" in place", it, iv)):
        assert_equal(host(t), rt, "t_first" + what)
        assert_equal(np.isnan(host(v)), np.isnan(rv), "v_first not a number" + what)
        assert_equal(np.nan_to_num(host(v), nan=-1.0), np.nan_to_num(rv, nan=-1.0), "v_first" + what)
    assert_equal(host(ow), orc.expand_wave(rt, T), "wave")
    assert_equal(host(gp), rp, "masked potentials")


# Both forms, on both sides of the rule between them: one thread per location (few features, many
# or large maps) and workgroups that share a run's features (many features, few small maps); with
# the wave and the potentials the workgroups take larger maps too
@pytest.mark.parametrize("case", [(2, 31, 14, 14), (2, 32, 14, 14), (65, 64, 14, 14), (66, 64, 14, 14),
                                  (1, 40, 20, 22), (1, 40, 20, 23), (1, 100, 7, 9), (80, 100, 7, 9),
                                  (2049, 40, 2, 2), (3, 7, 16, 16), (3, 8, 16, 16), (26, 8, 39, 41),
                                  (4097, 9, 2, 2)])
@pytest.mark.parametrize("put", [dev, dev_shifted])
def test_pointwise_inhibition_forms(case, put):
    B, C, H, W = case
    T = 4
    g = synth.rng(760 + C + H, 0)
    tf = g.integers(0, T + 1, case).astype(np.uint8)
    vf = (g.integers(0, 5, case) * 0.5).astype(np.float32)
    pot = g.normal(0, 3, (B, T, C, H, W)).astype(np.float32)
    rt, rv, rp = orc.pointwise_inhibition(tf, vf, T, pot)
    gp, it, iv = put(pot), put(tf), put(vf)
    first = spk.spk_pointwise_inhibition(it, iv, T)
    steps = spk.spk_pointwise_inhibition(it, iv, T, out_wave=None, potentials=gp)
    spk.spk_pointwise_inhibition(it, iv, T, out_t_first=it, out_v_first=iv)
    sync()
    for what, (t, v) in (("first spikes", first[:2]), ("with steps", steps[:2]), ("in place", (it, iv))):
        assert_equal(host(t), rt, "t_first, " + what)
        assert_equal(host(v), rv, "v_first, " + what)
    assert_equal(host(steps[2]), orc.expand_wave(rt, T), "wave")
    assert_equal(host(gp), rp, "masked potentials")


def test_pointwise_inhibition_many_small_images():
    # more images than one launch has workgroups of 512 threads (2^23): the result of 1009 distinct
    # images, repeated
    T, C, n, B = 5, 3, 1009, (1 << 23) + 700
    g = synth.rng(735, 0)
    tf = g.integers(0, T + 1, (n, C, 1, 1)).astype(np.uint8)
    vf = (g.integers(0, 4, (n, C, 1, 1)) * 0.5).astype(np.float32)
    rt, rv = orc.pointwise_inhibition(tf, vf, T)
    reps = -(-B // n)

    def many(a):
        return dev(a).repeat(reps, 1, 1, 1)[:B].contiguous()

    ot, ov, _ = spk.spk_pointwise_inhibition(many(tf), many(vf), T)
    sync()
    assert torch.equal(ot, many(rt)), "t_first"
    assert torch.equal(ov, many(rv)), "v_first"


@pytest.mark.parametrize("shape", [(2, 5, 27, 38), (1, 9, 40, 41), (3, 7, 1, 1)])
def test_pointwise_inhibition_copies_the_winners_bits(shape):
    # a winner's potential is copied: one that is no number keeps its sign and payload
    T = 3
    g = synth.rng(730 + shape[1], 0)
    tf = g.integers(0, T + 1, shape).astype(np.uint8)
    vf = (g.integers(-3, 4, shape) * 0.5).astype(np.float32)
    nan = g.random(shape) < 0.4
    vf[nan] = (g.integers(0x7FC00000, 0x7FD00000, shape) | g.integers(0, 2, shape) << 31).astype(np.uint32).view(
        np.float32)[nan]
    rt, rv = orc.pointwise_inhibition(tf, vf, T)
    ot, ov, _ = spk.spk_pointwise_inhibition(dev(tf), dev(vf), T)
    sync()
    assert_equal(host(ot), rt, "t_first")
    assert_equal(host(ov).view(np.uint32), rv.view(np.uint32), "v_first (bits)")


@pytest.mark.parametrize("shape,T", [((3, 250, 14, 14), 1), ((1, 250, 14, 14), 15), ((2, 64, 40, 41), 1)])
def test_pointwise_inhibition_outputs_over_inputs(shape, T):
    # one step's potentials are the potentials at the first spike, and one step's wave has the size of
    # the first-spike map; of one image, any step of the potentials may be the input.  All of a
    # location's inputs are read before anything is written there, whichever output lies over them.
    B, C, H, W = shape
    g = synth.rng(740 + C + T, 0)
    tf = synth.times_uniform_or_silent(g, shape, T, 0.5)
    pot = g.normal(0, 3, (B, T, C, H, W)).astype(np.float32)
    vf = np.ascontiguousarray(pot[:, T - 1])
    rt, rv, rp = orc.pointwise_inhibition(tf, vf, T, pot)
    gp = dev(pot)
    over = gp[:, T - 1]
    assert over.is_contiguous()
    ot, ov, _ = spk.spk_pointwise_inhibition(dev(tf), over, T, potentials=gp)
    sync()
    assert_equal(host(ot), rt, "t_first, potentials over v_first")
    assert_equal(host(ov), rv, "v_first, potentials over v_first")
    assert_equal(host(gp), rp, "masked potentials over v_first")
    if T == 1:
        it = dev(tf)
        ot, ov, ow = spk.spk_pointwise_inhibition(it, dev(vf), T, out_wave=it.view(B, T, C, H, W))
        sync()
        assert_equal(host(ot), rt, "t_first, wave over t_first")
        assert_equal(host(ov), rv, "v_first, wave over t_first")
        assert_equal(host(ow), orc.expand_wave(rt, T), "wave over t_first")


# 2x2 windows of stride 2 on widths that are multiples of 4 take 16-byte loads of
# two rows (the 28x28 map; an odd height, whose last row no window covers); the
# rest one output per thread
@pytest.mark.parametrize("case", [(2, 15, 30, 28, 28, 2, 2, 0), (2, 15, 250, 14, 14, 3, 3, 0),
                                  (1, 5, 4, 9, 11, 3, 2, 1), (1, 3, 2, 7, 7, 4, 3, 2), (2, 4, 3, 5, 6, 1, 1, 0),
                                  (2, 3, 5, 9, 12, 2, 2, 0), (1, 2, 3, 6, 10, 2, 2, 0),
                                  (2, 3, 5, 7, 14, 2, 2, 0), (1, 2, 3, 2, 2, 2, 2, 0)])  # (even widths: 8-byte loads)
def test_pool_potentials_parity(case):
    B, T, C, H, W, P, R, D = case
    g = synth.rng(800 + P + C, 0)
    pot = (g.integers(-8, 9, (B, T, C, H, W)) * 0.25).astype(np.float32)  # ties, zeros and negatives
    pot[..., 0, 0] = -0.0
    out = spk.spk_pool_potentials(dev(pot), P, R, D)
    sync()
    ref = orc.pool_potentials(pot, P, R, D)
    assert_equal(host(out).view(np.uint32), ref.view(np.uint32), "pooled potentials (bit patterns)")


# ---------------------------------------------------------------- kWTA
# (B, T, C, H, W, k, radius).  Per-position top-k path: the first five, the
# 1x1 and 1x9 maps, (300 maps of 10x10: feature split with the stash) and
# (k = 16); units: (40x300 maps), (k = 20 > 16) and (k = 16 with lists beyond
# LDS), KWTA_UNIT_CASES and test_kwta_large_tiles.
KWTA_CASES = [(4, 15, 30, 28, 28, 5, 3), (3, 15, 250, 14, 14, 8, 1), (6, 15, 200, 4, 4, 1, 0),
              (2, 30, 20, 10, 25, 1, 5), (3, 4, 3, 5, 7, 12, 1), (2, 15, 5, 40, 300, 6, 2),
              (3, 15, 40, 1, 1, 4, 0), (2, 15, 7, 1, 9, 3, 1), (2, 15, 300, 10, 10, 8, 2),
              (2, 15, 64, 6, 6, 16, 1), (2, 15, 30, 12, 12, 20, 1), (2, 15, 20, 30, 40, 16, 0),
              # below 8 images the lists come from a grid of (image, feature split) workgroups;
              # from 8 on from the rounds' own workgroup (1 to 13 feature splits per position)
              (1, 15, 250, 14, 14, 8, 1), (8, 15, 250, 14, 14, 8, 1), (9, 15, 30, 28, 28, 5, 3),
              (8, 15, 64, 6, 6, 10, 1), (8, 15, 7, 3, 5, 3, 1), (8, 15, 40, 8, 12, 11, 2),
              # the rounds keep each position's best key in registers when a thread owns at most
              # 4 positions (256 images: 256 threads, 3 or 4 positions each), else they walk the
              # lists in LDS every round (65x65 maps: 896 threads, up to 5 positions each)
              (256, 15, 30, 28, 28, 5, 3), (2, 15, 2, 65, 65, 1, 3)]


def kwta_inputs(seed, B, T, C, H, W, ties=True):
    g = synth.rng(300 + seed, 0)
    tf = synth.times_uniform_or_silent(g, (B, C, H, W), T, 0.6)
    if ties:
        vf = (g.integers(0, 6, (B, C, H, W)) * 0.5).astype(np.float32)
    else:
        vf = g.uniform(0, 40, (B, C, H, W)).astype(np.float32)
    vf[tf >= T] = 0
    return tf, vf


@pytest.mark.parametrize("case", KWTA_CASES)
@pytest.mark.parametrize("ties", [True, False])
def test_kwta_parity(case, ties):
    B, T, C, H, W, k, r = case
    tf, vf = kwta_inputs(C + H, B, T, C, H, W, ties)
    win, nw = spk.spk_kwta(dev(tf), dev(vf), T, k, r)
    sync()
    rw, rn = orc.kwta(tf, vf, T, k, r)
    assert_equal(host(nw), rn, "n_winners")
    assert_equal(host(win), rw, "winners")


@pytest.mark.parametrize("case", KWTA_CASES[:2] + [(9, 15, 30, 28, 28, 5, 3)])
def test_kwta_unaligned_inputs(case):
    B, T, C, H, W, k, r = case
    tf, vf = kwta_inputs(C + H + 1, B, T, C, H, W, False)
    win, nw = spk.spk_kwta(dev_shifted(tf), dev_shifted(vf), T, k, r)
    sync()
    rw, rn = orc.kwta(tf, vf, T, k, r)
    assert_equal(host(nw), rn, "n_winners")
    assert_equal(host(win), rw, "winners")


# Units of 64 positions (below 4096 of them) or 256 (aligned or not) times 1 to 4096 maps
KWTA_UNIT_CASES = [(1, 15, 4096, 1, 1, 40, 0), (2, 255, 300, 8, 8, 32, 2), (2, 15, 70, 13, 5, 17, 1),
                   (3, 15, 5, 63, 65, 20, 3), (2, 15, 9, 64, 64, 20, 90), (1, 15, 40, 65, 64, 33, 5),
                   (1, 20, 3, 256, 256, 3, 4), (2, 15, 600, 17, 40, 32, 2)]


@pytest.mark.parametrize("case", KWTA_UNIT_CASES)
@pytest.mark.parametrize("kind", ["ties", "shared", "dominated"])
def test_kwta_units(case, kind):
    """Random keys with ties; features that see the same input (their maxima at the same places);
    features of which each is the best almost everywhere until it is retired."""
    B, T, C, H, W, k, r = case
    tf, vf = kwta_inputs(C + W, B, T, C, H, W, True)
    g = synth.rng(330 + C, 0)
    if kind == "shared":
        tf = np.broadcast_to(g.integers(0, T + 1, (B, 1, H, W)), (B, C, H, W)).astype(np.uint8)
        vf = (g.normal(40, 4, (B, 1, H, W)) + g.normal(0, 0.01, (B, C, H, W))).astype(np.float32)
    elif kind == "dominated":
        tf = np.zeros((B, C, H, W), np.uint8)
        vf = (g.permutation(C)[None, :, None, None] * 100.0 + g.uniform(0, 40, (B, 1, H, W))).astype(np.float32)
    vf[tf >= T] = 0
    rw, rn = orc.kwta(tf, vf, T, k, r)
    for put in (dev, dev_shifted):
        win, nw = spk.spk_kwta(put(tf), put(vf), T, k, r)
        sync()
        assert_equal(host(nw), rn, "n_winners")
        assert_equal(host(win), rw, "winners")


# Runs of 7 maps, whose retired ones lie in two words of the bitmap; more rounds than maps; a last
# run of one map; runs of 9 maps, read in two parts (256 groups of positions); fewer units than
# waves; shared places, so that one winner's window invalidates all runs
@pytest.mark.parametrize("case", [(2, 6, 33, 20, 20, 40, 0), (3, 5, 9, 9, 9, 17, 1), (1, 8, 130, 256, 256, 20, 3),
                                  (2, 15, 250, 14, 14, 20, 1), (1, 15, 512, 7, 7, 20, 0), (9, 7, 17, 64, 64, 25, 2)])
def test_kwta_units_runs(case):
    B, T, C, H, W, k, r = case
    g = synth.rng(880 + C + H, 0)
    place = g.integers(0, T + 3, (B, 1, H, W))
    tf = np.minimum(place + (g.random((B, C, H, W)) < 0.2), T).astype(np.uint8)
    vf = (g.integers(0, 7, (B, C, H, W)) * 0.5).astype(np.float32)
    vf[tf >= T] = 0
    win, nw = spk.spk_kwta(dev(tf), dev(vf), T, k, r)
    sync()
    rwin, rnw = orc.kwta(tf, vf, T, k, r)
    assert_equal(host(nw), rnw, "n_winners")
    assert_equal(host(win), rwin, "winners")


@pytest.mark.parametrize("B,C", [((1 << 23) + 700, 2), ((1 << 17) + 5, 4096)])
def test_kwta_units_many_small_images(B, C):
    # more images than one launch holds workgroups of 512 threads (2^23 of 2 neurons) or of 4 units
    # (2^24, 128 an image): the winners of 503 distinct images, repeated
    T, k, n = 4, 17, 503
    tf, vf = kwta_inputs(C, n, T, C, 1, 1, True)
    reps = -(-B // n)

    def many(a):
        return dev(a).repeat((reps,) + (1,) * (a.ndim - 1))[:B].contiguous()

    win, nw = spk.spk_kwta(many(tf), many(vf), T, k, 0)
    sync()
    rw, rn = orc.kwta(tf, vf, T, k, 0)
    assert torch.equal(nw, many(rn)), "n_winners"
    assert torch.equal(win, many(rw)), "winners"


def test_kwta_toy_t3_and_silent(golden):
    g = golden("t3_kwta.txt")
    T = int(g["T"][0])
    tf, vf = dev(g["t_first"].astype(np.uint8)), dev(g["v_first"].astype(np.float32))
    for k, r, key in ((2, 0, "win_k2_r0"), (2, 1, "win_k2_r1"), (5, 1, "win_k5_r1")):
        win, nw = spk.spk_kwta(tf, vf, T, k, r)
        sync()
        assert_equal(host(win), g[key].astype(np.int32), key)
    win, nw = spk.spk_kwta(dev(g["tie_t_first"].astype(np.uint8)), dev(g["tie_v_first"].astype(np.float32)), T, 1, 0)
    sync()
    assert_equal(host(win), g["tie_win"].astype(np.int32), "tie")
    silent = np.full((2, 3, 4, 4), 9, np.uint8)
    win, nw = spk.spk_kwta(dev(silent), dev(np.zeros((2, 3, 4, 4), np.float32)), 9, 3, 1)
    sync()
    assert host(nw).tolist() == [0, 0] and (host(win) == -1).all()


def test_kwta_large_tiles():
    # 256 maps of 256x256: several rows per tile, the multi-row recompute path
    B, T, C, H, W, k, r = 1, 64, 256, 256, 256, 32, 4
    g = synth.rng(77, 0)
    tf = synth.times_geometric(g, (B, C, H, W), T, 0.05)
    vf = g.uniform(0, 100, (B, C, H, W)).astype(np.float32)
    vf[tf >= T] = 0
    win, nw = spk.spk_kwta(dev(tf), dev(vf), T, k, r)
    sync()
    rw, rn = orc.kwta(tf, vf, T, k, r)
    assert_equal(host(nw), rn, "n_winners")
    assert_equal(host(win), rw, "winners")


# ---------------------------------------------------------------- encoding
def test_encode_toy_t4(golden):
    # rank-order only: a 1-channel identity filter passes the intensities through
    g = golden("t4_rank.txt")
    I = g["intensity"].astype(np.float32)[0]  # [1,2,3]
    img = np.clip(I * 10, 0, 255).astype(np.uint8)  # positives keep their order and ties
    ident = np.ones((1, 1, 1), np.float32)
    for T in (2, 3):
        wave, tf, inten = spk.spk_encode_latency(dev(img), dev(ident), T, intensities=None)
        sync()
        assert_equal(host(tf), g[f"t_first_T{T}"].astype(np.uint8), f"T{T}")


ENC_CASES = [("dog", 3, 28, 28, 15, 0.0), ("gabor", 2, 160, 250, 30, 0.0), ("dog", 2, 28, 28, 1, 0.0),
             ("dog", 2, 28, 28, 64, 0.0), ("dog", 1, 28, 28, 255, 0.0), ("rand", 2, 19, 23, 15, 3.0),
             ("pos", 2, 40, 50, 15, 0.0), ("pos", 1, 41, 50, 15, 0.0), ("pos", 3, 1, 1, 15, 0.0),
             ("dog", 1, 100, 300, 15, 0.0),  # 13x13 filters on a wide image: bands of rows
             ("float", 3, 28, 28, 15, 0.0),  # general float taps: the sum order decides the bits
             ("float", 2, 9, 13, 30, -0.5),  # ragged width, negative threshold
             ("flat", 2, 40, 40, 15, 0.0),  # all intensities equal: the index decides every rank
             ("edge", 2, 28, 28, 15, 0.0),  # integer filter form near its int32 bound; a zero channel
             ("bound", 2, 20, 24, 15, 0.0),  # one bit past the integer form's bound: the double form
             # the targets' first digits hold 936 and 968 (padded) keys, and 584 and 592: ranked
             # directly, past the 512 of 64-bit keys the rank step once held
             ("pos", 2, 16, 24, 15, 0.0), ("noise", 2, 40, 40, 15, 0.0)]


@pytest.mark.parametrize("case", ENC_CASES)
def test_encode_parity(case):
    kind, B, H, W, T, thr = case
    g = synth.rng(400 + T, 0)
    if kind == "dog":
        img, bank = synth.stroke_images(g, B, H, W), synth.dog_bank()
    elif kind == "gabor":
        img, bank = synth.pink_noise_images(g, B, H, W), synth.gabor_bank()
    elif kind == "noise":
        img, bank = synth.pink_noise_images(g, B, H, W), synth.dog_bank()
    elif kind == "pos":  # 4 positive filters on a noise image: every entry is ranked
        img = g.integers(1, 256, (B, H, W)).astype(np.uint8)
        bank = (g.integers(1, 65, (4, 3, 3)) / 64.0).astype(np.float32)
    elif kind == "float":
        # channels 1 = -0 and 5 = -4 are exact negations (computed once on the GPU); 3 is
        # -2 but for one tap; 4 = -3 although 3 is itself nearly a negation; taps spread
        # over 2^-20..2^2, so partial sums round and only the defined order reproduces them
        img = synth.stroke_images(g, B, H, W) if H >= 8 else g.integers(0, 256, (B, H, W)).astype(np.uint8)
        base = (g.normal(0, 1, (3, 5, 5)) * np.exp2(g.integers(-20, 3, (3, 5, 5)))).astype(np.float32)
        bank = np.stack([base[0], -base[0], base[1], -base[1], base[2], -base[2]])
        bank[3, 2, 2] += np.float32(0.25)
        bank[4] = -bank[3]
        bank[5] = -bank[4]
    elif kind == "edge":
        # taps k / 2^10, |k| < 2^14: exponent 3 + 10 fraction bits = 13 <= 14, and
        # 169 * 255 * 2^14 < 2^31; sums reach ~2^29 on random pixels.  Channel 1 is
        # all zeros, channel 2 the negation of channel 0 (derived)
        img = g.integers(0, 256, (B, H, W)).astype(np.uint8)
        k = g.integers(-16383, 16384, (13, 13))
        k[6, 6] = 16383
        bank = np.stack([k / 1024.0, np.zeros((13, 13)), -k / 1024.0]).astype(np.float32)
    elif kind == "bound":
        # taps k / 2^11, |k| < 2^15, and one tap k = 2^15 (16.0): one bit past the
        # integer form's int16 limit, so the double form
        img = g.integers(0, 256, (B, H, W)).astype(np.uint8)
        k = g.integers(-32767, 32768, (2, 5, 5))
        k[1, 2, 2] = 32768
        bank = (k / 2048.0).astype(np.float32)
    elif kind == "flat":  # a constant image through a 1x1 filter
        img = np.full((B, H, W), 200, np.uint8)
        img[1, :3, :5] = 0
        bank = np.ones((1, 1, 1), np.float32)
    else:
        img = g.integers(0, 256, (B, H, W)).astype(np.uint8)
        bank = (g.integers(-64, 65, (5, 7, 7)) / 64.0).astype(np.float32)
    wave, tf, inten = spk.spk_encode_latency(dev(img), dev(bank), T, thr, intensities=None)
    sync()
    I, rtf, rwave = orc.encode(img, bank, T, thr)
    assert_equal(host(inten), I, "intensities")
    assert_equal(host(tf), rtf, "t_first")
    assert_equal(host(wave), rwave, "wave")


@pytest.mark.parametrize("B,H,W", [(2, 160, 250), (2, 156, 286), (3, 100, 120)])
def test_encode_few_images_stay_in_their_buffers(B, H, W):
    # few images: the filter's bands are cut thinner than LDS asks for, and a height that they
    # do not divide must not leave workgroups for images past the batch
    g = synth.rng(460, H)
    img, bank = synth.pink_noise_images(g, B, H, W), synth.gabor_bank()
    room = torch.full((3 * B, 4, H, W), -7.0, dtype=torch.float32, device="cuda")
    _, tf, inten = spk.spk_encode_latency(dev(img), dev(bank), 15, wave=False, intensities=room[:B])
    sync()
    I, rtf, _ = orc.encode(img, bank, 15, 0.0)
    assert_equal(host(inten), I, "intensities")
    assert_equal(host(tf), rtf, "t_first")
    assert (host(room[B:]) == -7.0).all(), "intensities past the batch were written"


@pytest.mark.parametrize("B,C,H,W", [(2, 65, 160, 30), (2, 70, 101, 22), (3, 65, 100, 40)])
def test_encode_few_images_by_bands_stay_in_their_buffers(B, C, H, W):
    # more than 64 channels are filtered by bands of rows, cut thinner for few images: heights that
    # the bands do not divide (160 rows and 64 bands asked for: 54 of 3 rows) must not leave
    # workgroups for images past the batch
    g = synth.rng(463, C + H)
    img = g.integers(0, 256, (B, H, W)).astype(np.uint8)
    bank = (g.integers(-64, 65, (C, 3, 3)) / 64.0).astype(np.float32)
    room = torch.full((3 * B, C, H, W), -7.0, dtype=torch.float32, device="cuda")
    _, tf, inten = spk.spk_encode_latency(dev(img), dev(bank), 15, wave=False, intensities=room[:B])
    sync()
    I, rtf, _ = orc.encode(img, bank, 15, 0.0)
    assert_equal(host(inten), I, "intensities")
    assert_equal(host(tf), rtf, "t_first")
    assert (host(room[B:]) == -7.0).all(), "intensities past the batch were written"


# Filter by tiles (more than 2^19 outputs): sides of one tile and a little more (33 rows, evened out:
# 17 and 16; 65 columns: 64 and 1), of less than a group of 8 columns, whole tiles; both
# arithmetic forms; channels that negate the one before; more channels than tiles count digits for
@pytest.mark.parametrize("kind", ["dog", "integer", "double"])
@pytest.mark.parametrize("B,H,W", [(60, 33, 65), (31, 64, 64), (170, 400, 3), (900, 28, 28), (5, 161, 253)])
def test_encode_tiles_parity(kind, B, H, W):
    g = synth.rng(464, H + len(kind))
    n = 3 if B > 3 else B  # distinct images, repeated
    img = g.integers(0, 256, (n, H, W)).astype(np.uint8)
    bank = {"dog": synth.dog_bank, "integer": lambda: (g.integers(-64, 65, (5, 7, 7)) / 64.0).astype(np.float32),
            "double": lambda: g.normal(0, 1, (40 if B == 900 else 7, 5, 5)).astype(np.float32)}[kind]()
    assert B * len(bank) * H * W > 1 << 19
    wave, tf, inten = spk.spk_encode_latency(dev(img[np.arange(B) % n]), dev(bank), 7, 0.5, intensities=None)
    _, _, lone = spk.spk_encode_latency(dev(img[np.arange(B) % n]), dev(bank), 7, 0.5, wave=False, t_first=False,
                                        intensities=None)
    sync()
    I, rtf, rwave = orc.encode(img, bank, 7, 0.5)
    pick = torch.arange(B, device="cuda") % n
    assert torch.equal(lone, dev(I)[pick]), "intensities alone"
    assert torch.equal(inten, dev(I)[pick]), "intensities"
    assert torch.equal(tf, dev(rtf)[pick]), "t_first"
    assert torch.equal(wave, dev(rwave)[pick]), "wave"


def test_encode_more_tiles_than_a_launch_has_workgroups():
    # 2^24 tiles of 32x64: narrow images, which are filtered by bands then; 64 distinct ones, repeated
    B, n, H = (1 << 18) + 64, 64, 2048
    g = synth.rng(462, 0)
    img = g.integers(0, 256, (n, H, 1)).astype(np.uint8)
    bank = (g.integers(-64, 65, (1, 3, 3)) / 64.0).astype(np.float32)
    _, _, inten = spk.spk_encode_latency(dev(img).repeat(B // n, 1, 1), dev(bank), 5, wave=False, t_first=False,
                                         intensities=None)
    sync()
    I, _, _ = orc.encode(img, bank, 5, 0.0)
    assert torch.equal(inten, dev(I).repeat(B // n, 1, 1, 1)), "intensities"


@pytest.mark.parametrize("r,shape", [(0, (3, 6, 28, 28)), (2, (3, 6, 28, 28)), (8, (3, 6, 28, 28)),
                                     (30, (3, 6, 28, 28)), (8, (1, 2, 100, 250)), (3, (2, 1, 37, 5))])
def test_local_normalization_parity(r, shape):
    # (8, 100x250): rows split over several workgroups; general floats, so the fixed order decides
    g = synth.rng(900 + r + shape[2], 0)
    x = np.abs(g.normal(0, 40, shape)).astype(np.float32)
    x[:, :, :4] = 0.0
    out = spk.spk_local_normalization(dev(x), r, 1e-6)
    sync()
    assert_equal(host(out).view(np.uint32), orc.local_normalize(x, r, 1e-6).view(np.uint32), "normalised (bits)")


@pytest.mark.parametrize("shape,T", [((3, 6, 28, 28), 15), ((2, 4, 41, 50), 15), ((2, 2, 5, 7), 30)])
def test_rank_latency_parity(shape, T):
    g = synth.rng(950 + T + shape[1], 0)
    x = (g.integers(-20, 60, shape) * 0.5).astype(np.float32)  # ties and non-positive entries
    wave, tf = spk.spk_rank_latency(dev(x), T)
    sync()
    rtf = orc.rank_latency(x, T)
    assert_equal(host(tf), rtf, "t_first")
    assert_equal(host(wave), orc.expand_wave(rtf, T), "wave")


@pytest.mark.parametrize("run", [1, 383, 384, 385, 4096, 4097, 40000])
@pytest.mark.parametrize("spread", [0, 1, 300])
def test_rank_latency_ties_at_the_boundary(run, spread):
    # T = 4: two boundaries inside a run of entries that are equal, or of `spread` neighbouring floats
    # with the same second digit (bits 17..8), at random places; direct ranks up to 384 keys, then digit
    # passes without the digits that are the same everywhere, in LDS' reach up to 4096 and past it
    N = 4 * run + 8200
    g = synth.rng(958 + spread, run)
    x = np.empty(N, np.float32)
    lo = N // 4 - run // 4  # larger values before the run
    x[:lo] = 4.0 + g.random(lo, dtype=np.float32) * 100
    x[lo:lo + run] = (np.float32(1.5).view(np.uint32) + (g.integers(0, spread, run) % 256 if spread else 0)).astype(
        np.uint32).view(np.float32)
    x[lo + run:] = g.random(N - lo - run, dtype=np.float32) * np.float32(0.9)
    x = x[g.permutation(N)].reshape(1, 1, 1, N)
    _, tf = spk.spk_rank_latency(dev(x), 4, wave=False)
    sync()
    assert_equal(host(tf), orc.rank_latency(x, 4), "t_first")


def test_rank_latency_more_images_than_a_grid_side():
    # 65535 workgroups are a grid's second side: 66000 images of just more than 8192 entries, 40 of
    # them distinct
    B, n, T = 66000, 40, 5
    g = synth.rng(957, 0)
    x = g.normal(0, 40, (n, 1, 1, 8196)).astype(np.float32)
    rtf = orc.rank_latency(x, T)
    _, tf = spk.spk_rank_latency(dev(x).repeat(B // n, 1, 1, 1), T, wave=False)
    sync()
    assert torch.equal(tf, dev(rtf).repeat(B // n, 1, 1, 1)), "t_first"


# Maps of more than 8192 entries: many workgroups per image.  A first digit's segment is resolved
# in LDS up to 4096 keys and 384 with the boundaries' second digits, else by digit passes; the
# last entries of an image are no whole 16; up to 254 boundaries, in one digit or one per digit.
RANK_LARGE = [("floats", (2, 4, 60, 61), 30), ("floats", (1, 1, 97, 173), 255), ("flat", (2, 4, 60, 61), 30),
              ("flat", (1, 3, 53, 53), 255), ("few", (2, 4, 60, 61), 15), ("few", (1, 6, 91, 93), 255),
              ("narrow", (1, 2, 70, 90), 20), ("narrow", (1, 2, 70, 90), 255), ("sparse", (3, 2, 64, 65), 15),
              ("extreme", (2, 3, 55, 51), 64), ("floats", (1, 2, 64, 65), 2), ("floats", (2, 2, 64, 65), 1)]


def rank_map(kind, g, shape):
    if kind == "floats":
        return g.normal(0, 40, shape).astype(np.float32)
    if kind == "flat":  # one value: the index decides every rank
        return np.full(shape, 3.25, np.float32)
    if kind == "few":  # a handful of values, as a binarised image gives: long runs of ties
        return g.integers(-1, 4, shape).astype(np.float32)
    if kind == "narrow":  # one first digit, with equal second digits: 1 + m 2^-23, m < 4096
        return (1.0 + g.integers(0, 4096, shape) * 2.0 ** -23).astype(np.float32)
    if kind == "sparse":  # image 0 blank, image 1 with one positive entry, image 2 with 7
        x = -np.abs(g.normal(0, 1, shape)).astype(np.float32)
        x[1].reshape(-1)[-1] = 0.5
        x[2].reshape(-1)[11:18] = 2.0
        return x
    x = np.exp2(g.integers(-149, 128, shape).astype(np.float64)).astype(np.float32)  # subnormals to 2^127
    x.reshape(-1)[::97] = np.inf
    x.reshape(-1)[::89] = -np.inf
    return x


@pytest.mark.parametrize("kind,shape,T", RANK_LARGE)
def test_rank_latency_large_maps(kind, shape, T):
    x = rank_map(kind, synth.rng(970 + T, 0), shape)
    wave, tf = spk.spk_rank_latency(dev(x), T)
    sync()
    rtf = orc.rank_latency(x, T)
    assert_equal(host(tf), rtf, "t_first")
    assert_equal(host(wave), orc.expand_wave(rtf, T), "wave")
    # written through addresses of any alignment
    N = x[0].size
    sx, stf = dev_shifted(x), dev_shifted(np.zeros(x.shape, np.uint8), 3)
    swv = dev_shifted(np.zeros((x.shape[0], T) + x.shape[1:], np.uint8), 1)
    spk.spk_rank_latency(sx, T, wave=swv, t_first=stf)
    sync()
    assert N > 8192
    assert_equal(host(stf), rtf, "t_first, unaligned")
    assert_equal(host(swv), orc.expand_wave(rtf, T), "wave, unaligned")


# Larger maps' filter by tiles of 32x64: ragged tiles, an unaligned width, the double form, banks
# whose digits are counted in a pass of their own (33 channels) or filtered by bands (65 channels)
@pytest.mark.parametrize("C,KF,H,W,form", [(6, 13, 33, 65, "int"), (5, 7, 47, 129, "float"), (33, 3, 19, 64, "int"),
                                           (65, 3, 19, 30, "int"), (4, 31, 70, 71, "float"), (2, 1, 64, 70, "int")])
def test_encode_large_maps(C, KF, H, W, form):
    g = synth.rng(480 + C, KF)
    img = synth.pink_noise_images(g, 2, H, W)
    if form == "int":
        bank = (g.integers(-64, 65, (C, KF, KF)) / 64.0).astype(np.float32)
        bank[C - 1] = -bank[C - 2]  # a derived channel
    else:
        bank = (g.normal(0, 1, (C, KF, KF)) * np.exp2(g.integers(-20, 3, (C, KF, KF)))).astype(np.float32)
    wave, tf, inten = spk.spk_encode_latency(dev(img), dev(bank), 15, 0.5, intensities=None)
    only = spk.spk_encode_latency(dev(img), dev(bank), 15, 0.5, wave=False, t_first=False, intensities=None)[2]
    sync()
    I, rtf, rwave = orc.encode(img, bank, 15, 0.5)
    assert_equal(host(inten), I, "intensities")
    assert_equal(host(only), I, "intensities alone")
    assert_equal(host(tf), rtf, "t_first")
    assert_equal(host(wave), rwave, "wave")


def test_chain_encode_with_local_normalization():
    # filter -> local normalisation (radius 8, the tutorial's) -> rank-order code, against the oracle's steps
    from paper_1903_02440_amd.pipeline import chain_for
    wl = synth.mnist_single(4)
    inp = synth.make_inputs(wl)
    ch = chain_for(wl, inp["bank"], local_norm=(8, 1e-12))
    ch.set_weights([torch.from_numpy(w) for w in inp["weights"]])
    ch.set_input(image=torch.from_numpy(inp["image"]))
    ch.forward()
    sync()
    I = orc.filter_images(inp["image"], inp["bank"], 0.0)
    rtf = orc.rank_latency(orc.local_normalize(I, 8, 1e-12), wl.T)
    assert_equal(host(ch.input_tf), rtf, "t_first")
    assert_equal(host(ch.input_wave), orc.expand_wave(rtf, wl.T), "wave")


def test_encode_blank_image_never_spikes():
    img = np.zeros((2, 28, 28), np.uint8)
    wave, tf, _ = spk.spk_encode_latency(dev(img), dev(synth.dog_bank()), 15)
    sync()
    assert (host(tf) == 15).all() and not host(wave).any()


def test_expand_and_validate():
    g = synth.rng(9, 0)
    tf = synth.times_uniform_or_silent(g, (3, 5, 7, 9), 11, 0.3)
    wave = spk.spk_expand_wave(dev(tf), 11)
    bad = spk.spk_validate_wave(wave)
    sync()
    assert_equal(host(wave), orc.expand_wave(tf, 11), "expand")
    assert bad.item() == 0
    w2 = host(wave).copy()
    w2[0, 10, 0, 0, 0] = 0 if w2[0, 9, 0, 0, 0] else w2[0, 10, 0, 0, 0]
    w2[1, 0, 1, 1, 1] = 3
    bad = spk.spk_validate_wave(dev(w2))
    sync()
    assert bad.item() == orc.count_invalid(w2)


# ---------------------------------------------------------------- plasticity
def layer_case(seed, B, T, Cin, H, W, Cout, K, pad, thr, k, r):
    g = synth.rng(500 + seed, 0)
    wave = wave_of(synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5), T)
    Wt = synth.normal_weights(g, (Cout, Cin, K, K), 0.8, 0.05)
    _, _, tf, vf = orc.conv_fire(wave, Wt, pad, thr)
    win, nw = orc.kwta(tf, vf, T, k, r)
    return wave, Wt, win, nw


STDP_CASES = [(1, 8, 15, 6, 28, 28, 30, 5, 2, 15.0, 5, 3), (2, 4, 15, 30, 14, 14, 250, 3, 1, 10.0, 8, 1),
              (3, 6, 15, 250, 4, 4, 200, 5, 2, math.inf, 1, 0)]


@pytest.mark.parametrize("case", STDP_CASES)
def test_stdp_parity(case):
    wave, Wt, win, nw = layer_case(*case)
    pad = case[8]
    Wg = dev(Wt)
    spk.spk_stdp(Wg, pad, dev(wave), dev(win), dev(nw), 0.004, -0.003)
    sync()
    assert_equal(host(Wg), orc.stdp(Wt, wave, pad, win, nw, 0.004, -0.003), "weights")


@pytest.mark.parametrize("case", STDP_CASES)
@pytest.mark.parametrize("images", ["batch", "one"])
def test_stdp_first_spike_input(case, images):
    # the layer input given by its first-spike map: the same updates as Eq.4 on its wave
    wave, Wt, win, nw = layer_case(*case)
    if images == "one":
        wave, win, nw = wave[:1], win[:1], nw[:1]
    T, pad = wave.shape[1], case[8]
    tf = orc.first_spike(wave)
    Wg = dev(Wt)
    spk.spk_stdp_first_spike(Wg, pad, dev(tf), T, dev(win), dev(nw), 0.004, -0.003)
    torch.cuda.synchronize()
    assert_equal(host(Wg), orc.stdp(Wt, wave, pad, win, nw, 0.004, -0.003), "STDP weights")
    reward = synth.rng(560, 0).choice(np.array([1, -1, 0], np.int8), wave.shape[0])
    Wg = dev(Wt)
    spk.spk_rstdp_first_spike(Wg, pad, dev(tf), T, dev(win), dev(nw), dev(reward), 0.004, -0.003)
    torch.cuda.synchronize()
    assert_equal(host(Wg), orc.stdp(Wt, wave, pad, win, nw, 0.004, -0.003, reward=reward), "R-STDP weights")


@pytest.mark.parametrize("case", STDP_CASES)
@pytest.mark.parametrize("rew", [None, 1, -1, 0])
def test_stdp_single_image(case, rew):
    # one image (the online step's direct update): oracle parity for STDP and R-STDP
    wave, Wt, win, nw = layer_case(*case)
    wave, win, nw = wave[:1], win[:1], nw[:1]
    pad = case[8]
    Wg = dev(Wt)
    if rew is None:
        spk.spk_stdp(Wg, pad, dev(wave), dev(win), dev(nw), 0.004, -0.003)
        ref = orc.stdp(Wt, wave, pad, win, nw, 0.004, -0.003)
    else:
        reward = np.array([rew], np.int8)
        spk.spk_rstdp(Wg, pad, dev(wave), dev(win), dev(nw), dev(reward), 0.004, -0.003)
        ref = orc.stdp(Wt, wave, pad, win, nw, 0.004, -0.003, reward=reward)
    sync()
    assert_equal(host(Wg), ref, "weights")


def test_stdp_single_image_odd_records_match_replay():
    # records the replay skips (a repeated feature, a step outside [0, T), a feature
    # out of range): the one-image path applies the same updates as the batched
    # replay of a two-image batch whose second image has no winners
    wave, Wt, win, nw = layer_case(*STDP_CASES[0])
    T, pad, k = wave.shape[1], 2, win.shape[1]
    w1 = win[:1].copy()
    w1[0, 1] = w1[0, 0]                    # the first record's feature again, other step and place
    w1[0, 1, 1] = (w1[0, 0, 1] + 3) % T
    w1[0, 1, 2:] = (5, 7)
    w1[0, 2, 1] = T                        # a step outside [0, T)
    w1[0, 3, 0] = 999                      # a feature out of range
    n1 = np.array([k], np.int32)
    wave2 = np.concatenate([wave[:1], wave[1:2]])
    win2 = np.concatenate([w1, np.full_like(w1, -1)])
    n2 = np.array([k, 0], np.int32)
    for rates in [(0.004, -0.003), (0.6, -0.5)]:
        Wa, Wb = dev(Wt), dev(Wt)
        spk.spk_stdp(Wa, pad, dev(wave[:1]), dev(w1), dev(n1), *rates)
        spk.spk_stdp(Wb, pad, dev(wave2), dev(win2), dev(n2), *rates)
        sync()
        assert_equal(host(Wa), host(Wb), f"one image vs replay, rates {rates}")


def test_rstdp_and_bounds_variant():
    wave, Wt, win, nw = layer_case(*STDP_CASES[2])
    B = wave.shape[0]
    reward = np.array([1, -1, 0, -1, 1, 1], np.int8)[:B]
    Wg = dev(Wt)
    spk.spk_rstdp(Wg, 2, dev(wave), dev(win), dev(nw), dev(reward), 0.004, -0.003)
    sync()
    assert_equal(host(Wg), orc.stdp(Wt, wave, 2, win, nw, 0.004, -0.003, reward=reward), "R-STDP")
    # stabilizer off, bounds [0.2, 0.8] (the tutorial's variant for its last layer)
    Wg = dev(Wt)
    spk.spk_rstdp(Wg, 2, dev(wave), dev(win), dev(nw), dev(reward), 0.05, -0.04, 0.2, 0.8, stabilizer=False)
    sync()
    ref = orc.stdp(Wt, wave, 2, win, nw, 0.05, -0.04, 0.2, 0.8, stabilizer=False, reward=reward)
    assert_equal(host(Wg), ref, "R-STDP clamp")


@pytest.mark.parametrize("rates", [(0.004, -0.003), (0.7, -0.6)])
def test_stdp_weights_outside_bounds(rates):
    # the first update of a chain starts from a weight outside [lb, ub]; with small
    # rates the later updates skip the clamp, with large ones they keep it
    wave, Wt, win, nw = layer_case(*STDP_CASES[0])
    Wt = Wt.copy()
    g = synth.rng(650, 0)
    flat = Wt.reshape(-1)
    idx = g.choice(flat.size, flat.size // 4, replace=False)
    flat[idx] = g.choice(np.array([-0.25, 1.5, 0.0, 1.0, -0.0], np.float32), idx.size)
    Wg = dev(Wt)
    spk.spk_stdp(Wg, 2, dev(wave), dev(win), dev(nw), *rates)
    sync()
    assert_equal(host(Wg), orc.stdp(Wt, wave, 2, win, nw, *rates), "weights")


def test_stdp_ordered_replay_many_images():
    # more images than one scan chunk, features winning repeatedly: order matters
    g = synth.rng(600, 0)
    B, T, Cin, H, W, Cout, K, pad, k = 2500, 5, 2, 6, 6, 4, 3, 1, 2
    wave = wave_of(synth.times_uniform_or_silent(g, (B, Cin, H, W), T, 0.5), T)
    Wt = synth.normal_weights(g, (Cout, Cin, K, K), 0.5, 0.2)
    win = np.full((B, k, 4), -1, np.int32)
    nw = g.integers(0, k + 1, B).astype(np.int32)
    for b in range(B):
        fs = g.choice(Cout, size=nw[b], replace=False)
        for j, f in enumerate(fs):
            win[b, j] = (f, g.integers(0, T), g.integers(0, H), g.integers(0, W))
    Wg = dev(Wt)
    spk.spk_stdp(Wg, pad, dev(wave), dev(win), dev(nw), 0.02, -0.015)
    sync()
    assert_equal(host(Wg), orc.stdp(Wt, wave, pad, win, nw, 0.02, -0.015), "weights")


def test_decide_parity():
    g = synth.rng(700, 0)
    B, k = 1500, 1
    win = np.full((B, k, 4), -1, np.int32)
    nw = (g.random(B) < 0.9).astype(np.int32)
    win[nw == 1, 0, 0] = g.integers(0, 200, (nw == 1).sum())
    labels = synth.labels(g, B)
    dec, rew = spk.spk_decide(dev(win), dev(nw), dev(labels), 10)
    sync()
    rd, rr = orc.decide(win, nw, labels, 10)
    assert_equal(host(dec), rd, "decision")
    assert_equal(host(rew), rr, "reward")
