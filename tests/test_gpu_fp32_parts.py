"""GPU: the fp32 path's arithmetic on three bf16 parts per operand and six of the
nine partial products (conv_fc1_f32.hip): every product to fp32's precision, and
what parts cannot hold (infinities, NaNs, values near the end of the range)
as fp32 arithmetic gives it."""

import sys

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

F = np.float32
POS, CH = 44 * 44, 48


def say(*a):
    print(*a, flush=True, file=sys.stderr)


@pytest.fixture(scope="module")
def pid():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_04509_amd import binding
    return binding


def classify(pid, w, P):
    h = pid.pointid_create(w, "fp32", 0)
    got = pid.pointid_classify_patches(h, torch.from_numpy(np.ascontiguousarray(P, F)).cuda()).cpu().numpy()
    h.close()
    return got


def network(w, P):
    """Scores in 64 bits; conv maps and FC1 sums past fp32's range are infinite.  A
    pair of positions x, x + 1 shares a window of six columns: the column that
    a position does not use meets a tap of 0, which an infinite or NaN pixel
    makes NaN.  NaN maps and sums are 0 behind a ReLU."""
    w = {k: np.asarray(v, np.float64) for k, v in w.items()}
    X = P.astype(np.float64)
    with np.errstate(all="ignore"):
        cols = np.stack([X[:, u:u + 44, v:v + 44] for u in range(5) for v in range(5)], -1)
        maps = (cols[..., None, :] * w["conv_w"].reshape(48, 25)).sum(-1) + w["conv_b"]
        bad = ~np.isfinite(X)
        rows = np.stack([bad[:, u:u + 44] for u in range(5)]).any(0)          # [n][44][48]
        maps[:, :, 0::2][rows[:, :, 5::2]] = np.nan
        maps[:, :, 1::2][rows[:, :, 0:44:2]] = np.nan
        maps = np.fmax(maps.astype(F).astype(np.float64), 0)
        h1 = (maps.reshape(len(X), -1) @ w["fc1_w"]).astype(F).astype(np.float64) + w["fc1_b"]
        h2 = np.fmax(np.fmax(h1, 0) @ w["fc2_w"] + w["fc2_b"], 0)
        z = h2 @ w["cls_w"] + w["cls_b"].reshape(-1)
        q = h2 @ w["mic_w"].reshape(32, 1) + w["mic_b"].reshape(-1)
        e = np.exp(z - np.fmax(np.fmax(z[:, :1], z[:, 1:2]), z[:, 2:]))
        s = np.exp(-np.abs(q))
        return np.concatenate([e / e.sum(1, keepdims=True), np.where(q >= 0, 1 / (1 + s), s / (1 + s))], 1)


def test_scores_to_single_precision(pid):
    """Without any one of the six products the scores of these patches are off by
    1e-5 or more (1.2e-5 without one that takes a low part); with all of them by
    about 1e-7, the sums' rounding."""
    w = synth.he_normal_weights()
    P = synth.config4_patches(40, seed=7)
    err = np.abs(classify(pid, w, P) - network(w, P)).max()
    say(f"max |d score| {err:.2e}")
    assert err <= 2e-6


@pytest.mark.parametrize("kind", ["any", "parts"])
def test_single_products(pid, kind):
    """Networks in which a score rests on one conv product and one FC1 product: each
    of 128 outputs reads one map value behind one filter tap, its bias takes all
    but 2^-13 of the sum away (an exact subtraction) and FC2 multiplies the rest
    by 2^15, so that the score shows the sum to far below its last bit.

    Bounds, in units of 2^-24 of the sum.  A product leaves out 2^-24.2 = 0.87 at
    most; adding its largest part last loses one unit in the last place, 2 units,
    also where the MFMA cuts; the other additions are 2^-8 of that; the map is
    taken apart exactly: 2 x 2.9 for both products.  "parts": pixels just below
    1 + 2^-7 times 1 + 2^-8, FC1 weights powers of two.  Of the pixel's parts
    rounded to nearest nothing is left out and the FC1 product is exact: 2 units
    and, also where the MFMA cuts, 1 on average, 0.05 for the score's own rounding
    (of parts cut off, up to 2^-23 more: -1.21 on average)."""
    rng = np.random.default_rng(5)
    f = np.zeros
    n = 32
    a = (1 + rng.random(CH)).astype(F)
    wt = (0.5 + 0.5 * rng.random(128)).astype(F)
    x0 = (1 + rng.random(128)).astype(F)
    x = (x0[:, None] * (1 + 2.0**-13 * rng.random((128, n)))).astype(F)
    if kind == "parts":
        a[:] = 1 + 2.0**-8
        wt = 2.0 ** rng.integers(-3, 3, 128).astype(F)
        x = (1 + 2.0**-7 - 2.0**-23 * rng.integers(1, 200, (128, n))).astype(F)
        x0 = x.min(1)
    pos, ch = rng.choice(POS, 128, replace=False), rng.integers(0, CH, 128)
    s0 = x0.astype(np.float64) * a[ch] * wt
    w = {"conv_w": f((CH, 5, 5), F), "conv_b": f(CH, F), "fc1_w": f((POS * CH, 128), F),
         "fc1_b": (-s0 * (1 - 2.0**-14)).astype(F), "fc2_w": f((128, 32), F), "fc2_b": f(32, F),
         "cls_w": f((32, 3), F), "cls_b": f(3, F), "mic_w": f((32, 1), F), "mic_b": np.full(1, -4, F)}
    w["conv_w"][:, 2, 2] = a
    w["fc1_w"][pos * CH + ch, np.arange(128)] = wt
    gain = 2.0 ** (15 - np.floor(np.log2(s0)))           # exact in fp32
    w["fc2_w"][:, 0] = gain
    w["mic_w"][0] = 1
    P = f((128, n, 48, 48), F)
    P[np.arange(128)[:, None], np.arange(n), (pos // 44 + 2)[:, None], (pos % 44 + 2)[:, None]] = x
    got = classify(pid, w, P.reshape(-1, 48, 48))[:, 3].astype(np.float64).reshape(128, n)
    s = x.astype(np.float64) * a[ch][:, None] * wt[:, None]
    q = np.log(got / (1 - got))
    e = ((q + 4) / gain[:, None] - w["fc1_b"].astype(np.float64)[:, None] - s) / s * 2.0**24
    say(f"{kind}: max {np.abs(e).max():.2f} rms {np.sqrt((e * e).mean()):.2f} mean {e.mean():.2f} x 2^-24")
    assert np.abs(e).max() <= (5.8 if kind == "any" else 2.05)
    assert kind == "any" or abs(e.mean()) <= 1.05


def one_signed(w, sign):
    return {**w, "fc1_w": sign * np.abs(w["fc1_w"])}


@pytest.mark.parametrize("n", [3, 300, 600, 1100])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, -3.0e38, 1e37])
def test_pixels_out_of_range(pid, value, n):
    """A few patches with an infinite, NaN or huge pixel, in every shape of block;
    FC1 weights of one sign make infinite sums of either sign, of both signs NaN
    ones (0 behind the ReLU).  The other patches keep their bits."""
    base = synth.he_normal_weights()
    P = synth.config4_patches(n, seed=n).astype(F)
    clean = P.copy()
    rng = np.random.default_rng(n)
    at = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 6)]))
    for i in at:
        P[i, rng.integers(0, 48), rng.integers(0, 48)] = value
    P[at[0], 0, 0], P[at[1], 47, 47] = value, value      # pixels of one position, and of the last range
    nets = {"both": base, "plus": one_signed(base, 1), "minus": one_signed(base, -1),
            "small": {**base, "fc1_w": base["fc1_w"] * F(2.0**-100)}}
    if np.isfinite(value):      # (with the others FC2's sums would pass the range in one order and not in another)
        nets = {"small": nets["small"]}
    for name, w in nets.items():
        say(f"{value} {n} {name}")
        got = classify(pid, w, P)
        want = network(w, P[at])
        assert np.array_equal(np.isnan(got[at]), np.isnan(want)), name
        assert np.nanmax(np.abs(got[at] - want), initial=0) <= 1e-4, name
        rest = np.setdiff1d(np.arange(n), at)
        assert np.array_equal(got[rest].view(np.uint32), classify(pid, w, clean)[rest].view(np.uint32)), name


@pytest.mark.parametrize("where, value", [("conv_w", np.inf), ("conv_w", np.nan), ("conv_b", -np.inf), ("conv_b", np.inf),
                                          ("conv_w", 3.4e38), ("fc1_w", np.inf), ("fc1_w", -np.inf), ("fc1_w", np.nan),
                                          ("fc1_w", 3.4e38)])
def test_weights_out_of_range(pid, where, value):
    """One weight past the range, all patches computed in plain fp32."""
    base = {k: np.array(v) for k, v in synth.he_normal_weights().items()}
    P = np.abs(synth.config4_patches(20, seed=3)).astype(F) + F(0.1)
    for w in (base, one_signed(base, 1)):
        w = {k: np.array(v) for k, v in w.items()}
        v = w[where].reshape(-1)
        v[len(v) // 2] = value
        got, want = classify(pid, w, P), network(w, P)
        say(where, value, want[0])
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.nanmax(np.abs(got - want), initial=0) <= 1e-4


def test_overflown_sums_in_every_block_shape(pid):
    """FC1 sums of two outputs overflow to minus infinity (0 behind the ReLU): the
    others keep their bits, whichever outputs share a block."""
    w = {k: np.array(v) for k, v in synth.he_normal_weights().items()}
    w["fc1_w"][5000::9000, 5] = -3.0e38
    w["fc1_w"][100::9000, 90] = -3.0e38
    P = (synth.config4_patches(1100, seed=4) * 20).astype(F)
    full = classify(pid, w, P)
    want = network(w, P[:20])
    assert np.isfinite(full).all() and np.abs(full[:20] - want).max() <= 1e-4
    for n in (1, 20, 200, 400, 700):
        assert np.array_equal(classify(pid, w, P[:n]).view(np.uint32), full[:n].view(np.uint32)), n


@pytest.mark.parametrize("value", [3.0e38, 1e30, 1e-30, 2.0**-100])
def test_scale_of_one_pixel(pid, value):
    """Patches of one pixel each, filters scaled to it: the scores rest on the pixel's parts alone."""
    w = {k: np.array(v) for k, v in synth.he_normal_weights().items()}
    rng = np.random.default_rng(2)
    P = np.zeros((40, 48, 48), F)
    for i in range(40):
        P[i, rng.integers(0, 48), rng.integers(0, 48)] = value * (0.5 + 0.5 * rng.random()) * rng.choice([-1, 1])
    w["conv_w"] = (w["conv_w"] / value * 100).astype(F)
    got, want = classify(pid, w, P), network(w, P)
    assert np.abs(want - want[0]).max() > 1e-2           # the pixel is what tells them apart
    assert np.abs(got - want).max() <= 2e-6 * 100
