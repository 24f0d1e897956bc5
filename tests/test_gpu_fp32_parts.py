"""GPU: the fp32 path's arithmetic on three bf16 parts per operand and six of the
nine partial products (conv_fc1_f32.hip): every product to fp32's precision."""

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
