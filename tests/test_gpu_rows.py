"""GPU: the fused kernels' sources of patch rows and their block shapes.

Batches of up to one round of blocks (and every batch of the fp32 path) read the rows of their hits
from the plane images themselves: hits must get exactly the bits that the
oracle's patches of the same hits get as pre-cut patches, at every edge of the
planes, at any image alignment and row pitch, for one array of hits, requests,
and tick columns.  Large batches run blocks of several position ranges: every
patch must get the bits it gets in a small batch.
"""

import sys

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PRECS = ["fp32", "bf16", "fp16", "fp8"]


def say(*a):
    print(*a, flush=True, file=sys.stderr)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def bits(x):
    return x.cpu().numpy().view(np.uint32)


@pytest.fixture(scope="module")
def pid():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_04509_amd import binding
    return binding


@pytest.fixture(scope="module")
def handles(pid):
    w = synth.he_normal_weights()
    return {p: pid.pointid_create(w, p, 0) for p in PRECS}


def edge_hits(rng, planes, n):
    """n hits around every edge of the planes, some far outside, some on planes
    that do not exist."""
    p = rng.integers(0, len(planes), n)
    W = np.array([im.shape[0] for im in planes])[p]
    T = np.array([im.shape[1] for im in planes])[p]
    w = np.where(rng.random(n) < 0.5, rng.integers(-30, 30, n), W - rng.integers(-30, 30, n))
    k = np.where(rng.random(n) < 0.5, rng.integers(-30, 30, n), T - rng.integers(-30, 30, n))
    mid = rng.random(n) < 0.3
    k = np.where(mid, rng.integers(0, T), k)
    h = np.stack([p, w, k], 1)
    h[::41, 0] = len(planes)
    h[5::43, 0] = -1
    h[7::47, 1:] = [2**31 - 1, -2**31]
    return h.astype(np.int32)


@pytest.mark.parametrize("prec", PRECS)
def test_hits_get_the_bits_of_their_patches(pid, handles, prec):
    h = handles[prec]
    rng = np.random.default_rng(91)
    dims = [(60, 100), (37, 101), (90, 47), (3, 5), (50, 130)]
    imgs, dev = [], []
    for k, (W, T) in enumerate(dims):
        im = rng.normal(0, 4, (W, T)).astype(np.float32)
        buf = t(np.concatenate([np.zeros(k % 4, np.float32), im.ravel()]))
        imgs.append(im)
        dev.append(buf[k % 4:].view(W, T))               # base 0, 4, 8 or 12 bytes past 16
    for n in (1, 16, 17, 129, 300, 513, 1024, 1025, 1500, 2048, 2049, 3072, 3073):
        hh = edge_hits(rng, imgs, n)
        say(f"{prec} {n} hits at the edges")
        want = bits(pid.pointid_classify_patches(h, t(oracle.gather_patches_planes(imgs, hh))))
        assert np.array_equal(bits(pid.pointid_classify_planes(h, dev, t(hh))), want), n
        if n > 2:                                        # the same as three requests
            cut = [0, n // 3, n // 3 + 1, n]
            got = pid.pointid_classify_requests(
                h, dev, [(-1, t(hh[a:b]), None) for a, b in zip(cut, cut[1:])])
            assert np.array_equal(np.concatenate([bits(x) for x in got]), want), n
    D = 3
    hh = edge_hits(rng, imgs, 200)
    binned = [oracle.downsample_plane(im, D).astype(np.float32) for im in imgs]
    hb = hh.astype(np.int64)
    hb[:, 2] = np.floor_divide(hb[:, 2], D)
    want = bits(pid.pointid_classify_patches(h, t(oracle.gather_patches_planes(binned, hb.astype(np.int32)))))
    assert np.array_equal(bits(pid.pointid_classify_planes_ds(h, dev, t(hh), D)), want)


@pytest.mark.parametrize("prec", PRECS)
def test_large_batches_give_the_bits_of_small_ones(pid, handles, prec):
    """On a 256-CU device the 16-bit path runs 20,641 patches in blocks of four,
    two and one ranges of 96 patches and of 64, 7,000 in blocks of two and one,
    5,100 and 3,973 in blocks of two ranges of 64; the fp32 path runs batches
    past 512 in tiles of 64 and 32 and smaller ones in tiles of 32 and 16 whose
    outputs are shared out over 2 or 4 blocks."""
    h = handles[prec]
    P = t(synth.config4_patches(20641, seed=5))
    full = bits(pid.pointid_classify_patches(h, P))
    for lo, hi in [(0, 300), (3000, 3900), (9000, 10024), (12277, 12300), (18400, 18450),
                   (20000, 20641), (13000, 20000), (100, 5200), (16668, 20641), (500, 1900)]:
        say(f"{prec} patches {lo}:{hi}")
        assert np.array_equal(bits(pid.pointid_classify_patches(h, P[lo:hi].contiguous())), full[lo:hi]), (lo, hi)


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_gathered_batches_give_the_bits_of_small_ones(pid, handles, prec):
    """Hits past one round of 64-patch tiles come as 16-bit patches from the gather.
    On a 256-CU device the sizes are on both sides of every change of the blocks: 96-patch
    tiles (one range; from 6,144 hits two, from 12,288 four), 64-patch ones
    (one range, two from two rounds on: 3,073 to 4,096 hits, or behind 96-patch
    tiles), odd numbers of tiles in every kind."""
    h = handles[prec]
    rng = np.random.default_rng(17)
    imgs = [rng.normal(0, 4, (W, T)).astype(np.float32) for W, T in [(200, 700), (90, 333), (37, 101)]]
    dev = [t(im) for im in imgs]
    n_all = 21000
    p = rng.integers(0, 3, n_all)
    hh = np.stack([p, rng.integers(0, np.array([200, 90, 37])[p]),
                   rng.integers(0, np.array([700, 333, 101])[p])], 1).astype(np.int32)
    d = t(hh)
    want = np.concatenate([bits(pid.pointid_classify_planes(h, dev, d[a:a + 1000].contiguous()))
                           for a in range(0, n_all, 1000)])
    for n in (2049, 3072, 3073, 3137, 4095, 4096, 4097, 5121, 6143, 6145, 7000, 8193, 9217, 12287, 12289,
              13000, 15361, 16384, 18433, 20641, 21000):
        say(f"{prec} {n} gathered hits")
        assert np.array_equal(bits(pid.pointid_classify_planes(h, dev, d[:n].contiguous())), want[:n]), n


@pytest.mark.parametrize("prec", ["fp32", "fp8"])
def test_block_shapes_at_their_edges(pid, handles, prec):
    """Batches on both sides of every change of a block shape on a 256-CU device
    give one set of bits.  fp32: 16 patches, a quarter of the outputs up to 128; 32
    patches, a quarter up to 256, half up to 512, all up to 1,024; then 64.  fp8: 16
    patches, a quarter of the outputs up to 128, half up to 256, all up to 512; 32
    patches up to 1,024; then 64."""
    h = handles[prec]
    P = t(synth.config4_patches(4200, seed=6))
    full = bits(pid.pointid_classify_patches(h, P))
    for n in (1, 15, 16, 17, 127, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 3072, 3073, 4096, 4097):
        say(f"{prec} {n} patches")
        for lo in (0, 4200 - n):
            got = bits(pid.pointid_classify_patches(h, P[lo:lo + n].contiguous()))
            assert np.array_equal(got, full[lo:lo + n]), (n, lo)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.0e38, 1e-30])
def test_fp32_extreme_pixels(pid, handles, value):
    """One extreme pixel in every other patch: an infinite one makes every FC1 sum NaN
    (weights of both signs), which the ReLU takes to 0 as it takes a NaN map value
    to 0, so that these patches all have the scores of the biases; a finite one
    leaves the other patches as they are.  Against the network in 64 bits, the
    tolerance that of the other fp32 tests."""
    h = handles["fp32"]
    w = {k: np.asarray(v, np.float64) for k, v in synth.he_normal_weights().items()}
    P = synth.config4_patches(40, seed=7).astype(np.float32)
    rng = np.random.default_rng(3)
    for i in range(1, 40, 2):                            # every other patch keeps its own pixels
        P[i, rng.integers(0, 48), rng.integers(0, 48)] = value
    got = pid.pointid_classify_patches(h, t(P)).cpu().numpy()
    X = P.astype(np.float64)
    with np.errstate(all="ignore"):
        cols = np.stack([X[:, u:u + 44, v:v + 44] for u in range(5) for v in range(5)], -1)
        maps = np.fmax(cols @ w["conv_w"].reshape(48, 25).T + w["conv_b"], 0)
        # (a pair of positions x, x + 1 shares a window of six columns, whose sixth
        # pixel meets a tap of 0: 0 times NaN takes the other position with it)
        pair = np.isnan(cols).any(-1).reshape(40, 44, 22, 2).any(-1).repeat(2, -1)
        maps[pair] = 0
        h1 = np.fmax(maps.reshape(40, -1) @ w["fc1_w"] + w["fc1_b"], 0)
    if not np.isfinite(value):
        assert np.isfinite(h1).all()
    if np.isinf(value):
        assert (h1[1::2] == 0).all()
        assert np.array_equal(got[1::2].view(np.uint32), np.repeat(got[1:2], 20, 0).view(np.uint32))
    if value == 3.0e38:                                  # past fp32's range further on: only the others
        got, h1 = got[::2], h1[::2]
    h2 = np.maximum(h1 @ w["fc2_w"] + w["fc2_b"], 0)
    z = h2 @ w["cls_w"] + w["cls_b"].reshape(-1)
    e = np.exp(z - z.max(1, keepdims=True))
    q = h2 @ w["mic_w"].reshape(32, 1) + w["mic_b"].reshape(-1)
    want = np.concatenate([e / e.sum(1, keepdims=True), 1 / (1 + np.exp(-q))], 1)
    assert np.abs(got - want).max() <= 1e-4
