"""Performance cases of the classifier: what a reconstruction job or an inference
server asks of it, through the public entry points.

A case is one call (``call``) on inputs like those of ProtoDUNE-SP: planes of
deconvolved charge (Gaussian noise of 2.5 ADC, straight tracks, showers) with
hits at the signal peaks, or pre-cut patches (N(0, 1) and one line each), and
He-normal weights.  Calls:

``classify``   hits (wire, tick) on one plane
``planes``     hits (plane, wire, tick) over an event's planes
``patches``    pre-cut fp32 patches, as an inference server receives them
``requests``   many clients' requests merged into one batch
``ds``         hits on planes binned into columns of ``ticks_per_column`` ticks
``find_hits``  hit finding on an event's planes
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2009_04509_amd import binding as pid

PATCH = 48
FMAP = 44
FC1_IN = FMAP * FMAP * 48
FC1_OUT = 128
# multiply-adds of one patch: conv, FC1, FC2, heads
FLOPS = 2 * (FMAP * FMAP * 48 * 25 + FC1_IN * FC1_OUT + FC1_OUT * 32 + 32 * 4)
WEIGHT_VALUES = 48 * 25 + 48 + FC1_IN * FC1_OUT + FC1_OUT + FC1_OUT * 32 + 32 + 32 * 4 + 4
WEIGHT_BYTES = {"fp32": 4, "bf16": 2, "fp16": 2, "fp8": 1}
NOISE = 2.5


def _case(name, call, precision="fp16", planes=0, wires=0, ticks=0, n=0, requests=0,
          ticks_per_column=1, threshold=0.0):
    return {"name": name, "call": call, "precision": precision, "planes": planes, "wires": wires,
            "ticks": ticks, "n": n, "requests": requests, "ticks_per_column": ticks_per_column,
            "threshold": threshold}


def listed():
    return [
        # a small detector region, the least that is sent for classification
        _case("tiny_fp16", "classify", "fp16", 1, 128, 512, 128),
        # one client's small request against a resident collection plane, 8-bit operation
        _case("request_235_fp8", "classify", "fp8", 1, 480, 6000, 235),
        # the small batch of an inference client that sends ready patches, single precision
        _case("patches_235_fp32", "patches", "fp32", n=235),
        # all hits of one collection plane
        _case("plane_fp16", "classify", "fp16", 1, 480, 6000, 3000),
        # a whole event (18 planes) in one call: the job's main use, at each arithmetic
        _case("event_fp16", "planes", "fp16", 18, 800, 6000, 50000),
        _case("event_fp32", "planes", "fp32", 18, 800, 6000, 50000),
        _case("event_fp8", "planes", "fp8", 18, 800, 6000, 50000),
        # the large batch of such a client
        _case("patches_1693_bf16", "patches", "bf16", n=1693),
        # a throughput server's full batch
        _case("patches_16384_bf16", "patches", "bf16", n=16384),
        # a batching server's turn: 64 clients' small requests on 8 resident planes
        _case("requests_64x235_fp16", "requests", "fp16", 8, 480, 6000, 235, requests=64),
        # the step before the classification, on the event's planes
        _case("find_hits_event", "find_hits", "fp16", 18, 800, 6000, threshold=10.0),
        # the event with four ticks to a patch column
        _case("event_ds4_fp16", "ds", "fp16", 18, 800, 6000, 50000, ticks_per_column=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["classify", "planes", "patches", "requests", "ds", "find_hits"])
    precision = rng.choice(["fp16", "fp16", "bf16", "fp8", "fp32"])
    planes = 1 if call == "classify" else rng.randint(2, 18)
    wires = _log_int(rng, 48, 800)
    ticks = _log_int(rng, 300, 6000)
    most = 12000 if precision == "fp32" else 40000
    n = _log_int(rng, 1, most)
    if call == "patches":
        case = _case("", call, precision, n=_log_int(rng, 1, min(most, 20000)))
    elif call == "requests":
        case = _case("", call, precision, planes, wires, ticks, _log_int(rng, 1, most // 80),
                     requests=rng.randint(2, 70))
    elif call == "find_hits":
        case = _case("", call, "fp16", planes, wires, ticks, threshold=rng.choice([5.0, 10.0, 40.0]))
    elif call == "ds":
        case = _case("", call, precision, planes, wires, ticks, n, ticks_per_column=rng.randint(2, 8))
    else:
        case = _case("", call, precision, planes, wires, ticks, n)
    del case["name"]
    return case


# ---- inputs

def _wires(case):
    """Wires of each plane: two induction planes and a shorter collection plane in turn."""
    w = case["wires"]
    return [w if p % 3 < 2 else max(1, w * 3 // 5) for p in range(case["planes"])] if case["planes"] > 1 else [w]


def _weights(seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)

    def he(fan_in, *shape):
        return (torch.randn(shape, generator=g, device="cuda") * math.sqrt(2.0 / fan_in)).cpu().numpy()

    def bias(n):
        return ((torch.rand(n, generator=g, device="cuda") - 0.5) * 0.2).cpu().numpy()

    return {"conv_w": he(25, 48, 5, 5), "conv_b": bias(48), "fc1_w": he(FC1_IN, FC1_IN, FC1_OUT),
            "fc1_b": bias(FC1_OUT), "fc2_w": he(FC1_OUT, FC1_OUT, 32), "fc2_b": bias(32),
            "cls_w": he(32, 32, 3), "cls_b": bias(3), "mic_w": he(32, 32), "mic_b": bias(1)}


def _plane(W, T, rng, g):
    """One plane image on the GPU, and its hit candidates (wire, tick) on the GPU.

    Every object is added by itself with distinct indices, so that the image
    does not depend on the order of the additions."""
    img = torch.randn((W, T), generator=g, device="cuda") * NOISE
    tracks = max(3, 40 * W * T // (480 * 6000)) if W * T < 480 * 6000 else 40
    found = []
    lines = []
    for _ in range(tracks):
        w0, w1 = sorted(rng.uniform(0, W, 2))
        t0, t1 = rng.uniform(0, T, 2)
        amp, width = rng.uniform(20, 80), rng.uniform(1, 2)
        lo, hi = int(math.ceil(w0)), min(int(w1), W - 1)
        if hi < lo:
            continue
        slope = (t1 - t0) / max(w1 - w0, 1e-6)
        along = math.sqrt(1 + slope * slope)
        half = min(int(3 * width * along) + 1, 64)
        w = torch.arange(lo, hi + 1, device="cuda")
        centre = t0 + (w - w0) * slope
        t = centre.round().long()[:, None] + torch.arange(-half, half + 1, device="cuda")
        d = (t - centre[:, None]) / along
        ok = (t >= 0) & (t < T)
        at = (w[:, None] * T + t)[ok]
        img.view(-1)[at] += (amp * torch.exp(-0.5 * (d / width) ** 2))[ok].float()
        lines.append((w, centre))
    for _ in range(max(1, tracks // 8)):
        amp = rng.uniform(20, 60)
        wc, tc, sw, st = rng.uniform(0, W), rng.uniform(0, T), rng.uniform(3, 10), rng.uniform(10, 40)
        wa, wb = max(0, int(wc - 4 * sw)), min(W, int(wc + 4 * sw) + 1)
        ta, tb = max(0, int(tc - 4 * st)), min(T, int(tc + 4 * st) + 1)
        dw = (torch.arange(wa, wb, device="cuda") - wc) / sw
        dt = (torch.arange(ta, tb, device="cuda") - tc) / st
        img[wa:wb, ta:tb] += (amp * torch.exp(-0.5 * (dw[:, None] ** 2 + dt[None, :] ** 2))).float()
        hw = np.clip(np.rint(rng.normal(wc, sw, 400)), 0, W - 1)
        ht = np.clip(np.rint(rng.normal(tc, st, 400)), 0, T - 1)
        found.append(torch.from_numpy(np.stack([hw, ht], 1).astype(np.int64)).cuda())
    for w, centre in lines:                      # the peak within 5 ticks of the track
        t = (centre.round().long()[:, None] + torch.arange(-5, 6, device="cuda")).clamp(0, T - 1)
        best = img[w[:, None], t].argmax(1)
        found.append(torch.stack([w, t.gather(1, best[:, None])[:, 0]], 1))
    key = torch.unique(torch.cat([f[:, 0] * T + f[:, 1] for f in found]))
    return img, torch.stack([key // T, key % T], 1)


def _pick(cand, n, rng):
    """n hits of the candidates in random order, without repeats where there are enough."""
    if n <= len(cand):
        at = rng.permutation(len(cand))[:n]
    else:
        at = rng.integers(0, len(cand), n)
    return cand[torch.from_numpy(at).cuda()].to(torch.int32)


def _inputs(case, seed):
    """(images, hits or a list of (plane, hits), patches) on the GPU."""
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["call"] == "patches":
        n = case["n"]
        r = torch.arange(PATCH, device="cuda", dtype=torch.float32)
        u = torch.rand((n, 4), generator=g, device="cuda")
        off, ang, amp = u[:, :2] * 8 - 4, u[:, 2] * math.pi, 3 + 7 * u[:, 3]
        d = ((r[None, :, None] - 24 - off[:, 0, None, None]) * torch.sin(ang)[:, None, None]
             - (r[None, None, :] - 24 - off[:, 1, None, None]) * torch.cos(ang)[:, None, None])
        noise = torch.randn((n, PATCH, PATCH), generator=g, device="cuda")
        return None, None, noise + amp[:, None, None] * torch.exp(-0.5 * d * d)
    wires = _wires(case)
    made = [_plane(w, case["ticks"], rng, g) for w in wires]
    images = [m[0] for m in made]
    if case["call"] == "find_hits":
        return images, None, None
    if case["call"] == "classify":
        return images, _pick(made[0][1], case["n"], rng), None
    if case["call"] == "requests":
        planes = rng.integers(0, len(images), case["requests"])
        return images, [(int(p), _pick(made[p][1], case["n"], rng)) for p in planes], None
    # an event's hits, plane by plane in proportion to their wires
    quota = [case["n"] * w // sum(wires) for w in wires]
    quota[-1] += case["n"] - sum(quota)
    parts = []
    for p, q in enumerate(quota):
        h = _pick(made[p][1], q, rng)
        parts.append(torch.cat([torch.full((q, 1), p, dtype=torch.int32, device="cuda"), h], 1))
    return images, torch.cat(parts).contiguous(), None


def prepare(case, seed):
    images, hits, patches = _inputs(case, seed)
    state = {"case": case, "images": images, "hits": hits, "patches": patches,
             "handle": pid.pointid_create(_weights(seed), case["precision"], 0)}
    if case["call"] == "find_hits":
        # a buffer for one hit in ten samples, far more than are found
        cap = sum(im.numel() for im in images) // 10 + 64
        state["hits_out"] = torch.zeros((cap, 3), dtype=torch.int32, device="cuda")
        state["n_found"] = torch.zeros((1,), dtype=torch.int64, device="cuda")
    return state


def run(state):
    case, h = state["case"], state["handle"]
    call = case["call"]
    if call == "classify":
        return pid.pointid_classify(h, state["images"][0], state["hits"])
    if call == "planes":
        return pid.pointid_classify_planes(h, state["images"], state["hits"])
    if call == "patches":
        return pid.pointid_classify_patches(h, state["patches"])
    if call == "requests":
        return torch.cat(pid.pointid_classify_requests(
            h, state["images"], [(p, x, None) for p, x in state["hits"]]))
    if call == "ds":
        return pid.pointid_classify_planes_ds(h, state["images"], state["hits"],
                                              case["ticks_per_column"])
    return pid.pointid_find_hits(h, state["images"], case["threshold"],
                                 hits_out=state["hits_out"], n_found=state["n_found"])


def work(case):
    """Inputs, weights and outputs once.  Of the planes only what the hits' windows
    can hold is needed (all of them are for hit finding and tick binning)."""
    pixels = sum(_wires(case)) * case["ticks"] if case["planes"] else 0
    if case["call"] == "find_hits":
        return {"bytes": 4 * pixels, "flops": 0}
    n = case["n"] * max(1, case["requests"])
    weights = WEIGHT_VALUES * WEIGHT_BYTES[case["precision"]]
    seen = n * PATCH * PATCH * 4
    if case["call"] == "ds":
        image = 4 * pixels
    else:
        image = min(4 * pixels, seen) if pixels else seen
    hits = 0 if case["call"] == "patches" else 12 * n
    return {"bytes": image + hits + weights + 16 * n, "flops": n * FLOPS}


def tolerance(case):
    """About four times the distance from 64 bits that each arithmetic shows: 2e-6 in single
    precision; 2e-3 and 3e-3 to 1e-2 where operands are rounded to fp16 and bf16 (the logits reach
    100 with untrained weights); 8-bit operation against the network with its operands
    rounded, where one e4m3 step taken the other way moves a score by up to 1e-2."""
    if case["call"] == "find_hits":
        return "exact"
    return {"fp32": {"rel": 1e-5, "max": 1e-3}, "bf16": {"rel": 2e-2, "max": 0.4},
            "fp16": {"rel": 6e-3, "max": 0.2}, "fp8": {"rel": 2e-3, "max": 0.2}}[case["precision"]]


# ---- the same in 64 bits

def _windows(images, plane, wire, tick):
    """fp64 patches [n][48][48] of hits (plane, wire, tick); 0 outside the plane."""
    out = torch.zeros((len(plane), PATCH, PATCH), dtype=torch.float64, device="cuda")
    o = torch.arange(PATCH, device="cuda") - PATCH // 2
    for p, im in enumerate(images):
        at = (plane == p).nonzero()[:, 0]
        if not len(at):
            continue
        w, t = wire[at, None] + o, tick[at, None] + o
        ok = ((w >= 0) & (w < im.shape[0]))[:, :, None] & ((t >= 0) & (t < im.shape[1]))[:, None, :]
        v = im[w.clamp(0, im.shape[0] - 1)[:, :, None], t.clamp(0, im.shape[1] - 1)[:, None, :]]
        out[at] = torch.where(ok, v.double(), 0.0)
    return out


def _eight_bit(w):
    """(maps of fp64 patches, FC1 filter) in fp64 of a network whose FC1 takes e4m3
    operands: patches and conv filter in fp16, the maps clamped to 448, FC1 column n
    multiplied by the largest power of two that keeps it within 448, and by its inverse after."""
    e4m3 = torch.float8_e4m3fn
    big = w["fc1_w"].abs().amax(0)
    k = torch.floor(torch.log2(448.0 / big))
    k = torch.where(big * torch.exp2(k) > 448, k - 1, torch.where(big * torch.exp2(k + 1) <= 448, k + 1, k))
    fc1 = (w["fc1_w"] * torch.exp2(k)).float().to(e4m3).double() * torch.exp2(-k)
    kern = w["conv_w"].half().double().reshape(48, 25).t().contiguous()
    hi = w["conv_b"].half().double()
    bias = hi + (w["conv_b"] - hi).half().double()

    def maps(x):
        return _conv(x.half().double(), kern, bias).clamp(max=448).float().to(e4m3).double()
    return maps, fc1


def _conv(x, kern, bias):
    cols = torch.stack([x[:, u:u + FMAP, v:v + FMAP].reshape(-1) for u in range(5) for v in range(5)], 1)
    return torch.relu(cols @ kern + bias).reshape(len(x), FC1_IN)


def _network(patches_of, n, weights, precision):
    """Scores [n][4] in fp64; patches_of(a, b) gives the fp64 patches a .. b - 1."""
    w = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda().double() for k, v in weights.items()}
    kern, fc1 = w["conv_w"].reshape(48, 25).t().contiguous(), w["fc1_w"]
    maps = lambda x: _conv(x, kern, w["conv_b"])  # noqa: E731
    if precision == "fp8":
        maps, fc1 = _eight_bit(w)
    out = []
    for a in range(0, n, 512):
        h1 = torch.relu(maps(patches_of(a, min(a + 512, n))) @ fc1 + w["fc1_b"])
        h2 = torch.relu(h1 @ w["fc2_w"] + w["fc2_b"])
        p = torch.softmax(h2 @ w["cls_w"] + w["cls_b"], 1)
        q = torch.sigmoid(h2 @ w["mic_w"].reshape(32, 1) + w["mic_b"])
        out.append(torch.cat([p, q], 1))
    return torch.cat(out)


def _hits_in_order(images, threshold):
    rows = []
    for p, im in enumerate(images):
        inf = torch.full((im.shape[0], 1), -math.inf, device="cuda")
        before, after = torch.cat([inf, im[:, :-1]], 1), torch.cat([im[:, 1:], inf], 1)
        at = ((im > threshold) & (im > before) & (im >= after)).nonzero()
        rows.append(torch.cat([torch.full((len(at), 1), p, device="cuda"), at], 1))
    return torch.cat(rows).to(torch.int32)


def exact(case, seed):
    images, hits, patches = _inputs(case, seed)
    if case["call"] == "find_hits":
        rows = _hits_in_order(images, case["threshold"])
        out = torch.zeros((sum(im.numel() for im in images) // 10 + 64, 3), dtype=torch.int32, device="cuda")
        out[:min(len(rows), len(out))] = rows[:len(out)]
        return out, torch.tensor([len(rows)], dtype=torch.int64, device="cuda")
    weights = _weights(seed)
    if case["call"] == "patches":
        return _network(lambda a, b: patches[a:b].double(), case["n"], weights, case["precision"])
    if case["call"] == "requests":
        hits = torch.cat([torch.cat([torch.full((len(x), 1), p, dtype=torch.int32, device="cuda"), x], 1)
                          for p, x in hits])
    elif case["call"] == "classify":
        hits = torch.cat([torch.zeros((len(hits), 1), dtype=torch.int32, device="cuda"), hits], 1)
    plane, wire, tick = (hits[:, k].long() for k in range(3))
    if case["call"] == "ds":
        D = case["ticks_per_column"]
        pad = -case["ticks"] % D
        images = [torch.nn.functional.pad(im.double(), (0, pad)).reshape(im.shape[0], -1, D).sum(2)
                  for im in images]
        tick = torch.div(tick, D, rounding_mode="floor")
    return _network(lambda a, b: _windows(images, plane[a:b], wire[a:b], tick[a:b]), len(hits), weights,
                    case["precision"])
