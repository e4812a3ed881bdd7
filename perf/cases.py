"""Performance cases of the difference-imaging library: what its users run.

``listed()`` names the cases, ``draw(rng)`` draws further ones of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass through the public entry points, ``work(case)`` is
the traffic and arithmetic that a pass cannot do without, and
``exact(case, seed)`` gives the outputs in 64 bits from plain torch.

Kinds of case
  difference   one science frame against a resident reference: calibrate, fit,
               expand, subtract, detect (``Pipeline.difference``)
  reference    raw reference frames to a clipped coadd (``build_reference``),
               fused or by way of calibrated frames
  sources      background cells, filter, map and full-frame source detection
  matched      matched-filter coadd of calibrated frames
  healpix      a calibrated frame resampled into its NSIDE = 256 segments
  zogy         ZOGY subtraction on overlapping square tiles
  batch        constant-kernel differences of cutouts in one persistent launch
  train        one epoch of surrogate training and the updated weights
  surrogate    surrogate kernel per tile, judged against the plain fit
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2207_14304_amd import argus, surrogate
from paper_2207_14304_amd.pipeline import Pipeline

SIGMAS, DEGREES = (0.7, 1.5, 3.0), (4, 3, 2)
SKY, READ_NOISE, SCALE = 800.0, 1.7, 1.05
PRECISION = {"fp32": argus.FP32, "bf16x3": argus.BF16X3, "fp64": argus.FP64}
FULL_W, FULL_H = 9576, 6388


# ------------------------------------------------------------------ the cases
def _diff(W, H, D, h, tiles=1, precision="fp32", n_ref=5, name=None):
    c = {"kind": "difference", "W": W, "H": H, "D": D, "h": h, "tiles": tiles,
         "precision": precision, "n_ref": n_ref}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a postage-stamp pair: launches and host work count
        _diff(256, 224, 1, 7, 1, "fp32", 3, "difference 256x224"),
        # an odd-sized frame of the size the precision study uses, degree-2 kernel
        _diff(1100, 977, 2, 7, 16, "fp32", 5, "difference 1100x977"),
        # a quarter-scale frame with FP64 row moments, for poorly conditioned fields
        _diff(2394, 1597, 1, 10, 8, "fp64", 5, "difference fp64 2394x1597"),
        # the full frame of the benchmark
        _diff(FULL_W, FULL_H, 2, 10, 16, "fp32", 5, "difference full"),
        # a new pointing: the reference of the full frame
        {"name": "reference full", "kind": "reference", "W": FULL_W, "H": FULL_H, "n": 5,
         "fused": True},
        # background map and source list of every full frame (astrometry, photometry)
        {"name": "sources full", "kind": "sources", "W": FULL_W, "H": FULL_H, "box": 64,
         "map": True, "r": 7},
        # point-source coadd of half-scale frames
        {"name": "matched 4788x3194", "kind": "matched", "W": 4788, "H": 3194, "n": 5, "r": 7},
        # the full frame into its sky segments
        {"name": "healpix full", "kind": "healpix", "W": FULL_W, "H": FULL_H, "m": 600,
         "dec": 35.0},
        # the full frame covered by overlapping 512^2 tiles
        {"name": "zogy full", "kind": "zogy", "W": FULL_W, "H": FULL_H, "L": 512, "r": 7},
        # target cutouts of one camera, sides 64 to 512
        {"name": "batch 1500", "kind": "batch", "W": 4788, "H": 3194, "n": 1500, "h": 7,
         "precision": "fp64"},
        # an epoch over a small training set, minibatches of 32 tiles
        {"name": "train 256 tiles", "kind": "train", "N": 256, "batch": 32, "stamps": 16},
        # a frame of 4 x 4 tiles through the network and the acceptance test
        {"name": "surrogate 1024", "kind": "surrogate", "W": 1024, "H": 1024, "tiles": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame_size(rng, lo):
    W = _log(rng, lo, FULL_W)
    return W, max(lo * 2 // 3, min(FULL_H, int(W * rng.uniform(0.6, 0.9))))


def draw(rng):
    kind = rng.choice(["difference"] * 4 + ["reference"] * 2 + ["sources", "matched", "healpix",
                                                                "zogy", "batch", "train",
                                                                "surrogate"])
    if kind == "difference":
        D = rng.choice([0, 1, 2, 2])
        h = rng.choice([7, 7, 10])
        # a degree-2 kernel on every fit pixel of a small frame is poorly determined
        W, H = _frame_size(rng, (160, 384, 1024)[D])
        return _diff(W, H, D, h, rng.choice([1, 4, 16]),
                     rng.choice(["fp32"] * 4 + ["fp64", "bf16x3"]), rng.randint(1, 5))
    if kind == "reference":
        W, H = _frame_size(rng, 300)
        return {"kind": kind, "W": W, "H": H, "n": rng.randint(2, 8),
                "fused": rng.random() < 0.7}
    if kind == "sources":
        W, H = _frame_size(rng, 500)
        return {"kind": kind, "W": W, "H": H, "box": rng.choice([32, 64, 64]),
                "map": rng.random() < 0.7, "r": rng.randint(4, 9)}
    if kind == "matched":
        W, H = _frame_size(rng, 500)
        W, H = min(W, 4788), min(H, 3194)
        return {"kind": kind, "W": W, "H": H, "n": rng.randint(2, 5), "r": rng.randint(4, 9)}
    if kind == "healpix":
        W, H = _frame_size(rng, 1200)
        return {"kind": kind, "W": W, "H": H, "m": rng.choice([300, 600, 600]),
                "dec": round(rng.uniform(-75.0, 75.0), 2)}
    if kind == "zogy":
        L = rng.choice([256, 512, 512, 1024])
        W, H = _frame_size(rng, 1200)
        return {"kind": kind, "W": W, "H": H, "L": L, "r": rng.randint(5, 8)}
    if kind == "batch":
        return {"kind": kind, "W": 4788, "H": 3194, "n": _log(rng, 40, 1500), "h": 7,
                "precision": rng.choice(["fp64", "fp64", "fp32"])}
    if kind == "train":
        b = rng.choice([16, 32, 32])
        return {"kind": kind, "N": b * rng.randint(2, 8), "batch": b,
                "stamps": rng.randint(6, 16)}
    return {"kind": kind, "W": rng.randint(800, 1600), "H": rng.randint(700, 1500), "tiles": 4}


# ------------------------------------------------------------------ synthetic sky
def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 7919 * k + 1)
    return g


def _blur(img, sigma):
    """Unit-sum double Gaussian (a core and a fifth of the flux in wings)."""
    out = torch.zeros_like(img)
    for frac, s in ((0.8, sigma), (0.2, 2.0 * sigma)):
        R = int(math.ceil(4.0 * s))
        k = torch.exp(-0.5 * (torch.arange(-R, R + 1, dtype=torch.float64) / s) ** 2)
        k = (k / k.sum()).tolist()
        H, W = img.shape
        t = torch.zeros_like(img)
        p = torch.nn.functional.pad(img, (R, R))
        for i, w in enumerate(k):
            t.add_(p[:, i:i + W], alpha=w)
        p = torch.nn.functional.pad(t, (0, 0, R, R))
        for i, w in enumerate(k):
            out.add_(p[i:i + H], alpha=frac * w)
    return out


def _scene(W, H, seed, varying, n_stars=None):
    """(reference, science) scenes in electrons: stars dN/df ~ f^-1.75 and, in
    the science frame, transients; with ``varying`` the seeing grows along x."""
    g = _gen(seed, 0)
    n = max(40, int(60000 * W * H / (FULL_W * FULL_H))) if n_stars is None else n_stars
    at = torch.unique(torch.randint(0, W * H, (n,), generator=g, device="cuda"))
    u = torch.rand(at.numel(), generator=g, device="cuda", dtype=torch.float64)
    a, b = 1e6 ** -0.75, 1e2 ** -0.75
    pts = torch.zeros(W * H, device="cuda")
    pts[at] = ((a + u * (b - a)) ** (-4.0 / 3.0)).float()
    new = torch.unique(torch.randint(0, W * H, (20,), generator=g, device="cuda"))
    add = torch.zeros(W * H, device="cuda")
    add[new] = (1e3 * 100.0 ** torch.rand(new.numel(), generator=g, device="cuda")).float()
    pts, add = pts.view(H, W), (SCALE * pts + add).view(H, W)
    if not varying:
        return _blur(pts, 0.85), _blur(add, 1.10)
    t = torch.linspace(0.0, 1.0, W, device="cuda")
    ref = _blur(pts, 0.8) * (1 - t) + _blur(pts, 1.3) * t
    return ref, _blur(add, 1.05) * (1 - t) + _blur(add, 1.7) * t


def _u16(t):
    return (t.clamp(0, 65535).round().to(torch.int32) & 0xFFFF).to(torch.int16).view(torch.uint16)


def _counts(raw, dtype):
    return (raw.view(torch.int16).to(torch.int32) & 0xFFFF).to(dtype)


def _masters(W, H, seed, plain=False):
    """dark (with hot pixels), vignetted flat, bad-pixel mask."""
    if plain:
        return (torch.zeros((H, W), device="cuda"), torch.ones((H, W), device="cuda"), None)
    g = _gen(seed, 1)
    dark = torch.full((H, W), 100.0, device="cuda")
    dark += (torch.rand((H, W), generator=g, device="cuda") < 5e-4) * 2000.0
    y = torch.linspace(-1, 1, H, device="cuda")[:, None] ** 2
    x = torch.linspace(-1, 1, W, device="cuda")[None, :] ** 2
    flat = (1 - 0.075 * (x + y)) * (1 + 0.01 * torch.randn((H, W), generator=g, device="cuda"))
    bpm = (torch.rand((H, W), generator=g, device="cuda") < 1e-4).to(torch.uint8)
    return dark, flat, bpm


def _expose(scene, masters, seed, k, cosmics=0.0):
    g = _gen(seed, 2 + k)
    dark, flat, bpm = masters
    e = flat * (scene + SKY)
    if cosmics:
        e = e + (torch.rand(e.shape, generator=g, device="cuda") < cosmics) * 5000.0
    adu = torch.poisson(e, generator=g)
    adu += READ_NOISE * torch.randn(e.shape, generator=g, device="cuda") + dark
    if bpm is not None:
        adu = torch.where(bpm != 0, 65535.0 * (torch.rand(e.shape, generator=g, device="cuda") < 0.5),
                          adu)
    return _u16(adu)


def _raws(case, seed, n_ref, plain=False):
    W, H = case["W"], case["H"]
    m = _masters(W, H, seed, plain)
    ref, sci = _scene(W, H, seed, case.get("D", 0) > 0)
    return m, [_expose(ref, m, seed, 1 + k, 1e-5) for k in range(n_ref)], _expose(sci, m, seed, 0)


def _calibrated(raw, masters):
    """64-bit calibration: value, variance, mask."""
    dark, flat, bpm = masters
    f, c = flat.double(), _counts(raw, torch.float64)
    s = c - dark.double()
    cal, var = s / f, (s.clamp(min=0) + READ_NOISE ** 2) / (f * f)
    mask = torch.zeros(raw.shape, dtype=torch.uint8, device="cuda")
    if bpm is not None:
        bad = bpm != 0
        cal[bad] = 0.0
        var[bad] = 0.0
        mask[bad] = argus.BAD
    mask[c >= 65535] |= argus.SAT
    return cal, var, mask


def _single(case, seed, k=0, plain=False):
    """One calibrated frame as a program holds it (32-bit planes), without the rest."""
    W, H = case["W"], case["H"]
    m = _masters(W, H, seed, plain)
    ref, sci = _scene(W, H, seed, False)
    c, v, mask = _calibrated(_expose(sci if k == 0 else ref, m, seed, k), m)
    return c.float(), v.float(), mask


def _psf(r, sigma):
    u = np.arange(-r, r + 1, dtype=np.float64)
    p = np.exp(-0.5 * (u[:, None] ** 2 + u[None, :] ** 2) / sigma ** 2)
    return (p / p.sum()).astype(np.float32)


def _dev(a):
    return torch.as_tensor(a).cuda()


def _empty(shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _spec(case):
    return argus.make_spec(half_width=case["h"], spatial_degree=case["D"], bg_degree=case["D"],
                           tiles_x=case["tiles"], tiles_y=case["tiles"],
                           precision=PRECISION[case["precision"]])


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return state["pass"](state)


def _candidates(buf, dtype):
    """Integer and floating columns of a candidate buffer (views)."""
    n = dtype.itemsize // 4
    t = buf.view(torch.int32).view(-1, n)
    return t[:, :2], t.view(torch.float32)[:, 2:]


def _prepare_difference(case, seed):
    m, raws, sci = _raws(case, seed, case["n_ref"])
    pipe = Pipeline(argus.Context(0), case["W"], case["H"], _spec(case), _psf(7, 1.3),
                    capacity=16384)
    pipe.cands.zero_()
    pipe.set_masters(m[0].cpu().numpy(), m[1].cpu().numpy(), m[2].cpu().numpy())
    pipe.build_reference(raws)
    at, values = _candidates(pipe.cands, argus.CANDIDATE_DTYPE)
    # the product of the path: the images and the candidates (the kernel between fit and
    # subtraction is in every pixel of `diff`, chi2 a sum over it)
    return {"pass": _run_difference, "pipe": pipe, "sci": sci,
            "out": {"diff": pipe.diff, "diff_var": pipe.diff_var, "diff_mask": pipe.diff_mask,
                    "snr": pipe.snr, "det_mask": pipe.det_mask, "n_fit": pipe.n_fit,
                    "n_chi2": pipe.n_chi2, "status": pipe.status, "n_cands": pipe.n_cands,
                    "cand_at": at, "cand_values": values}}


def _run_difference(s):
    s["pipe"].difference(s["sci"])
    return s["out"]


def _prepare_reference(case, seed):
    m, raws, _ = _raws(case, seed, case["n"])
    pipe = Pipeline(argus.Context(0), case["W"], case["H"], argus.make_spec(), _psf(7, 1.3),
                    capacity=16)
    pipe.set_masters(m[0].cpu().numpy(), m[1].cpu().numpy(), m[2].cpu().numpy())
    return {"pass": _run_reference, "pipe": pipe, "raws": raws, "fused": case["fused"],
            "out": {"ref": pipe.ref, "ref_var": pipe.ref_var, "ref_mask": pipe.ref_mask,
                    "n_used": pipe.n_used}}


def _run_reference(s):
    s["pipe"].build_reference(s["raws"], fused=s["fused"])
    return s["out"]


def _grid_shape(case):
    return -(-case["H"] // case["box"]), -(-case["W"] // case["box"])


def _prepare_sources(case, seed):
    W, H, r = case["W"], case["H"], case["r"]
    cap = 32768
    src = _empty(cap * argus.SOURCE_DTYPE.itemsize, torch.uint8)
    at, values = _candidates(src, argus.SOURCE_DTYPE)
    out = {"grid": _empty(_grid_shape(case)), "snr": _empty((H, W)),
           "det_mask": _empty((H, W), torch.uint8), "n_sources": _empty(1, torch.int32),
           "source_at": at, "source_values": values}
    if case["map"]:
        out["map"] = _empty((H, W))
    return {"pass": _run_sources, "ctx": argus.Context(0), "planes": _single(case, seed),
            "psf": _dev(_psf(r, 1.1)), "r": r, "box": case["box"], "src": src, "cap": cap,
            "out": out}


def _run_sources(s):
    o, (cal, var, mask) = s["out"], s["planes"]
    s["ctx"].background(cal, mask, s["box"], o["grid"], None, o.get("map"))
    s["ctx"].detect_sources(cal, var, mask, o["grid"], s["box"], 5.0, s["psf"], s["r"], o["snr"],
                            o["det_mask"], s["src"], s["cap"], o["n_sources"])
    return o


def _matched_inputs(case, seed):
    W, H = case["W"], case["H"]
    m, raws, _ = _raws(case, seed, case["n"])
    planes = [_calibrated(r, m) for r in raws]
    planes = [(c.float(), v.float(), k) for c, v, k in planes]
    g = _gen(seed, 50)
    grids = [SKY + 5 * torch.rand((-(-H // 64), -(-W // 64)), generator=g, device="cuda")
             for _ in raws]
    psf = np.stack([_psf(case["r"], 0.9 + 0.1 * k) for k in range(case["n"])])
    scales = [1.0 + 0.03 * k for k in range(case["n"])]
    return planes, grids, psf, scales


def _prepare_matched(case, seed):
    W, H = case["W"], case["H"]
    planes, grids, psf, scales = _matched_inputs(case, seed)
    return {"pass": _run_matched, "ctx": argus.Context(0), "planes": list(zip(*planes)),
            "grids": grids, "psf": _dev(psf), "r": case["r"], "scales": scales,
            "out": {"score": _empty((H, W)), "score_var": _empty((H, W)), "snr": _empty((H, W))}}


def _run_matched(s):
    o, (cal, var, mask) = s["out"], s["planes"]
    s["ctx"].coadd_matched(cal, var, mask, s["psf"], s["r"], o["score"], o["score_var"], o["snr"],
                           s["grids"], 64, s["scales"])
    return o


def _wcs_values(case):
    s = 1.38 / 3600.0
    return (120.0, case["dec"], (case["W"] - 1) / 2.0, (case["H"] - 1) / 2.0,
            [[-s * math.cos(0.4), s * math.sin(0.4)], [s * math.sin(0.4), s * math.cos(0.4)]])


def _prepare_healpix(case, seed):
    wcs = argus.make_wcs(*_wcs_values(case))
    tiles = _dev(argus.healpix_tiles(wcs, case["W"], case["H"], 256, 32))
    shape = (tiles.shape[0], case["m"], case["m"])
    return {"pass": _run_healpix, "ctx": argus.Context(0), "planes": _single(case, seed),
            "wcs": wcs, "tiles": tiles, "m": case["m"],
            "out": {"value": _empty(shape), "var": _empty(shape),
                    "mask": _empty(shape, torch.uint8)}}


def _run_healpix(s):
    o = s["out"]
    s["ctx"].resample_healpix(*s["planes"], s["wcs"], 256, s["m"], s["tiles"], o["value"],
                              o["var"], o["mask"])
    return o


ZOGY_SCALARS = (1.05, 1.0, 28.5, 28.4)      # Fn, Fr, sn, sr


def _zogy_inputs(case, seed):
    W, H, L, r = case["W"], case["H"], case["L"], case["r"]
    n, _, mn = _single(case, seed, 0)
    f, _, mr = _single(case, seed, 1)
    step = L - 4 * r
    at = [(x, y) for y in range(0, H, step) for x in range(0, W, step)]
    return (n - SKY, mn, f - SKY, mr, np.array(at, np.int32), _psf(r, 1.15), _psf(r, 0.9))


def _prepare_zogy(case, seed):
    n, mn, f, mr, at, pn, pr = _zogy_inputs(case, seed)
    shape = (len(at), case["L"], case["L"])
    return {"pass": _run_zogy, "ctx": argus.Context(0), "in": (n, mn, f, mr, _dev(at)),
            "L": case["L"], "psfs": (_dev(pn), _dev(pr), case["r"]),
            "out": {"D": _empty(shape), "snr": _empty(shape), "flux": _empty(shape),
                    "mask": _empty(shape, torch.uint8), "pd2": _empty(1, torch.float64)}}


def _run_zogy(s):
    o = s["out"]
    s["ctx"].zogy(*s["in"], s["L"], *s["psfs"], *ZOGY_SCALARS, o["D"], o["snr"], o["flux"],
                  o["mask"], o["pd2"])
    return o


def _cutouts(case, seed):
    n, W, H = case["n"], case["W"], case["H"]
    # the sides make the size of the case, the places come with the seed
    side = np.floor(64 * 8.0 ** np.random.default_rng(n).random(n)).astype(np.int64)
    rng = np.random.default_rng(seed)
    x0 = (rng.random(n) * (W - side)).astype(np.int64)
    y0 = (rng.random(n) * (H - side)).astype(np.int64)
    return x0, y0, side


def _pair(case, seed):
    m, (ref,), sci = _raws(case, seed, 1, plain=True)
    return tuple(p for raw in (ref, sci) for c in [_calibrated(raw, m)]
                 for p in (c[0].float(), c[1].float(), c[2]))


def _prepare_batch(case, seed):
    W, H = case["W"], case["H"]
    x0, y0, side = _cutouts(case, seed)
    ctx = argus.Context(0)
    spec = argus.make_spec(half_width=case["h"], precision=PRECISION[case["precision"]])
    b = argus.Batch(ctx, spec, [0] * case["n"], x0, y0, side, [W], [H])
    n = b.n
    out = {"diff": _empty(b.arena), "diff_var": _empty(b.arena),
           "diff_mask": _empty(b.arena, torch.uint8), "det_mask": _empty(b.arena, torch.uint8),
           "coeffs": _empty((n, 32), torch.float64), "chi2": _empty(n, torch.float64),
           "n_fit": _empty(n, torch.int64), "status": _empty(n, torch.int32),
           "n_cands": _empty(n, torch.int32)}
    return {"pass": _run_batch, "ctx": ctx, "batch": b, "frames": [_pair(case, seed)], "out": out}


def _run_batch(s):
    s["ctx"].batch_run(s["batch"], s["frames"], 5.0, *s["out"].values())
    return s["out"]


def _prepare_train(case, seed):
    """Star stamps (normalised, reference and science) of N tiles and standardized targets."""
    N, k, g = case["N"], case["stamps"], _gen(seed, 60)
    u = torch.arange(-15, 16, device="cuda", dtype=torch.float32)
    r2 = (u[:, None] ** 2 + u[None, :] ** 2).reshape(-1)
    s = 0.7 + 0.6 * torch.rand((N, 1, 1), generator=g, device="cuda")
    X = torch.zeros((N, argus.CNN_STAMPS, argus.CNN_NPX, 2), device="cuda")
    for j, grow in enumerate((1.0, 1.3)):
        p = torch.exp(-0.5 * r2 / (s * grow) ** 2)
        X[:, :k, :, j] = 100.0 * p / p.sum(-1, keepdim=True) + \
            0.1 * torch.randn((N, k, argus.CNN_NPX), generator=g, device="cuda")
    valid = torch.zeros((N, argus.CNN_STAMPS), dtype=torch.uint8, device="cuda")
    valid[:, :k] = 1
    w = torch.randn((1, surrogate.NB), generator=g, device="cuda")
    target = (s[:, 0] - 1.0) * 5.0 * w + 0.1 * torch.randn((N, surrogate.NB), generator=g,
                                                           device="cuda")
    cnn = argus.CNN(argus.Context(0), case["batch"])
    cnn.set_weights(surrogate.init_weights(seed))
    return {"pass": _run_train, "cnn": cnn, "X": X.to(torch.bfloat16), "valid": valid,
            "target": target.contiguous(), "batch": case["batch"]}


def _run_train(s):
    loss = surrogate.train(s["cnn"], s["X"], s["valid"], s["target"], 1, s["batch"], 1e-3)
    return {"weights": s["cnn"].get_weights(), "loss": np.asarray(loss, np.float32)}


def _prepare_surrogate(case, seed):
    T = case["tiles"]
    ctx = argus.Context(0)
    cnn = argus.CNN(ctx, T * T)
    cnn.set_weights(surrogate.init_weights(seed))
    path = surrogate.SurrogatePath(ctx, cnn, case["W"], case["H"], T)
    return {"pass": _run_surrogate, "ctx": ctx, "path": path, "planes": _pair(case, seed)}


def _run_surrogate(s):
    p = s["path"]
    plain = surrogate.TileFits(s["ctx"], s["planes"], p.sp)
    p.predict(s["planes"])
    p.select(plain)
    return {"network": p.out, "stamps": p.stamps, "coeffs": p.coeffs, "chi2_dof": p.chi2_dof,
            "accepted": p.accepted, "plain_status": plain.status}


# ------------------------------------------------------------------ work
def work(case):
    """Bytes and operations of one pass: inputs read once, outputs written once,
    and the arithmetic of the method (moments, separable basis convolutions,
    taps, transforms)."""
    k = case["kind"]
    n = float(case["W"] * case["H"]) if "W" in case else 0.0
    if k in ("difference", "surrogate"):
        D, h = case.get("D", 0), case.get("h", 7)
        taps = (2 * h + 1) ** 2 * {0: 4, 1: 7, 2: 9}[D]
        conv = 2 * 43 * (2 * h + 1)                   # 12 row and 31 column filters
        f = n * (2 * 528 * (2 * D + 1) + conv + taps)
        if k == "difference":
            return {"bytes": n * (11 + 9 + 14), "flops": f}
        return {"bytes": n * 18, "flops": f + n * (taps + 20)}
    if k == "reference":
        return {"bytes": n * (2 * case["n"] + 19), "flops": n * 20 * case["n"]}
    if k == "sources":
        return {"bytes": n * (9 + 5 + 4 * case["map"]), "flops": n * 20}
    if k == "matched":
        return {"bytes": n * (9 * case["n"] + 12),
                "flops": n * case["n"] * 4 * (2 * case["r"] + 1) ** 2}
    if k == "healpix":
        return {"bytes": n * 9 * 2, "flops": n * 100}
    if k == "zogy":
        L = case["L"]
        step = L - 4 * case["r"]
        t = -(-case["W"] // step) * -(-case["H"] // step) * L * L
        return {"bytes": t * (10 + 13.0), "flops": t * (2 * 2 * 5 * math.log2(L) + 60)}
    if k == "batch":
        p = case["n"] * 64.0 ** 2 * (64 - 1) / (2 * math.log(8))      # mean of side^2
        h = case["h"]
        return {"bytes": p * (18 + 10), "flops": p * (2 * 528 + 86 * (2 * h + 1)
                                                      + 4 * (2 * h + 1) ** 2)}
    stamps = case["N"] * case["stamps"]
    return {"bytes": stamps * 961 * 4.0 * 3,
            "flops": stamps * 961 * 32 * (2 * (18 + 3 * 288) + 3 * 288) * 2.0}


# ------------------------------------------------------------------ exact (64 bits)
def exact(case, seed):
    """The outputs in 64 bits from plain torch.  Integers, and lists whose
    members a threshold chooses, have no such value; nor have the surrogate's
    outputs (its stamps are chosen by rank and its weights are bf16 values
    that every training step rounds)."""
    f = globals().get("_exact_" + case["kind"])
    return f(case, seed) if f else None


def _median(x, ok):
    """Median over dim 0 of the entries marked ok (the mean of the middle two)."""
    n = ok.sum(0)
    s = torch.where(ok, x, torch.full_like(x, math.inf)).sort(0).values
    lo = ((n - 1).clamp(min=0) // 2)[None]
    hi = (n // 2).clamp(max=x.shape[0] - 1)[None]
    return 0.5 * (s.gather(0, lo)[0] + s.gather(0, hi)[0])


def _coadd(planes):
    """Clipped mean of calibrated frames: reject |x - median| > 3 sigma, up to 5 passes."""
    x, v = (torch.stack([p[i] for p in planes]) for i in (0, 1))
    m = torch.stack([p[2] for p in planes])
    S = (m & (argus.BAD | argus.SAT)) == 0
    for _ in range(5):
        n = S.sum(0)
        rej = S & ((x - _median(x, S)).abs() > 3.0 * _median(v, S).sqrt())
        go = (n > 2) & (rej.sum(0) > 0) & (n - rej.sum(0) >= 2)
        S = S & ~(rej & go)
    n = S.sum(0)
    ref = torch.where(S, x, 0.0).sum(0) / n.clamp(min=1)
    var = torch.where(S, v, 0.0).sum(0) / n.clamp(min=1) ** 2
    mask = torch.where(n == 0, argus.NODATA, 0).to(torch.uint8)
    return ref, var, mask | torch.where(((m & argus.SAT) != 0).any(0), argus.SAT, 0).to(torch.uint8)


def _reference64(raws, masters):
    H = raws[0].shape[0]
    rows = max(1, (1 << 23) // raws[0].shape[1])
    parts = []
    for y in range(0, H, rows):
        ms = tuple(None if t is None else t[y:y + rows] for t in masters)
        parts.append(_coadd([_calibrated(r[y:y + rows], ms) for r in raws]))
    return tuple(torch.cat(p) for p in zip(*parts))


def _exact_reference(case, seed):
    m, raws, _ = _raws(case, seed, case["n"])
    ref, var, _ = _reference64(raws, m)
    return {"ref": ref, "ref_var": var, "ref_mask": None, "n_used": None}


def _basis(h):
    u = np.arange(-h, h + 1, dtype=np.float64)
    U, V = np.meshgrid(u, u)
    B, even = [], []
    for s, d in zip(SIGMAS, DEGREES):
        for i in range(d + 1):
            for j in range(d - i + 1):
                B.append(np.exp(-(U * U + V * V) / (2 * s * s)) * U ** i * V ** j)
                even.append(i % 2 == 0 and j % 2 == 0)
    B = np.stack(B)
    B[0] /= B[0].sum()
    for k in range(1, len(B)):
        if even[k]:
            B[k] -= B[k].sum() * B[0]
        B[k] /= math.sqrt((B[k] ** 2).sum())
    return torch.as_tensor(B).cuda()


def _windows(img, h, y0, y1):
    """[(y1 - y0) (W - 2h)][(2h+1)^2] footprints, flipped for true convolution."""
    K = 2 * h + 1
    w = img[y0 - h:y1 + h].unfold(0, K, 1).unfold(1, K, 1)
    return w.flip(2, 3).reshape(-1, K * K)


def _difference64(planes, h, D):
    """(coefficients, difference, variance, chi2) of the global fit."""
    ref, rv, rm, sci, sv, sm = planes
    H, W = ref.shape
    B = _basis(h)
    nb, mon = B.shape[0], [(p, q) for p in range(D + 1) for q in range(D - p + 1)]
    foot = (rm != 0)
    wide = foot.clone()
    for k in range(1, h + 1):
        wide[:, k:] |= foot[:, :-k]
        wide[:, :-k] |= foot[:, k:]
    foot = wide.clone()
    for k in range(1, h + 1):
        foot[k:] |= wide[:-k]
        foot[:-k] |= wide[k:]
    clean = ~foot & (sm == 0)
    clean[:h] = clean[H - h:] = False
    clean[:, :h] = clean[:, W - h:] = False
    xt = (2.0 * torch.arange(W, device="cuda", dtype=torch.float64) - (W - 1)) / (W - 1)
    yt = (2.0 * torch.arange(H, device="cuda", dtype=torch.float64) - (H - 1)) / (H - 1)
    ref64, rv64 = ref.double(), rv.double()
    rows = max(1, (1 << 17) // (W - 2 * h))
    n = nb * len(mon) + len(mon)
    A, b = (torch.zeros(s, device="cuda", dtype=torch.float64) for s in ((n, n), (n,)))

    def chunk(y0):
        y1 = min(y0 + rows, H - h)
        at = (slice(y0, y1), slice(h, W - h))
        P = torch.stack([(xt[None, h:W - h] ** p * yt[y0:y1, None] ** q).reshape(-1)
                         for p, q in mon], 1)
        C = _windows(ref64, h, y0, y1) @ B.reshape(nb, -1).T
        X = torch.cat([(C[:, :, None] * P[:, None, :]).reshape(len(P), -1), P], 1)
        var = (sv[at].double() + rv64[at]).reshape(-1)
        ok = clean[at].reshape(-1) & (var > 0)
        return y1, at, P, X, torch.where(ok, 1.0 / torch.where(ok, var, 1.0), 0.0)

    for y0 in range(h, H - h, rows):
        _, at, _, X, w = chunk(y0)
        wX = X * w[:, None]
        A += X.T @ wX
        b += wX.T @ sci[at].double().reshape(-1)
    A, b = A.cpu(), b.cpu()
    d = A.diagonal().sqrt()
    a = (torch.linalg.solve(A / d[:, None] / d[None, :], b / d) / d).cuda()
    stamps = torch.einsum("km,kv->mv", a[:nb * len(mon)].view(nb, len(mon)), B.reshape(nb, -1))
    diff, dvar = torch.zeros_like(ref64), torch.zeros_like(ref64)
    chi2 = 0.0
    for y0 in range(h, H - h, rows):
        y1, at, P, X, w = chunk(y0)
        keep = clean[at]
        r = sci[at].double() - (X @ a).view(keep.shape)
        v = ((P @ stamps) ** 2 * _windows(rv64, h, y0, y1)).sum(1).view(keep.shape)
        diff[at] = torch.where(keep, r, 0.0)
        dvar[at] = torch.where(keep, sv[at].double() + v, 0.0)
        chi2 = chi2 + (w * r.reshape(-1) ** 2).sum()
    return a, diff, dvar, chi2


def _snr(diff, var):
    return torch.where(var > 0, diff / torch.where(var > 0, var, 1.0).sqrt(), 0.0)


def _exact_difference(case, seed):
    m, raws, sci = _raws(case, seed, case["n_ref"])
    planes = _reference64(raws, m) + _calibrated(sci, m)
    _, diff, var, _ = _difference64(planes, case["h"], case["D"])
    none = ("diff_mask", "det_mask", "n_fit", "n_chi2", "status", "n_cands", "cand_at",
            "cand_values")
    return {"diff": diff, "diff_var": var, "snr": _snr(diff, var),
            **dict.fromkeys(none)}


def _cells(n, box):
    """Per pixel of an axis: left node, right node and the right node's weight."""
    a = np.arange(0, n, box)
    c = (a + np.minimum(a + box, n) - 1) / 2.0
    x = np.arange(n, dtype=np.float64)
    i = np.clip(np.searchsorted(c, x, side="right") - 1, 0, len(c) - 1)
    j = np.minimum(i + 1, len(c) - 1)
    t = np.where((x >= c[0]) & (j > i), (x - c[i]) / np.maximum(c[j] - c[i], 1e-9), 0.0)
    return _dev(i), _dev(j), _dev(t)


def _bilinear(grid, W, H, box):
    i, i1, t = _cells(W, box)
    j, j1, s = _cells(H, box)
    g = grid.double()
    top = g[j][:, i] + t * (g[j][:, i1] - g[j][:, i])
    bot = g[j1][:, i] + t * (g[j1][:, i1] - g[j1][:, i])
    return top + s[:, None] * (bot - top)


def _exact_sources(case, seed):
    cal, var, mask = _single(case, seed)
    W, H, box = case["W"], case["H"], case["box"]
    gy, gx = _grid_shape(case)
    pad = (0, gx * box - W, 0, gy * box - H)
    x = torch.nn.functional.pad(cal.double(), pad)
    ok = torch.nn.functional.pad(mask == 0, pad)
    cell = [t.view(gy, box, gx, box).permute(1, 3, 0, 2).reshape(box * box, gy, gx)
            for t in (x, ok)]
    some = cell[1].any(0)
    lev = torch.nn.functional.pad(torch.where(some, _median(*cell), 0.0).float().double(), (1,) * 4)
    ok = torch.nn.functional.pad(some, (1,) * 4)
    nine = [torch.stack([t[j:j + gy, i:i + gx] for j in range(3) for i in range(3)])
            for t in (lev, ok)]
    grid = torch.where(nine[1].any(0), _median(*nine), 0.0)
    bg = _bilinear(grid, W, H, box)
    good = (mask == 0) & (var > 0)
    d = torch.where(good, cal.double() - bg, 0.0)
    out = {"grid": grid, "snr": _snr(d, torch.where(good, var.double(), 0.0)),
           **dict.fromkeys(("det_mask", "n_sources", "source_at", "source_values"))}
    return dict(out, map=bg) if case["map"] else out


def _exact_matched(case, seed):
    W, H, r = case["W"], case["H"], case["r"]
    planes, grids, psf, scales = _matched_inputs(case, seed)
    S, V = (torch.zeros((H, W), device="cuda", dtype=torch.float64) for _ in range(2))
    for (cal, var, mask), grid, P, F in zip(planes, grids, psf, scales):
        ok = (mask == 0) & (var > 0)
        b = torch.where(ok, 1.0 / torch.where(ok, var.double(), 1.0), 0.0)
        a = (cal.double() - _bilinear(grid, W, H, 64)) * b
        a, b = (torch.nn.functional.pad(t, (r,) * 4) for t in (a, b))
        F = float(np.float32(F))
        for v in range(2 * r + 1):
            for u in range(2 * r + 1):
                p = F * float(P[v, u])
                S.add_(a[v:v + H, u:u + W], alpha=p)
                V.add_(b[v:v + H, u:u + W], alpha=p * p)
    return {"score": S, "score_var": V, "snr": _snr(S, V)}


def _exact_healpix(case, seed):
    cal, var, mask = _single(case, seed)
    W, H, m = case["W"], case["H"], case["m"]
    ra0, dec0, cx, cy, cd = _wcs_values(case)
    # the tile list is an input of the call
    tiles = argus.healpix_tiles(argus.make_wcs(ra0, dec0, cx, cy, cd), W, H, 256, 32)
    inv = np.linalg.inv(np.array(cd))
    a0, d0 = math.radians(ra0), math.radians(dec0)
    k = torch.arange(m, device="cuda", dtype=torch.float64)
    out = [torch.zeros((len(tiles), m, m), device="cuda", dtype=torch.float64) for _ in range(2)]
    q = math.pi / 4
    for t, (f, I, J) in enumerate(tiles.tolist()):
        a, b = (I * m + k[None, :] + 0.5) / (256 * m), (J * m + k[:, None] + 0.5) / (256 * m)
        xc, yc = ((q + f * 2 * q, q) if f < 4 else ((f - 4) * 2 * q, 0.0) if f < 8
                  else (q + (f - 8) * 2 * q, -q))
        xs = torch.remainder(xc + q * (a - b), 2 * math.pi)
        ys = yc + q * (a + b - 1)
        sig = 2.0 - ys.abs() / q
        pc = q + torch.floor(xs / (2 * q)) * 2 * q
        cap = ys.abs() > q
        z = torch.where(cap, ys.sign() * (1 - sig * sig / 3), ys * 8 / (3 * math.pi))
        phi = torch.where(cap, pc + (xs - pc) / torch.where(cap, sig, 1.0), xs)
        c = (1 - z * z).sqrt()
        den = z * math.sin(d0) + c * math.cos(d0) * torch.cos(phi - a0)
        xi = torch.rad2deg(c * torch.sin(phi - a0) / den)
        eta = torch.rad2deg((z * math.cos(d0) - c * math.sin(d0) * torch.cos(phi - a0)) / den)
        x = inv[0, 0] * xi + inv[0, 1] * eta + cx
        y = inv[1, 0] * xi + inv[1, 1] * eta + cy
        ok = (den > 0) & (x >= 0) & (x <= W - 1) & (y >= 0) & (y <= H - 1)
        x0, y0 = x.floor().clamp(0, W - 2).long(), y.floor().clamp(0, H - 2).long()
        fx, fy = x - x0, y - y0
        at = [(y0 + j) * W + x0 + i for j in (0, 1) for i in (0, 1)]
        w = [(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy]
        for p in at:
            ok &= mask.view(-1)[p] == 0
        out[0][t] = torch.where(ok, sum(wi * cal.view(-1)[p].double() for wi, p in zip(w, at)), 0.0)
        out[1][t] = torch.where(ok, sum(wi * wi * var.view(-1)[p].double()
                                        for wi, p in zip(w, at)), 0.0)
    return {"value": out[0], "var": out[1], "mask": None}


def _exact_zogy(case, seed):
    n, mn, f, mr, at, pn, pr = _zogy_inputs(case, seed)
    H, W = n.shape
    L, r = case["L"], case["r"]
    Fn, Fr, sn, sr = ZOGY_SCALARS

    def hat(P):
        big = torch.zeros((L, L), device="cuda", dtype=torch.float64)
        big[:2 * r + 1, :2 * r + 1] = _dev(P).double()
        return torch.fft.fft2(big.roll((-r, -r), (0, 1)))

    Pn, Pr = hat(pn), hat(pr)
    den = (sn ** 2 * Fr ** 2 * Pr.abs() ** 2 + sr ** 2 * Fn ** 2 * Pn.abs() ** 2).sqrt()
    FD = Fn * Fr / math.sqrt(sn ** 2 * Fr ** 2 + sr ** 2 * Fn ** 2)
    PD = Fr * Fn * Pr * Pn / (FD * den)
    pd2 = (PD.abs() ** 2).sum() / L ** 2
    bad = (mn != 0) | (mr != 0)
    big = []
    for t, fill in ((torch.where(bad, 0.0, n), 0.0), (torch.where(bad, 0.0, f), 0.0), (bad, True)):
        big.append(torch.nn.functional.pad(t, (0, L, 0, L), value=fill))
    out = {k: torch.zeros((len(at), L, L), device="cuda", dtype=torch.float64)
           for k in ("D", "snr", "flux")}
    for t, (x, y) in enumerate(at.tolist()):
        N, R, B = (p[y:y + L, x:x + L] for p in big)
        Dh = (Fr * Pr * torch.fft.fft2(N.double()) - Fn * Pn * torch.fft.fft2(R.double())) / den
        flag = B.clone()
        for axis in (0, 1):
            one = flag.clone()
            for k in range(1, 2 * r + 1):
                lo, hi = one.narrow(axis, 0, L - k), one.narrow(axis, k, L - k)
                flag.narrow(axis, k, L - k).logical_or_(lo)
                flag.narrow(axis, 0, L - k).logical_or_(hi)
        flag[:r] = flag[L - r:] = True
        flag[:, :r] = flag[:, L - r:] = True
        S = torch.fft.ifft2(Dh * PD.conj()).real
        for k, v in (("D", torch.fft.ifft2(Dh).real), ("snr", S / pd2.sqrt()),
                     ("flux", S / (FD * pd2))):
            out[k][t] = torch.where(flag, 0.0, v)
    return {**out, "mask": None, "pd2": pd2.view(1)}


def _exact_batch(case, seed):
    planes = _pair(case, seed)
    x0, y0, side = _cutouts(case, seed)
    parts = {"coeffs": [], "chi2": [], "diff": [], "diff_var": []}
    for x, y, L in zip(x0.tolist(), y0.tolist(), side.tolist()):
        a, d, v, chi2 = _difference64([p[y:y + L, x:x + L] for p in planes], case["h"], 0)
        for k, t in zip(parts, (a[None], chi2.view(1), d.reshape(-1), v.reshape(-1))):
            parts[k].append(t)
    return {**{k: torch.cat(v) for k, v in parts.items()},
            **dict.fromkeys(("diff_mask", "det_mask", "n_fit", "status", "n_cands"))}
