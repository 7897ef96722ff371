"""The work that a user has the spot fitter do, as cases that can be timed and checked.

A case is a dict of plain values:
  path      the calls of one pass:
            "fit"       spotfit_fit_spots on a batch in device memory
            "raw"       spotfit_fit_raw: pixels in, start values and fits out
            "protocol"  the paper's accuracy runs: brightest-pixel start values, the fit from
                        them with its evaluation counts, and the stop statistics
            "graph"     a captured fit of one camera frame with its copies from and to the host
            "serve"     one camera frame through the serving loop, host arrays in and out
  n         spots
  sides     the ROI sides that occur, "7,9,11" or "7-32"; one of them, at random, per spot
  rect      width and height drawn apart (else square)
  model     "sym", "ell" or "both" (half and half)
  dtype     pixels, "u16" or "f32"
  schedule  "uniform" or "mixed" (size classes), plan "throughput" or "latency"
  sigma_lo, sigma_hi, alpha_lo, alpha_hi, alpha_log, beta_lo, beta_hi, read_sd
            the laws of the spots: width, peak, background, sd of the read noise

Pixels are seeded draws: centre within one pixel of the ROI centre, counts point-sampled at the
pixel centres, Poisson noise plus read noise, rounded to whole counts for 16-bit data.  Start values
are the moment estimate a camera pipeline hands on.
"""
import math

import numpy as np
import torch

import paper_2106_02045_amd as sf

DEV = "cuda:0"

#: laws of the spots (the named workloads of this repository's generator)
BRIGHT = dict(sigma_lo=1.0, sigma_hi=3.0, alpha_lo=100.0, alpha_hi=10000.0, alpha_log=True,
              beta_lo=10.0, beta_hi=200.0, read_sd=2.0)
DIM = dict(sigma_lo=1.5, sigma_hi=6.0, alpha_lo=50.0, alpha_hi=300.0, alpha_log=False,
           beta_lo=200.0, beta_hi=1000.0, read_sd=0.0)
SMALL = dict(sigma_lo=1.2, sigma_hi=2.0, alpha_lo=500.0, alpha_hi=2000.0, alpha_log=False,
             beta_lo=100.0, beta_hi=100.0, read_sd=0.0)
MARKER = dict(sigma_lo=1.5, sigma_hi=2.5, alpha_lo=1000.0, alpha_hi=5000.0, alpha_log=False,
              beta_lo=150.0, beta_hi=150.0, read_sd=0.0)
LAWS = {"bright": BRIGHT, "dim": DIM, "small": SMALL, "marker": MARKER}


def _case(path, n, sides, model, law, *, rect=False, dtype="u16", schedule="uniform",
          plan="throughput", name=None):
    c = dict(path=path, n=int(n), sides=sides, rect=rect, model=model, dtype=dtype,
             schedule=schedule, plan=plan, **LAWS[law])
    if name is not None:
        c["name"] = name
    return c


def listed():
    """Cases from one camera frame to batches of millions of spots."""
    return [
        # fixed ROIs around 32 fiducial markers: the frame that is replayed at the camera's rate
        _case("graph", 32, "13", "sym", "marker", plan="latency", name="graph_markers_13x13"),
        # one camera frame of the serving loop: host pixels in, fits back on the host
        _case("serve", 110, "9,13,17,21", "sym", "marker", schedule="mixed", plan="latency",
              name="serve_frame"),
        # a burst of frames already on the device, fitted straight from their pixels
        _case("raw", 4000, "9,13,17,21", "sym", "marker", schedule="mixed", plan="latency",
              name="raw_frames_9to21"),
        # the smallest batch workload
        _case("fit", 1024, "11", "sym", "small", name="fit_small_11x11"),
        # an ordinary analysis batch of uneven, also non-square ROIs
        _case("fit", 10007, "7-32", "both", "bright", rect=True, schedule="mixed",
              name="fit_ragged_7to32"),
        # the paper's timing sweep at its largest batch
        _case("fit", 10000, "21", "sym", "bright", name="fit_sweep_21x21"),
        # the paper's accuracy protocol: its own start values, evaluation counts, statistics
        _case("protocol", 100000, "9", "sym", "small", name="protocol_9x9"),
        # float pixels (flat-fielded images), elliptical spots
        _case("fit", 200000, "17", "ell", "bright", dtype="f32", name="fit_float_17x17_ell"),
        # the benchmark's batch
        _case("fit", 1000000, "15", "sym", "bright", name="fit_scale_15x15"),
        # the same batch from its pixels alone
        _case("raw", 1000000, "15", "sym", "bright", name="raw_scale_15x15"),
        # the largest spots
        _case("fit", 500000, "32", "ell", "dim", name="fit_precision_32x32_ell"),
        # the largest batch: uneven sizes in one call
        _case("fit", 2000000, "7,9,11,15,21,25,32", "both", "bright", schedule="mixed",
              name="fit_mixed_7to32"),
    ]


#: pixels of the largest listed case, which no drawn case exceeds
_MOST_PIXELS = 500_000_000


def draw(rng):
    """One more case: a path, a size of batch and ROI, and the options it is used with."""
    path = rng.choice(["graph", "serve", "raw", "raw", "fit", "fit", "fit", "fit", "protocol"])
    law = rng.choice(["bright", "bright", "dim", "marker"])
    lo, hi = {"graph": (8, 256), "serve": (20, 200), "raw": (64, 500000), "fit": (64, 1000000),
              "protocol": (1000, 200000)}[path]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    a = rng.randint(7, 32)
    if path == "serve":
        sides, law = rng.choice(["9,13,17,21", "9-21", "7,11,15"]), "marker"
    elif path == "graph":
        sides, law = str(rng.randint(9, 21)), "marker"
    elif path == "protocol":
        sides, law = str(rng.randint(7, 15)), rng.choice(["small", "bright"])
    elif rng.random() < 0.5:
        sides = str(a)
    else:
        b = rng.randint(7, 32)
        sides = "%d-%d" % (min(a, b), max(a, b))
    if law == "dim" and min(_sides(sides)) < 16:
        law = "bright"
    most = int(_MOST_PIXELS / max(_sides(sides)) ** 2)
    uneven = len(_sides(sides)) > 1
    return _case(path, min(n, most), sides,
                 "sym" if path in ("graph", "serve", "protocol") else rng.choice(["sym", "ell", "both"]),
                 law, rect=uneven and path not in ("graph", "serve") and rng.random() < 0.4,
                 dtype="f32" if path in ("fit", "raw") and rng.random() < 0.2 else "u16",
                 schedule="mixed" if uneven else "uniform",
                 plan="latency" if path in ("graph", "serve") or (n <= 20000 and rng.random() < 0.4)
                 else "throughput")


# ---------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------

def _sides(text):
    if "-" in text:
        lo, hi = text.split("-")
        return list(range(int(lo), int(hi) + 1))
    return [int(t) for t in text.split(",")]


def _chunks(n, side):
    step = max(1, (1 << 26) // (side * side))
    return [(i, min(n, i + step)) for i in range(0, n, step)]


def _shapes(case, seed):
    """(w, h, model, offsets, generator) of the case's spots, on the GPU."""
    g = torch.Generator(DEV)
    g.manual_seed(int(seed))
    n, sides = case["n"], torch.tensor(_sides(case["sides"]), device=DEV)
    pick = lambda: sides[torch.randint(0, len(sides), (n,), generator=g, device=DEV)]
    w = pick()
    h = pick() if case["rect"] else w
    if case["model"] == "both":
        model = torch.randint(0, 2, (n,), generator=g, device=DEV)
    else:
        model = torch.full((n,), int(case["model"] == "ell"), device=DEV)
    offsets = torch.zeros(n, dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(w * h, 0)[:-1]
    return w, h, model, offsets, g


def _grid(w, h, shape=None):
    """Column and row numbers of the padded images, and which pixels lie inside."""
    H, W = shape or (int(h.max()), int(w.max()))
    xs = torch.arange(W, device=DEV, dtype=torch.float64)
    ys = torch.arange(H, device=DEV, dtype=torch.float64)
    inx = (xs[None, :] < w[:, None])
    iny = (ys[None, :] < h[:, None])
    return xs, ys, inx, iny


def _moment_start(img, w, h, model):
    """Centroid / second-moment start values of padded images [m, H, W] in 64 bits."""
    m = img.shape[0]
    k = torch.arange(int((2 * (w + h - 2)).max()), device=DEV)[None, :]
    W, H = w[:, None], h[:, None]
    nr = 2 * (W + H - 2)
    side = torch.clamp(k - 2 * W, min=0)
    top, bottom, left = k < W, k < 2 * W, k < 2 * W + H - 2
    r = torch.where(top, 0 * k, torch.where(bottom, H - 1, torch.where(left, side + 1, side - (H - 2) + 1)))
    c = torch.where(top, k, torch.where(bottom, k - W, torch.where(left, 0 * k, W - 1)))
    ok = k < nr
    flat = torch.where(ok, r, 0 * r) * img.shape[2] + torch.where(ok, c, 0 * c)
    ring = img.reshape(m, -1).gather(1, flat)
    ring = torch.where(ok, ring, torch.full_like(ring, math.inf)).sort(1).values
    half = (w + h - 2)[:, None]
    b0 = 0.5 * (ring.gather(1, half - 1) + ring.gather(1, half))[:, 0]
    xs, ys, inx, iny = _grid(w, h)
    wt = (img - b0[:, None, None]).clamp(min=0) * (iny[:, :, None] & inx[:, None, :])
    col, row = wt.sum(1), wt.sum(2)
    sw = col.sum(1)
    some = sw > 0
    s1 = torch.where(some, sw, torch.ones_like(sw))
    cx, cy = (col * xs).sum(1) / s1, (row * ys).sum(1) / s1
    vx = (col * (xs - cx[:, None]) ** 2).sum(1) / s1
    vy = (row * (ys - cy[:, None]) ** 2).sum(1) / s1
    sym = model == 0
    sx = torch.where(sym, 0.5 * (vx + vy), vx).sqrt()
    sy = torch.where(sym, 0.5 * (vx + vy), vy).sqrt()
    top = torch.maximum(w, h).double() / 4
    sx, sy = (torch.minimum(s.clamp(min=0.8), top) for s in (sx, sy))
    flat0 = torch.stack([(w - 1) / 2, (h - 1) / 2, 0 * sw + 1.5, 0 * sw + 1.5], 1).double()
    return torch.where(some[:, None], torch.stack([cx, cy, sx, sy], 1), flat0)


def _render(case, w, h, model, g):
    """Padded noisy images [m, H, W] (float64) of freshly drawn spots."""
    m = w.shape[0]
    u = lambda lo, hi, *s: lo + (hi - lo) * torch.rand(*s, generator=g, device=DEV, dtype=torch.float64)
    x, y = (w - 1) / 2 + u(-1, 1, m), (h - 1) / 2 + u(-1, 1, m)
    sx, sy = u(case["sigma_lo"], case["sigma_hi"], m), u(case["sigma_lo"], case["sigma_hi"], m)
    sy = torch.where(model == 0, sx, sy)
    if case["alpha_log"]:
        alpha = u(math.log(case["alpha_lo"]), math.log(case["alpha_hi"]), m).exp()
    else:
        alpha = u(case["alpha_lo"], case["alpha_hi"], m)
    beta = u(case["beta_lo"], case["beta_hi"], m)
    xs, ys, inx, iny = _grid(w, h)
    ex = torch.exp(-0.5 * ((xs - x[:, None]) / sx[:, None]) ** 2)
    ey = torch.exp(-0.5 * ((ys - y[:, None]) / sy[:, None]) ** 2) * alpha[:, None]
    rate = (ey[:, :, None] * ex[:, None, :] + beta[:, None, None]).float()
    img = torch.poisson(rate, generator=g)
    if case["read_sd"] > 0:
        img += case["read_sd"] * torch.randn(img.shape, generator=g, device=DEV)
    if case["dtype"] == "u16":
        img = img.round_().clamp_(0, 65535)
    else:
        img = img * 1.03125  # flat-fielded: no whole counts any more
    inside = iny[:, :, None] & inx[:, None, :]
    return img.double() * inside, inside


def _inputs(case, seed):
    """data, sizes, offsets, init of the case's spots, on the GPU."""
    w, h, model, offsets, g = _shapes(case, seed)
    n, side = case["n"], int(max(w.max(), h.max()))
    total = int((w * h).sum())
    u16 = case["dtype"] == "u16"
    data = torch.empty(total, dtype=torch.int16 if u16 else torch.float32, device=DEV)
    init = torch.empty((n, 4), dtype=torch.float32, device=DEV)
    at = 0
    for a, b in _chunks(n, side):
        img, inside = _render(case, w[a:b], h[a:b], model[a:b], g)
        px = img[inside]
        data[at:at + px.numel()] = px.to(torch.int32).to(torch.int16) if u16 else px.float()
        at += px.numel()
        if case["path"] in ("fit", "graph", "serve"):
            init[a:b] = _moment_start(img, w[a:b], h[a:b], model[a:b]).float()
        del img, inside, px
    sizes = torch.stack([w, h, model, 0 * w], 1).to(torch.uint8).contiguous()
    return (data.view(torch.uint16) if u16 else data), sizes, offsets, init


def _options(case):
    sides = _sides(case["sides"])
    return sf.default_options(
        max_side=max(sides), max_pixels=max(sides) ** 2,
        schedule=sf.SCHEDULE_MIXED if case["schedule"] == "mixed" else sf.SCHEDULE_UNIFORM,
        plan_hint=sf.PLAN_LATENCY if case["plan"] == "latency" else sf.PLAN_THROUGHPUT)


_context = []


def _ctx(n):
    """The program's one context, sized for its largest batch."""
    if not _context:
        _context.append(sf.Context(0))
    _context[0].reserve(n)
    return _context[0]


def prepare(case, seed):
    data, sizes, offsets, init = _inputs(case, seed)
    n, path, opts = case["n"], case["path"], _options(case)
    s = dict(path=path, opts=opts)
    f32 = lambda *shape: torch.empty(shape, dtype=torch.float32, device=DEV)
    i32 = lambda *shape: torch.empty(shape, dtype=torch.int32, device=DEV)
    if path == "serve":
        # host arrays, and a server that lives as long as the program
        s["server"] = sf.Server(0, opts, device_mem_budget=16 << 20, max_frames=64, n_streams=2)
        s["frame"] = (data.view(torch.int16).cpu().numpy().view(np.uint16), sizes.cpu().numpy(),
                      init.cpu().numpy())
        return s
    s.update(ctx=_ctx(n), data=data, sizes=sizes, offsets=offsets, init=init)
    s["out"] = dict(params=f32(n, 6), chi2=f32(n), iters=i32(n), status=i32(n))
    if path == "raw":
        s["out"]["init"] = init
    elif path == "protocol":
        s["out"]["evals"] = i32(n, 2)
    elif path == "graph":
        pin = lambda t: torch.empty(t.shape, dtype=t.dtype).pin_memory()
        host = {k: pin(v) for k, v in dict(s["out"], data=data, init=init).items()}
        host["data"].view(torch.int16).copy_(data.view(torch.int16))
        host["init"].copy_(init)
        s["host"] = host
        s["graph"] = s["ctx"].graph(data, sizes, offsets, init, opts, out=s["out"], host=host)
    return s


def run(s):
    path = s["path"]
    if path == "serve":
        ticket, out = s["server"].submit(*s["frame"])
        return s["server"].wait(ticket)
    if path == "graph":
        s["graph"].launch()
        return {k: s["host"][k] for k in ("params", "chi2", "iters", "status")}
    ctx, d = s["ctx"], (s["data"], s["sizes"], s["offsets"])
    if path == "raw":
        return ctx.fit_raw(*d, s["opts"], out=s["out"])
    if path == "protocol":
        ctx.peak_init(*d, s["opts"], out=s["init"])
        out = ctx.fit_spots(*d, s["init"], s["opts"], out=s["out"])
        stats = {k: np.asarray(v) for k, v in ctx.stats(out).items()}
        return dict(out, init=s["init"], stats=stats)
    return ctx.fit_spots(*d, s["init"], s["opts"], out=s["out"])


def work(case):
    """Pixels, records and results once; two multiply-adds per pixel (the sums over rows and over
    columns) and one exponential per row and column for each of four evaluations of a fit."""
    sides = np.array(_sides(case["sides"]), dtype=np.float64)
    n = case["n"]
    npx = n * (sides.mean() ** 2 if case["rect"] else (sides ** 2).mean())
    size = 2 if case["dtype"] == "u16" else 4
    flops = 4 * (4.0 * npx + 20.0 * n * 2 * sides.mean())
    if case["path"] in ("raw", "protocol"):
        flops += 8.0 * npx
    return {"bytes": npx * size + n * (12 + 16 + 36), "flops": flops}


# ---------------------------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------------------------

def _peak_start(img, w, h):
    """Brightest pixel of the 3 x 3 moving average, sigma from the area above exp(-1/2)."""
    m, H, W = img.shape
    xs, ys, inx, iny = _grid(w, h)
    inside = iny[:, :, None] & inx[:, None, :]
    p = torch.nn.functional.pad(img, (1, 1, 1, 1))
    q = torch.nn.functional.pad(inside.double(), (1, 1, 1, 1))
    acc, cnt = torch.zeros_like(img), torch.zeros_like(img)
    for a in range(3):
        for b in range(3):
            acc += p[:, a:a + H, b:b + W]
            cnt += q[:, a:a + H, b:b + W]
    mean = torch.where(inside, acc / cnt.clamp(min=1), torch.full_like(acc, -math.inf)).reshape(m, -1)
    k = torch.arange(H * W, device=DEV)[None, :]
    first = torch.where(mean == mean.max(1, keepdim=True).values, k, H * W).min(1).values
    inf = torch.full_like(img, math.inf)
    lo = torch.where(inside, img, inf).amin((1, 2))
    hi = torch.where(inside, img, -inf).amax((1, 2))
    thr = (hi - lo) * math.exp(-0.5) + lo
    area = ((img > thr[:, None, None]) & inside).sum((1, 2)).double()
    s = (area / math.pi).sqrt().clamp(min=0.5)
    return torch.stack([(first % W).double(), (first // W).double(), s, s], 1)


def _model(img, w, h, p):
    """Amplitudes and error (Eqs. 2, 5, 6) and the pieces that the derivatives need."""
    xs, ys, inx, iny = _grid(w, h, img.shape[1:])
    dx, dy = xs - p[:, 0:1], ys - p[:, 1:2]
    ex = torch.exp(-0.5 * (dx / p[:, 2:3]) ** 2) * inx
    ey = torch.exp(-0.5 * (dy / p[:, 3:4]) ** 2) * iny
    N = (w * h).double()
    row = (img * ex[:, None, :]).sum(2)
    F = ex.sum(1) * ey.sum(1)
    FF = (ex * ex).sum(1) * (ey * ey).sum(1)
    G = img.sum((1, 2))
    FG = (row * ey).sum(1)
    D = N * FF - F * F
    a = (N * FG - F * G) / D
    b = (G * FF - F * FG) / D
    res = (a[:, None] * ey)[:, :, None] * ex[:, None, :]
    res += b[:, None, None]
    res -= img
    res *= iny[:, :, None]
    res *= inx[:, None, :]
    chi = res.square_().sum((1, 2))
    bad = ~((D > 0) & torch.isfinite(D) & torch.isfinite(chi) & torch.isfinite(a) & torch.isfinite(b))
    nan = torch.full_like(chi, math.nan)
    a, b, chi = (torch.where(bad, nan, v) for v in (a, b, chi))
    return a, b, chi, (dx, dy, ex, ey, N, row, F, FF, G, FG, D)


def _normal(img, model, p, a, b, parts):
    """J^T J and J^T (g - h) (Eqs. 7-9, 11) as 4 x 4 and 4, the symmetric model contracted."""
    dx, dy, ex, ey, N, row, F, FF, G, FG, D = parts
    col = (img * ey[:, :, None]).sum(1)
    X = [(dx ** k * ex * ex).sum(1) for k in range(5)]
    Y = [(dy ** k * ey * ey).sum(1) for k in range(5)]
    X1 = [(dx ** k * ex).sum(1) for k in range(3)]
    Y1 = [(dy ** k * ey).sum(1) for k in range(3)]
    sx, sy = p[:, 2], p[:, 3]
    wt = [sx ** -2, sy ** -2, sx ** -3, sy ** -3]
    ox, oy = (1, 0, 2, 0), (0, 1, 0, 2)
    gx = [(dx ** k * ex * col).sum(1) for k in range(3)]
    gy = [(dy ** k * ey * row).sum(1) for k in range(3)]
    dF = [wt[j] * X1[ox[j]] * Y1[oy[j]] for j in range(4)]
    fd = [wt[j] * X[ox[j]] * Y[oy[j]] for j in range(4)]
    gd = [wt[j] * (gx[ox[j]] if ox[j] else gy[oy[j]]) for j in range(4)]
    dd = [[wt[i] * wt[j] * X[ox[i] + ox[j]] * Y[oy[i] + oy[j]] for j in range(4)] for i in range(4)]
    sym = model == 0
    if bool(sym.any()):
        z = torch.zeros_like(F)
        fold = lambda v: [v[0], v[1], torch.where(sym, v[2] + v[3], v[2]), torch.where(sym, z, v[3])]
        dF, fd, gd = fold(dF), fold(fd), fold(gd)
        dd = [fold(r) for r in dd]
        dd = [dd[0], dd[1], [torch.where(sym, u + v, u) for u, v in zip(dd[2], dd[3])],
              [torch.where(sym, z, v) for v in dd[3]]]
    gam = [N * 2 * fd[j] - 2 * F * dF[j] for j in range(4)]
    da = [(N * gd[j] - G * dF[j] - a * gam[j]) / D for j in range(4)]
    db = [(2 * G * fd[j] - FG * dF[j] - F * gd[j] - b * gam[j]) / D for j in range(4)]
    A = [[da[i] * da[j] * FF + a * (da[i] * fd[j] + da[j] * fd[i]) + a * a * dd[i][j]
          + db[j] * (da[i] * F + a * dF[i]) + db[i] * (da[j] * F + a * dF[j]) + N * db[i] * db[j]
          for j in range(4)] for i in range(4)]
    v = [a * (gd[j] - a * fd[j] - b * dF[j]) for j in range(4)]
    one = torch.ones_like(F)
    A[3][3] = torch.where(sym, one, A[3][3])
    return torch.stack([torch.stack(r, 1) for r in A], 1), torch.stack(v, 1)


def _solve(A, v, k):
    """(A + 10^k diag A) delta = v (Eq. 14) by elimination; NaN where A is not positive definite."""
    lam = 10.0 ** k.double()
    M = [[A[:, i, j] * (1 + lam) if i == j else A[:, i, j] for j in range(4)] for i in range(4)]
    y = [v[:, i] for i in range(4)]
    ok = torch.ones_like(lam, dtype=torch.bool)
    for i in range(4):
        ok &= (M[i][i] > 0) & torch.isfinite(M[i][i])
        for r in range(i + 1, 4):
            f = M[r][i] / M[i][i]
            M[r] = [M[r][c] - f * M[i][c] if c > i else M[r][c] for c in range(4)]
            y[r] = y[r] - f * y[i]
    d = [None] * 4
    for i in (3, 2, 1, 0):
        t = y[i]
        for c in range(i + 1, 4):
            t = t - M[i][c] * d[c]
        d[i] = t / M[i][i]
    d = torch.stack(d, 1)
    return torch.where((ok & torch.isfinite(d).all(1))[:, None], d, torch.full_like(d, math.nan))


def _fit64(img, w, h, model, p):
    """The Fit2DGaussian loop on padded images, every spot at its own step: params [m, 6], chi^2."""
    m = img.shape[0]
    params = torch.full((m, 6), math.nan, dtype=torch.float64, device=DEV)
    chi2 = torch.full((m,), math.nan, dtype=torch.float64, device=DEV)
    sym = model == 0
    p = torch.where(sym[:, None], torch.stack([p[:, 0], p[:, 1], p[:, 2], p[:, 2]], 1), p)
    who = torch.arange(m, device=DEV)
    T = (w * h).double() / 3
    org = torch.stack([(w - 1) / 2, (h - 1) / 2, 0 * T, 0 * T], 1).double()
    smax = torch.maximum(w, h).double()

    def put(which, p, a, b, chi):
        params[who[which]] = torch.cat([p[which], a[which, None], b[which, None]], 1)
        chi2[who[which]] = chi[which]

    def trial(best, A, v, k):
        d = _solve(A, v, k)
        d = torch.where((model == 0)[:, None], torch.stack([d[:, 0], d[:, 1], d[:, 2], d[:, 2]], 1), d)
        q = best + d
        q = torch.stack([torch.minimum(q[:, 0].clamp(min=-0.5), w - 0.5),
                         torch.minimum(q[:, 1].clamp(min=-0.5), h - 0.5),
                         torch.minimum(q[:, 2].clamp(min=0.3), smax),
                         torch.minimum(q[:, 3].clamp(min=0.3), smax)], 1)
        return q, d

    a, b, chi, parts = _model(img, w, h, p)
    A, v = _normal(img, model, p, a, b, parts)
    k = torch.full((m,), -2, device=DEV)
    it = torch.ones(m, dtype=torch.int64, device=DEV)
    live = ~(torch.isnan(chi) | (chi < T))
    put(~live, p, a, b, chi)
    state = [img, w, h, model, who, T, org, smax, p, a, b, chi, A, v, k, it,
             torch.ones(m, dtype=torch.bool, device=DEV)]
    while bool(live.any()):
        state = [t[live] for t in state]
        img, w, h, model, who, T, org, smax, best, a0, b0, chi, A, v, k, it, first = state
        q, d = trial(best, A, v, k)
        a, b, Chi, parts = _model(img, w, h, q)
        k = torch.where(first & (Chi < chi), k - 1, k)
        small = (d.abs() < 1e-4 * (best - org).abs()).all(1)
        retry = ~small & (chi < Chi) & (k < 4)
        worse = ~retry & ((chi < Chi) | torch.isnan(Chi))
        stop = ~retry & ~worse & ((Chi < T) | (chi * (1.0 - 1e-6) < Chi) | small | (it >= 20))
        put(worse, best, a0, b0, chi)
        put(stop, q, a, b, Chi)
        go = ~retry & ~worse & ~stop
        An, vn = _normal(img, model, q, a, b, parts)
        sel = lambda x, y: torch.where(go.reshape([-1] + [1] * (x.dim() - 1)), x, y)
        state = [img, w, h, model, who, T, org, smax, sel(q, best), sel(a, a0), sel(b, b0),
                 sel(Chi, chi), sel(An, A), sel(vn, v), torch.where(retry, k + 1, k),
                 torch.where(go, it + 1, it), go]
        live = retry | go
    return params, chi2


def exact(case, seed):
    data, sizes, offsets, init = _inputs(case, seed)
    n = case["n"]
    w, h, model = (sizes[:, i].long() for i in range(3))
    side = int(max(w.max(), h.max()))
    params = torch.empty((n, 6), dtype=torch.float64, device=DEV)
    chi2 = torch.empty(n, dtype=torch.float64, device=DEV)
    start = init.double()
    step = max(1, (1 << 25) // (side * side))
    for a in range(0, n, step):
        b = min(n, a + step)
        W, H, M = w[a:b], h[a:b], model[a:b]
        xs, ys, inx, iny = _grid(W, H)
        inside = iny[:, :, None] & inx[:, None, :]
        img = torch.zeros(inside.shape, dtype=torch.float64, device=DEV)
        o = int(offsets[a])
        px = data[o:o + int((W * H).sum())]
        px = (px.view(torch.int16).to(torch.int32) & 0xFFFF) if case["dtype"] == "u16" else px
        img[inside] = px.double()
        if case["path"] == "raw":
            start[a:b] = _moment_start(img, W, H, M)
        elif case["path"] == "protocol":
            start[a:b] = _peak_start(img, W, H)
        params[a:b], chi2[a:b] = _fit64(img, W, H, M, start[a:b].float().double())
    out = dict(params=params, chi2=chi2, iters=None, status=None)
    if case["path"] in ("raw", "protocol"):
        out["init"] = start
    return out
