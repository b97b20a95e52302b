"""The work that programs built on this library have it do, as cases to be timed.

A case is one call sequence on one problem: a solve of a few tens of outer
iterations from a starting point (CT, seismic, radiotherapy and dense
problems, one slice or several slices sharing an operator, float32 or bf16
storage of A), a single feasibility step, or a query of the proximity and the
objective.  Sizes follow the repository's configurations (the dense 256 x 128
system, CT of 64^2 to 256^2 pixels with 8 and 32 slices, Fresnel-zone
seismic rows with DROP and L1, radiotherapy beamlets up to 19,881 columns,
dose-volume plans), scaled so that an operator is made in a second or two.

Every input is generated on the GPU from the case and a seed: the operator's
geometry (the first gantry angle, the wavelength), the phantom, the noise of
the data and the starting point.  Solves start near the solution with noise,
as a warm start does, so that perturbations of every kind act on them.

    listed()             the cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, operator, problem (and tuned launch shapes)
    run(state)           one pass through the public entry points
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the same result in float64, in plain torch
"""
import math

import numpy as np
import torch

import paper_2606_27086_amd as smx

DEV = "cuda"
F64 = torch.float64

OBJ = {"none": smx.OBJ_NONE, "sqnorm": smx.OBJ_SQNORM, "tv": smx.OBJ_TV2D, "linear": smx.OBJ_LINEAR, "l1": smx.OBJ_L1}
BASIC = {"simult": smx.BASIC_SIMULT, "drop": smx.BASIC_DROP, "cq": smx.BASIC_CQ, "el": smx.BASIC_EL,
         "emr": smx.BASIC_EMR}


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def _dense(**kw):
    return dict(kind="dense", call="solve", m=256, n=128, B=1, storage="f32", obj="sqnorm", basic="simult", K=40,
                tuned=False, **kw)


def _ct(rows, cols, angles, dets, **kw):
    c = dict(kind="ct", call="solve", rows=rows, cols=cols, angles=angles, dets=dets, B=1, storage="f32", obj="tv",
             basic="simult", K=20, tuned=True)
    c.update(kw)
    return c


def _seismic(N, sources, receivers, **kw):
    c = dict(kind="seismic", call="solve", N=N, sources=sources, receivers=receivers, B=1, storage="f32", obj="l1",
             basic="drop", K=20, tuned=True)
    c.update(kw)
    return c


def _rt(X, Y, Z, beams, nu, nw, **kw):
    c = dict(kind="rt", call="solve", X=X, Y=Y, Z=Z, beams=beams, nu=nu, nw=nw, B=1, storage="f32", obj="linear",
             basic="simult", K=20, tuned=True, dvc=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest solve: a dense consistent system, where launches and latency are all there is
        dict(_dense(), name="dense_256x128"),
        # one feasibility step on a small plan, as an outer loop of the caller's own makes it (no graph)
        dict(_rt(20, 18, 12, 9, 6, 6, call="step", obj="none", K=1, tuned=False), name="rt_small_step"),
        # proximity and objective of a given image: what a caller's stopping test or line search asks for
        dict(_ct(128, 128, 120, 182, call="query", K=1, tuned=False), name="ct128_query"),
        # a small CT slice (a preview, or a low-resolution level)
        dict(_ct(64, 64, 60, 91, K=40), name="ct64_tv"),
        # the ordinary CT slice: 180 angles x 363 detectors, TV
        dict(_ct(256, 256, 180, 363), name="ct256_tv"),
        # a ragged image in bf16 with the low-dose CT experiment's step and perturbation (EMR, four reductions)
        dict(_ct(187, 171, 101, 257, storage="bf16", basic="emr", gamma=5.0, n_red=4, restart_every=50),
             name="ct187x171_emr_bf16"),
        # several slices of one scan: 8 right-hand sides on one operator
        dict(_ct(128, 128, 180, 182, B=8), name="ct128_batch8"),
        # the solve server's group: 32 slots, bf16 operator, no refinement
        dict(_ct(256, 256, 180, 363, B=32, storage="bf16", refine=0), name="ct256_batch32_bf16"),
        # seismic tomography with Fresnel-zone rows: DROP, L1, four reductions a phase
        dict(_seismic(128, 48, 96, gamma=1.0, alpha=0.975, n_red=4, restart_every=50), name="seismic128_l1"),
        # radiotherapy at the full beamlet count, float32: the largest
        dict(_rt(112, 112, 56, 9, 47, 47), name="rt_19881_f32"),
        # an odd-sized plan in bf16 (the last iteration on the float32 copy, the default)
        dict(_rt(71, 67, 31, 7, 29, 31, storage="bf16"), name="rt_6293_bf16"),
        # a plan with dose-volume constraints (target D95, D5 and organ D5) under EMR
        dict(_rt(60, 60, 30, 9, 25, 25, basic="emr", dvc=True, gamma=1.0, alpha=0.7, restart_every=500),
             name="rt_5625_dose_volume"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dense", "ct", "ct", "ct_batch", "seismic", "rt", "rt", "rt_dvc", "rt_step", "ct_query"])
    storage = rng.choice(["f32", "f32", "bf16"])
    if kind == "dense":
        return dict(_dense(), m=_log_int(rng, 60, 700), n=_log_int(rng, 40, 400), K=rng.choice([20, 40, 60]))
    if kind == "ct":
        N = _log_int(rng, 48, 230)
        extra = {}
        if rng.random() < 0.3:
            extra = dict(basic=rng.choice(["emr", "drop", "el"]))
        if rng.random() < 0.3:
            extra.update(gamma=5.0, n_red=4, restart_every=50)
        return _ct(N, N + rng.randint(-9, 9), _log_int(rng, 40, 180), int(1.45 * N) + rng.randint(0, 5),
                   storage=storage, **extra)
    if kind == "ct_batch":
        N = _log_int(rng, 48, 150)
        B = rng.choice([2, 4, 8, 16, 32])
        return _ct(N, N + rng.randint(-9, 9), _log_int(rng, 60, 180), int(1.45 * N) + rng.randint(0, 5), B=B,
                   storage=storage, **(dict(refine=0) if storage != "f32" else {}))
    if kind == "seismic":
        N = _log_int(rng, 48, 140)
        return _seismic(N, rng.randint(16, 50), 2 * rng.randint(10, 48), obj=rng.choice(["l1", "sqnorm", "tv"]),
                        storage=storage, gamma=1.0, alpha=0.975, n_red=4, restart_every=50)
    if kind == "ct_query":
        N = _log_int(rng, 48, 200)
        return _ct(N, N + rng.randint(-9, 9), _log_int(rng, 40, 150), int(1.45 * N), call="query", K=1, tuned=False)
    if kind == "rt_step":
        s = _log_int(rng, 14, 40)
        b = rng.randint(5, 14)
        return _rt(s, s + rng.randint(-3, 3), max(6, s // 2), 9, b, b, call="step", obj="none", K=1, tuned=False,
                   storage=storage, basic=rng.choice(["simult", "cq", "drop"]))
    s = _log_int(rng, 24, 76)
    b = _log_int(rng, 8, 45)
    plan = _rt(s, s + rng.randint(-5, 5), max(8, s // 2 + rng.randint(-4, 4)), rng.choice([5, 7, 9]), b,
               b + rng.randint(-2, 2), storage=storage)
    if kind == "rt_dvc":
        plan.update(X=min(plan["X"], 60), Y=min(plan["Y"], 60), Z=min(plan["Z"], 30), storage="f32",
                    basic=rng.choice(["emr", "simult"]), dvc=True, gamma=1.0, alpha=0.7, restart_every=500)
    return plan


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

class Inputs:
    """A (CSR, float32 values), bands, box, starting point and parameters."""


def _segment_sums(values, row_ptr):
    """Sums of consecutive runs of `values`, in order (the same on every run)."""
    return torch.segment_reduce(values, "sum", offsets=row_ptr, axis=0)


def _times(D, x):
    """A x in float64 for one column x."""
    return _segment_sums(D.val.to(F64) * x.to(F64)[D.col], D.ptr)


def _from_mask(parts, rows):
    """CSR from consecutive blocks of rows, each (mask, columns, values)."""
    counts = torch.cat([m.sum(1) for m, _, _ in parts])
    ptr = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(counts, 0)
    return ptr, torch.cat([c[m] for m, c, _ in parts]), torch.cat([v[m] for m, _, v in parts]).float()


def _ct_rows(R, C, angles, dets, first):
    """Exact ray-pixel intersection lengths of a parallel-beam scan."""
    h = 1.0 / max(R, C)
    off = (torch.arange(dets, device=DEV, dtype=F64) - (dets - 1) / 2) * h
    gx = (torch.arange(C + 1, device=DEV, dtype=F64) - C / 2) * h
    gy = (torch.arange(R + 1, device=DEV, dtype=F64) - R / 2) * h
    parts, step = [], max(1, 16384 // dets)
    for a0 in range(0, angles, step):
        th = first + torch.arange(a0, min(angles, a0 + step), device=DEV, dtype=F64) * (math.pi / angles)
        nx, ny = torch.cos(th)[:, None, None], torch.sin(th)[:, None, None]
        px, py, dx, dy = off[None, :, None] * nx + ny, off[None, :, None] * ny - nx, -ny, nx
        safe = lambda d: torch.where(d.abs() < 1e-9, torch.full_like(d, 1e-9), d)  # noqa: E731
        t = torch.cat([(gx - px) / safe(dx), (gy - py) / safe(dy)], 2).clamp_(0.0, 2.0).sort(2).values
        ln, mid = t[..., 1:] - t[..., :-1], 0.5 * (t[..., 1:] + t[..., :-1])
        j = torch.floor((px + mid * dx) / h + C / 2).long()
        i = torch.floor((py + mid * dy) / h + R / 2).long()
        ok = (ln > 1e-9) & (i >= 0) & (i < R) & (j >= 0) & (j < C)
        flat = lambda v: v.reshape(-1, v.shape[-1])  # noqa: E731
        parts.append((flat(ok), flat(i * C + j), flat(ln)))
    return _from_mask(parts, angles * dets)


def _fresnel_rows(N, sources, receivers, wavelength):
    """Rows of pixels in a band around each source-receiver segment (Gaussian
    across it, half-width sqrt(wavelength L t (1-t)) + 1/2), summing to L."""
    half = receivers // 2
    ys = (torch.arange(sources, device=DEV, dtype=F64) + 0.5) * N / sources
    lft = (torch.arange(half, device=DEV, dtype=F64) + 0.5) * N / half
    top = (torch.arange(receivers - half, device=DEV, dtype=F64) + 0.5) * N / (receivers - half)
    rx, ry = torch.cat([torch.zeros_like(lft), top]), torch.cat([lft, torch.zeros_like(top)])
    pix = torch.arange(N * N, device=DEV)
    cx, cy = (pix % N).to(F64) + 0.5, (pix // N).to(F64) + 0.5
    parts = []
    for a in range(sources):
        vx, vy = rx - N, ry - ys[a]
        L = torch.hypot(vx, vy)
        t = (((cx - N) * vx[:, None] + (cy - ys[a]) * vy[:, None]) / (L * L)[:, None]).clamp_(0.0, 1.0)
        d = torch.hypot(cx - (N + t * vx[:, None]), cy - (ys[a] + t * vy[:, None]))
        w = torch.sqrt(wavelength * L[:, None] * t * (1 - t)) + 0.5
        ok = d <= 2 * w
        om = torch.where(ok, torch.exp(-(d / w) ** 2), torch.zeros_like(d))
        parts.append((ok, pix.expand_as(ok), om * (L / om.sum(1))[:, None]))
    return _from_mask(parts, sources * receivers)


def _rt_rows(case, first):
    """Dose of each beamlet in each voxel: depth attenuation times lateral
    fall-off within a cutoff; scaled to a mean target dose of 1 at x = 1."""
    X, Y, Z, beams, nu, nw = (case[k] for k in ("X", "Y", "Z", "beams", "nu", "nw"))
    pos = [torch.arange(s, device=DEV, dtype=F64) + 0.5 - s / 2 for s in (X, Y, Z)]
    px, py, pz = (p.reshape(-1) for p in torch.meshgrid(*pos, indexing="ij"))
    su, sw = max(X, Y) / nu, Z / nw  # beamlet spacings covering the field
    reach = 4
    off = torch.arange(-reach, reach + 1, device=DEV)
    du, dw = (o.reshape(-1) for o in torch.meshgrid(off, off, indexing="ij"))
    parts = []
    for v0 in range(0, px.numel(), 16384):
        s = slice(v0, v0 + 16384)
        C, V = [], []
        for b in range(beams):
            th = first + 2 * math.pi * b / beams
            depth = px[s] * math.cos(th) + py[s] * math.sin(th) + 0.5 * max(X, Y)
            fu = (py[s] * math.cos(th) - px[s] * math.sin(th)) / su + (nu - 1) / 2
            fw = pz[s] / sw + (nw - 1) / 2
            bu, bw = torch.round(fu)[:, None].long() + du, torch.round(fw)[:, None].long() + dw
            r = torch.hypot(fu[:, None] - bu, fw[:, None] - bw)  # in beamlets
            ok = (bu >= 0) & (bu < nu) & (bw >= 0) & (bw < nw) & (r <= 6.4 / 2.4)
            C.append(torch.where(ok, b * nu * nw + bu * nw + bw, torch.full_like(bu, -1)))
            V.append(torch.exp(-0.005 * depth.clamp_min(0.0))[:, None] * torch.exp(-r * 1.2))
        C, V = torch.cat(C, 1), torch.cat(V, 1)
        parts.append((C >= 0, C, V))
    ptr, col, val = _from_mask(parts, px.numel())
    rad = 0.25 * min(X, Y, 2 * Z)
    target = torch.sqrt(px * px + py * py + pz * pz) <= rad
    organ = (torch.hypot(px - 1.1 * rad, py) <= 0.45 * rad) & (pz.abs() <= 0.8 * rad)
    mean = _segment_sums(val.to(F64), ptr)[target].mean()
    return ptr, col, (val.to(F64) / mean).float(), target, organ


def _take_rows(ptr, rows):
    """Entry positions of the given rows, in order, and their counts."""
    counts = ptr[rows + 1] - ptr[rows]
    start = torch.repeat_interleave(ptr[rows] - (torch.cumsum(counts, 0) - counts), counts)
    return start + torch.arange(int(counts.sum()), device=DEV), counts


def _phantom(R, C, g, n=10):
    y = (torch.arange(R, device=DEV, dtype=F64) + 0.5 - R / 2)[:, None] / max(R, C)
    x = (torch.arange(C, device=DEV, dtype=F64) + 0.5 - C / 2)[None, :] / max(R, C)
    img = torch.where((x / 0.45) ** 2 + (y / 0.38) ** 2 <= 1, 0.2, 0.0).to(F64)
    u = torch.rand(n, 7, generator=g, device=DEV, dtype=F64).cpu().numpy()
    for a, b, p, q, s, t, v in u:
        cx, cy = 0.35 * math.sqrt(a) * math.cos(6.283 * b), 0.35 * math.sqrt(a) * math.sin(6.283 * b)
        th = math.pi * p
        e = (x - cx) * math.cos(th) + (y - cy) * math.sin(th)
        f = -(x - cx) * math.sin(th) + (y - cy) * math.cos(th)
        img = torch.where((e / (0.03 + 0.22 * q)) ** 2 + (f / (0.03 + 0.22 * s)) ** 2 <= 1, v + 0 * t, img)
    return img.reshape(-1)


def _slowness(N, g):
    i = torch.arange(N, device=DEV, dtype=F64) + 0.5
    base = torch.tensor([1.0, 0.9, 0.8, 0.7, 0.6], device=DEV, dtype=F64)[((i / N) * 5).long().clamp_max(4)]
    u = torch.rand(4, 4, generator=g, device=DEV, dtype=F64).cpu().numpy()
    bump = torch.zeros(N, N, device=DEV, dtype=F64)
    for a, b, c, s in u:
        r2 = (i - N * a)[:, None] ** 2 + (i - N * b)[None, :] ** 2
        bump += (0.1 if s > 0.5 else -0.1) * torch.exp(-r2 / (2 * (0.04 * N + 0.08 * N * c) ** 2))
    return (base[:, None] * (1 + bump)).reshape(-1)


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rand = lambda *s: torch.rand(*s, generator=g, device=DEV, dtype=F64)  # noqa: E731
    randn = lambda *s: torch.randn(*s, generator=g, device=DEV, dtype=F64)  # noqa: E731
    jitter = float(rand(1))
    D = Inputs()
    D.B, D.image, D.dvc, D.c, D.lam = case["B"], None, None, None, 1.0
    D.hi = None
    if case["kind"] == "dense":
        m, D.n = case["m"], case["n"]
        D.ptr = torch.arange(0, m * D.n + 1, D.n, device=DEV)
        D.col = torch.arange(D.n, device=DEV).repeat(m)
        D.val = randn(m * D.n).float()
        r = _times(D, rand(D.n))[:, None]
        D.lower, D.upper = (r - 0.05).float(), (r + 0.05).float()
        D.hi, D.x0 = torch.ones(D.n, device=DEV), torch.full((D.n, 1), 0.5, device=DEV) + 0.1 * rand(D.n, 1).float()
    elif case["kind"] == "ct":
        R, C = case["rows"], case["cols"]
        D.n, D.image = R * C, (R, C)
        D.ptr, D.col, D.val = _ct_rows(R, C, case["angles"], case["dets"], 0.01 + jitter * math.pi / case["angles"])
        truth = torch.stack([_phantom(R, C, g) for _ in range(D.B)], 1)
        p = torch.stack([_times(D, truth[:, s]) for s in range(D.B)], 1)
        counts = torch.poisson(1e4 * torch.exp(-p), generator=g).clamp_min(1.0)
        b, sig = -torch.log(counts / 1e4), 3.0 / torch.sqrt(counts)
        D.lower, D.upper, D.hi = (b - sig).float(), (b + sig).float(), torch.ones(D.n, device=DEV)
        D.x0 = (truth + 0.05 + 0.05 * randn(D.n, D.B)).clamp(0.0, 1.0).float()
    elif case["kind"] == "seismic":
        N = case["N"]
        D.n, D.image = N * N, (N, N)
        D.ptr, D.col, D.val = _fresnel_rows(N, case["sources"], case["receivers"], 0.9 + 0.2 * jitter)
        truth = _slowness(N, g)
        b = (_times(D, truth) * (1 + 0.05 * randn(D.ptr.numel() - 1)))[:, None]
        D.lower = D.upper = b.float()
        D.x0 = (truth * (1 + 0.1 * randn(D.n))).clamp_min(0.05).float()[:, None]
        D.lam = float(D.ptr.numel() - 1)  # DROP with uniform weights: lambda = m
    else:
        D.ptr, D.col, D.val, target, organ = _rt_rows(case, 0.01 + jitter * 2 * math.pi / case["beams"])
        D.n = case["beams"] * case["nu"] * case["nw"]
        lo = torch.where(target, 0.95, -math.inf)
        up = torch.where(organ & ~target, 0.5, 1.07)
        vox = D.ptr.numel() - 1
        D.c = torch.zeros(D.n, dtype=F64, device=DEV)
        order = torch.sort(D.col, stable=True)
        cnt = torch.bincount(order.values, minlength=D.n)
        off = torch.zeros(D.n + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(cnt, 0)
        D.c = _segment_sums(D.val.to(F64)[order.indices], off).float()  # summed dose
        # the overlap voxels again, with a band that contradicts the target's; and the
        # dose-volume structures' copies of their rows
        blocks = [(torch.nonzero(target & organ)[:, 0], -math.inf, 0.3)]
        if case["dvc"]:
            t, o = torch.nonzero(target)[:, 0], torch.nonzero(organ)[:, 0]
            D.dvc, at = [], vox + int(blocks[0][0].numel())
            for rows, sense, frac, dose in ((t, smx.DVC_MIN, 0.95, 0.97), (t, smx.DVC_MAX, 0.05, 1.03),
                                            (o, smx.DVC_MAX, 0.05, 0.16)):
                blocks.append((rows, -math.inf, math.inf))
                D.dvc.append(dict(row_begin=at, row_end=at + int(rows.numel()), sense=sense, fraction=frac, dose=dose))
                at += int(rows.numel())
        for rows, bl, bu in blocks:
            if not rows.numel():
                continue
            at, counts = _take_rows(D.ptr, rows)
            D.ptr = torch.cat([D.ptr, D.ptr[-1] + torch.cumsum(counts, 0)])
            D.col, D.val = torch.cat([D.col, D.col[at]]), torch.cat([D.val, D.val[at]])
            lo = torch.cat([lo, torch.full((rows.numel(),), bl, device=DEV)])
            up = torch.cat([up, torch.full((rows.numel(),), bu, device=DEV)])
        D.lower, D.upper = lo.float()[:, None], up.float()[:, None]
        D.x0 = (0.8 * (1 + 0.15 * randn(D.n, 1))).clamp_min(0.0).float()
    D.m = D.ptr.numel() - 1
    D.lam = D.lam if case["basic"] == "drop" and case["kind"] == "seismic" else 1.0
    D.eps = 1e-2  # a hundredth of the values' range
    return D


def _parameters(case):
    return dict(gamma=case.get("gamma", 1.0), alpha=case.get("alpha", 0.99), n_red=case.get("n_red", 1),
                restart_every=case.get("restart_every", 0))


# --------------------------------------------------------------------------
# what is timed
# --------------------------------------------------------------------------

class State:
    """What a program holds between solves: the problem, and the starting point."""


def prepare(case, seed):
    D = _inputs(case, seed)
    S = State()
    S.call, S.K = case["call"], case["K"]
    S.op = smx.Operator(D.m, D.n, D.ptr, D.col, D.val, storage=case["storage"], image=D.image)
    tv = case["obj"] == "tv"
    S.problem = smx.Problem(S.op, lower=D.lower, upper=D.upper, box_lo=torch.zeros(D.n), box_hi=D.hi, lam=D.lam,
                            obj=OBJ[case["obj"]], tv_rows=D.image[0] if tv else 0, tv_cols=D.image[1] if tv else 0,
                            tv_eps=D.eps if tv else 0.0, linear_c=D.c if case["obj"] == "linear" else None, B=D.B,
                            basic=BASIC[case["basic"]], dvc=D.dvc, refine_iters=case.get("refine", -1),
                            **_parameters(case))
    if case["tuned"]:
        S.problem.set_x(D.x0)
        S.problem.autotune(reps=5)
    S.x0 = D.x0.cpu().numpy() if S.call == "solve" else D.x0
    return S


def run(S):
    p = S.problem
    if S.call == "solve":  # a fresh solve: counters and iterate reset, K iterations by graph replay
        p.reset(S.x0)
        p.run(S.K, graph=True)
        return p.get_x()
    p.set_x(S.x0)
    if S.call == "step":
        p.run(1, perturb=False)
        return p.get_x()
    return p.query()


def _sizes(case):
    """(rows, columns, estimated entries) from the case alone."""
    if case["kind"] == "dense":
        return case["m"], case["n"], case["m"] * case["n"]
    if case["kind"] == "ct":
        # a ray of the mean chord crosses 4/pi of its length in pixels of each direction's lines
        rows, N2 = case["angles"] * case["dets"], case["rows"] * case["cols"]
        return rows, N2, int(case["angles"] * N2 * 4 / math.pi)
    if case["kind"] == "seismic":
        # mean of the band's pixels: twice the half-width on both sides over a mean chord of about 0.9 N
        L = 0.9 * case["N"]
        return case["sources"] * case["receivers"], case["N"] ** 2, int(
            case["sources"] * case["receivers"] * L * 4 * (math.pi / 8 * math.sqrt(L) + 0.5))
    vox = case["X"] * case["Y"] * case["Z"]
    per = case["beams"] * math.pi * (6.4 / 2.4) ** 2 * 0.91
    extra = 0.005 * vox if not case["dvc"] else 0.3 * vox
    return int(vox + extra), case["beams"] * case["nu"] * case["nw"], int((vox + extra) * per)


def work(case):
    """One iteration reads every entry of A once (value and index; A does not
    stay on chip from one iteration to the next), the rows' offsets, bands and
    weights, and reads and writes x; EMR needs A y besides.  Two
    multiply-adds an entry and slice (A z and A^T c), a third with EMR."""
    m, n, nnz = _sizes(case)
    B, K = case["B"], case["K"]
    value = 4 if case["storage"] == "f32" else 2
    index = 2 if n <= 65536 else 4
    reads = 2 if case["basic"] == "emr" else 1
    products = 1 if case["call"] == "query" else reads + 1
    per = reads * nnz * (value + index) + 4 * m + m * (8 * B + 8) + n * (8 * B + 8)
    return {"bytes": K * per, "flops": K * 2 * products * nnz * B}


# --------------------------------------------------------------------------
# the same in float64, in plain torch
# --------------------------------------------------------------------------

def _objective(case, D, x):
    if case["obj"] == "sqnorm":
        return (x * x).sum()
    if case["obj"] == "l1":
        return x.abs().sum()
    if case["obj"] == "linear":
        return (D.c.to(F64) * x).sum()
    X = x.reshape(D.image)
    a, b, c = X[:-1, :-1], X[1:, :-1], X[:-1, 1:]
    return torch.sqrt((b - a) ** 2 + (c - a) ** 2 + D.eps ** 2).sum()


def _gradient(case, D, x):
    if case["obj"] == "sqnorm":
        return 2 * x
    if case["obj"] == "l1":
        return torch.sign(x)
    if case["obj"] == "linear":
        return D.c.to(F64)
    X = x.reshape(D.image)
    dx, dy = X[1:, :-1] - X[:-1, :-1], X[:-1, 1:] - X[:-1, :-1]
    tau = torch.sqrt(dx ** 2 + dy ** 2 + D.eps ** 2)
    G = torch.zeros_like(X)
    G[:-1, :-1] -= (dx + dy) / tau
    G[1:, :-1] += dx / tau
    G[:-1, 1:] += dy / tau
    return G.reshape(-1)


def _bands(D, r, lower, upper):
    """Bands with the dose-volume rows' set by their ranking at r."""
    if not D.dvc:
        return lower, upper
    lower, upper = lower.clone(), upper.clone()
    for g in D.dvc:
        s = slice(g["row_begin"], g["row_end"])
        N = g["row_end"] - g["row_begin"]
        most = g["sense"] == smx.DVC_MAX
        k = math.floor(g["fraction"] * N) if most else math.ceil(g["fraction"] * N)
        high = torch.zeros(N, dtype=torch.bool, device=DEV)
        high[torch.sort(r[s], descending=True, stable=True).indices[:k]] = True
        lower[s] = torch.where(high & (not most), g["dose"], -math.inf)
        upper[s] = torch.where(~high & most, g["dose"], math.inf)
    return lower, upper


class _Operator64:
    """A and its transpose as gathers and sums of consecutive runs."""

    def __init__(self, D, val):
        self.ptr, self.col, self.val = D.ptr, D.col, val
        rows = torch.repeat_interleave(torch.arange(D.m, device=DEV), D.ptr[1:] - D.ptr[:-1])
        order = torch.sort(D.col, stable=True)
        self.off = torch.zeros(D.n + 1, dtype=torch.int64, device=DEV)
        self.off[1:] = torch.cumsum(torch.bincount(order.values, minlength=D.n), 0)
        self.row, self.tval = rows[order.indices], val[order.indices]
        self.q = _segment_sums(val * val, D.ptr)

    def times(self, x):
        return _segment_sums(self.val * x[self.col], self.ptr)

    def transposed_times(self, c):
        return _segment_sums(self.tval * c[self.row], self.off)


def _step(case, D, O, z, lower, upper, w, Z):
    r = O.times(z)
    lower, upper = _bands(D, r, lower, upper)
    t = torch.minimum(torch.maximum(r, lower), upper) - r
    dia = torch.where(O.q > 0, w / O.q, torch.zeros_like(O.q))
    basic = case["basic"]
    c = {"cq": t / O.q.sum(), "emr": w * t}.get(basic, dia * t)
    y = O.transposed_times(c)
    if basic == "drop":
        y = y * Z
    elif basic == "el":
        y = y * ((dia * t * t).sum() / (y * y).sum())
    elif basic == "emr":
        y = y * ((y * y).sum() / (w * O.times(y) ** 2).sum())
    x = z + D.lam * y
    return x.clamp(0.0, 1.0 if D.hi is not None else math.inf), 0.5 * (dia * t * t).sum()


def exact(case, seed):
    D = _inputs(case, seed)
    val = D.val.to(F64)
    full = _Operator64(D, val)
    low = full if case["storage"] == "f32" else _Operator64(D, D.val.bfloat16().to(F64))
    w = torch.full((D.m,), 1.0 / D.m, dtype=F64, device=DEV)
    Z = 1.0 / torch.bincount(D.col[D.val != 0], minlength=D.n).to(F64).clamp_min(1.0)
    P = _parameters(case)
    K = case["K"]
    tail = 0 if low is full else (case["refine"] if case.get("refine", -1) >= 0 else -(-K // 20))
    out, prox, obj = [], [], []
    for s in range(D.B):
        x, lo, up = D.x0[:, s].to(F64), D.lower[:, s].to(F64), D.upper[:, s].to(F64)
        if case["call"] == "query":
            prox.append(float(_step(case, D, full, x, lo, up, w, Z)[1]))
            obj.append(float(_objective(case, D, x)))
            continue
        ell = restarts = 0
        for k in range(K):
            z = x
            if case["obj"] != "none" and case["call"] == "solve":
                if P["restart_every"] and k and k % P["restart_every"] == 0:
                    restarts += 1
                    ell = restarts
                g = _gradient(case, D, x)
                v, f, phase = -g / g.norm(), _objective(case, D, x), bool(g.norm() > 0)
                for _ in range(P["n_red"]):
                    for trial in range(100):
                        if not phase:
                            break
                        zt = z + P["gamma"] * P["alpha"] ** ell * v
                        ell += 1
                        ft = _objective(case, D, zt)
                        if ft <= f:
                            z, f = zt, ft
                            break
                        phase = trial < 99
            x, _ = _step(case, D, full if k >= K - tail else low, z, lo, up, w, Z)
        out.append(x)
    if case["call"] == "query":
        return np.array(prox), np.array(obj)
    return torch.stack(out, 1)
