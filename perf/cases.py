"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case names a `path` through the public entry points (`paper_2501_12497_amd.binding`, `.autograd`), the
sizes of the image stack it runs on, the data type and the options of the call:

  project   H and H^T of a plan (parallel beam, fan beam, blur): one data-fit gradient
  edges     blur, weighted spatial gradient and its adjoint on a ragged batch
  motion    L(v), its adjoint and its derivative in v
  flow      the Horn-Schunck flow update with the reverse flow, in place on the tracked flow
  gks       the flow by GKS with GCV (Solve-OF)
  krylov    one projected step over a Krylov basis: Gram matrices, projected solve, new iterate
  autograd  forward and backward of a loss through the three differentiable operators
  solve     a whole MMGKS solve

Sizes are those of the repository's own workloads (32x32x8 disk, 128x128x16 ellipses, 256x256x16
differentiation, 40 ragged deblurring sequences, 1024x1024x64) and of the range between them.
"""
import math

import numpy as np
import torch

from paper_2501_12497_amd import _lib
from paper_2501_12497_amd import autograd as AG
from paper_2501_12497_amd import binding as B

DT = {"f32": torch.float32, "f64": torch.float64}
GOLDEN = math.pi * (math.sqrt(5.0) - 1.0) / 2.0


def listed():
    return [
        # the data-fit gradient of the 128x128x16 workload: the call an outer optimiser makes most often
        dict(name="radon_128", path="project", op="radon", dtype="f32", nt=16, ny=128, nx=128, angles=30),
        # the same at the size of the headline workload
        dict(name="radon_1024", path="project", op="radon", dtype="f32", nt=64, ny=1024, nx=1024, angles=90),
        # double precision: the Golub-Kahan start of every solve and every FP64 solve; rectangular odd frames
        dict(name="radon_odd_f64", path="project", op="radon", dtype="f64", nt=16, ny=251, nx=310, angles=45),
        # the flat-detector fan beam of the paper's tests, between its 128x128 frames and 1024x1024
        dict(name="fan_512", path="project", op="fan", dtype="f32", nt=16, ny=512, nx=512, angles=90),
        # batched deblurring: 40 sequences of uneven sizes in one call per operator
        dict(name="edges_ragged40", path="edges", dtype="f32", seqs=40, lo=64, hi=256, t_lo=8, t_hi=32, sizes=3),
        # the motion term in its three modes, as a motion-compensated loss evaluates it
        dict(name="motion_512", path="motion", dtype="f32", nt=32, ny=512, nx=512, direction=1, interp=0),
        # one warm-started flow update (200 sweeps) of a tracker
        dict(name="flow_256", path="flow", dtype="f32", nt=16, ny=256, nx=256, sweeps=200, scale=1, delta_r=1),
        # the paper's own flow solver at the paper's setting: frames reduced below 50x50
        dict(name="gks_128", path="gks", dtype="f32", nt=16, ny=128, nx=128, ell=10, iters=20, scale=-1, pq=2),
        # the projected step late in a 30-iteration solve of the 256x256x16 workload
        dict(name="krylov_39", path="krylov", dtype="f32", nt=16, ny=256, nx=256, cols=39),
        # the differentiation workload
        dict(name="autograd_256", path="autograd", dtype="f32", nt=16, ny=256, nx=256, angles=30),
        # the smallest solve: latency and launches count; a flow update in every iteration
        dict(name="solve_32", path="solve", op="radon", dtype="f64", nt=8, ny=32, nx=32, angles=10, flow=1, reg="psi",
             iters=20, tau=1, sweeps=200),
        # the largest solve: FP32 operators, the spatio-temporal regulariser of the paper's method table
        dict(name="solve_1024", path="solve", op="radon", dtype="f32", nt=64, ny=1024, nx=1024, angles=90, flow=0,
             reg="aniso", iters=30, tau=10, sweeps=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frames(rng, lo, hi, most, t_lo=2, t_hi=64):
    """Frame sides over [lo, hi] (square or not, odd ones among them) and frames up to `most` pixels."""
    ny = _log_int(rng, lo, hi)
    nx = ny if rng.random() < 0.4 else min(hi, max(lo, int(ny * rng.uniform(0.7, 1.4))))
    nt = min(_log_int(rng, t_lo, t_hi), max(t_lo, most // (ny * nx)))
    return dict(nt=nt, ny=ny, nx=nx)


def draw(rng):
    path = rng.choice(["project", "project", "edges", "motion", "flow", "gks", "krylov", "autograd", "solve"])
    dtype = rng.choice(["f32", "f32", "f64"])
    c = dict(path=path, dtype=dtype)
    if path == "project":
        op = rng.choice(["radon", "radon", "fan", "blur"])
        c.update(op=op, **_frames(rng, 24, 1024, 1 << 23))
        if op != "blur":
            c["angles"] = _log_int(rng, 8, 90)
    elif path == "edges":
        lo = _log_int(rng, 24, 128)
        c.update(seqs=rng.randint(1, 40), lo=lo, hi=rng.randint(lo, 2 * lo), t_lo=2, t_hi=rng.randint(4, 32),
                 sizes=rng.randint(1, 1 << 20))
    elif path == "motion":
        c.update(_frames(rng, 24, 1024, 1 << 24), direction=rng.choice([1, -1]), interp=rng.choice([0, 0, 1]))
    elif path == "flow":
        c.update(_frames(rng, 24, 512, 1 << 22), sweeps=_log_int(rng, 6, 200), scale=rng.choice([1, 1, 2, 4]),
                 delta_r=rng.choice([1, 1, 2]))
    elif path == "gks":
        c.update(_frames(rng, 40, 512, 1 << 22, t_hi=32), ell=rng.randint(5, 10), iters=rng.randint(5, 20), scale=-1,
                 pq=rng.choice([2, 2, 1]))
    elif path == "krylov":
        c.update(_frames(rng, 32, 512, 1 << 21), cols=rng.choice([rng.randint(10, 40), rng.randint(10, 40),
                                                                  rng.randint(41, 160)]))
    elif path == "autograd":
        c.update(_frames(rng, 32, 512, 1 << 22), angles=_log_int(rng, 8, 60))
    else:
        # solves with a motion term run in FP64: the reverse flow is decided by rounding positions to pixels,
        # so two correct FP32 solves differ in it
        flow = rng.choice([0, 1])
        reg = rng.choice(["psi", "aniso", "iso", "gs"])
        c.update(_frames(rng, 32, 256, 1 << 20, t_lo=4, t_hi=32), op=rng.choice(["radon", "blur"]), angles=_log_int(rng, 10, 45),
                 dtype="f64" if flow else dtype, flow=flow, reg=reg, iters=rng.randint(8, 30),
                 tau=rng.choice([5, 10]), sweeps=_log_int(rng, 20, 200))
    return c


# ------------------------------------------------------------------------------- inputs


def _sizes(case):
    if "seqs" in case:
        r = np.random.default_rng(case["sizes"])
        side = r.integers(case["lo"], case["hi"] + 1, size=case["seqs"])
        nt = r.integers(case["t_lo"], case["t_hi"] + 1, size=case["seqs"])
        return [(int(t), int(n), int(n) + int(t) % 3) for t, n in zip(nt, side)]
    return [(case["nt"], case["ny"], case["nx"])]


def _bins(ny, nx):
    return 2 * int(math.hypot(ny, nx) / 2.0) + 1


def _angles(case):
    t = np.arange(case["nt"])[:, None]
    return np.arange(case["angles"])[None, :] * (math.pi / case["angles"]) + t * GOLDEN


def _fan(case):
    """Source and detector distances and the bin width: one pixel per bin at the frame centre."""
    n = max(case["ny"], case["nx"])
    return 1.5 * n, 2.5 * n, 2.5 / 1.5


def _phantom(nt, ny, nx, rng, count):
    """Ellipses that move and turn, later ones over earlier ones: [nt, ny, nx], FP64 on the GPU."""
    n = min(ny, nx)
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[:, None]
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, :]
    u = torch.zeros(nt, ny, nx, dtype=torch.float64, device="cuda")
    for _ in range(count):
        a, b = rng.uniform(0.06 * n, 0.22 * n, size=2)
        cx, cy = rng.uniform(0.3 * nx, 0.7 * nx), rng.uniform(0.3 * ny, 0.7 * ny)
        vx, vy = rng.uniform(-2.0, 2.0, size=2) * min(1.0, n / (8.0 * nt))
        phi, om, val = rng.uniform(0, math.pi), math.radians(rng.uniform(-3, 3)), rng.uniform(0.3, 1.0)
        for t in range(nt):
            c, s = math.cos(phi + om * t), math.sin(phi + om * t)
            dx, dy = x - (cx + vx * t), y - (cy + vy * t)
            inside = ((c * dx + s * dy) / a) ** 2 + ((c * dy - s * dx) / b) ** 2 <= 1.0
            u[t].masked_fill_(inside, val)
    return u


def _stack(case, seed):
    """(sizes, frames): the image stack of a case, FP64, packed."""
    rng = np.random.default_rng(seed)
    sizes = _sizes(case)
    count = 12 if case.get("ny", 0) >= 512 else 3
    return sizes, torch.cat([_phantom(t, ny, nx, rng, count).ravel() for t, ny, nx in sizes])


def _noise(gen, *shape, dtype=torch.float64):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=dtype)


def _smooth_flow(gen, sizes, vmax=3.0):
    """A smooth flow of at most vmax pixels for every pair: packed [pair][2][ny][nx], FP64."""
    out = []
    for t, ny, nx in sizes:
        coarse = _noise(gen, t - 1, 2, 6, 6)
        f = torch.nn.functional.interpolate(coarse, size=(ny, nx), mode="bicubic", align_corners=True)
        out.append((f * (vmax / f.abs().max())).ravel())
    return torch.cat(out)


def _plan(case, stack):
    ang = _angles(case).ravel() if "angles" in case else None
    if case["op"] == "blur":
        return B.plan_blur(stack, 9, 2.0)
    nb = [_bins(case["ny"], case["nx"])]
    if case["op"] == "fan":
        return B.plan_fan(stack, [case["angles"]], nb, ang, *_fan(case))
    return B.plan_radon(stack, [case["angles"]], nb, ang)


class State:
    """What a user's program holds before the call."""

    def __init__(self, case, **kw):
        self.case = case
        self.__dict__.update(kw)


def _data(case, seed):
    """The tensors of a case (a dict, in the precision of the call), from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt, path = DT[case["dtype"]], case["path"]
    sizes, u = _stack(case, seed)
    P = sum((t - 1) * ny * nx for t, ny, nx in sizes)
    gx = sum(t * ny * (nx - 1) for t, ny, nx in sizes)
    gy = sum(t * (ny - 1) * nx for t, ny, nx in sizes)
    textured = u + 0.05 * _noise(gen, u.numel())
    d = {}
    if path == "project":
        m = u.numel() if case["op"] == "blur" else case["nt"] * case["angles"] * _bins(case["ny"], case["nx"])
        d = dict(u=textured, r=_noise(gen, m))
    elif path == "edges":
        # weights of the majorant at the current iterate, 1/sqrt(|Psi u|^2 + eps^2) in size
        d = dict(u=textured, gx=_noise(gen, gx), gy=_noise(gen, gy), wx=1.0 / (1e-3 + 0.1 * _noise(gen, gx).abs()),
                 wy=1.0 / (1e-3 + 0.1 * _noise(gen, gy).abs()))
    elif path == "motion":
        d = dict(u=textured, v=_smooth_flow(gen, sizes), r=_noise(gen, P))
    elif path == "flow":
        d = dict(u=textured, v=0.5 * _smooth_flow(gen, sizes))
    elif path == "gks":
        d = dict(u=textured)
    elif path == "krylov":
        # columns as a Golub-Kahan basis leaves them: unit norm, Theta v and H v of noise-like vectors
        n, K = u.numel(), case["cols"]
        m = max(n // 8, 2 * K)
        V = _noise(gen, K, n) / math.sqrt(n)
        AV = (_noise(gen, K, m) / math.sqrt(m)) * torch.logspace(0, -2, K, device="cuda", dtype=torch.float64)[:, None]
        b = AV.sum(0) + 0.02 * AV.sum(0).norm() / math.sqrt(m) * _noise(gen, m)
        d = dict(TV=_noise(gen, K, gx + gy) / math.sqrt(n), nu=0.1 * _noise(gen, gx + gy) ** 3, AV=AV)
        d = {k: x.to(dt) for k, x in d.items()}
        d.update(V=V, b=b)
        return sizes, d
    elif path == "autograd":
        m = case["nt"] * case["angles"] * _bins(case["ny"], case["nx"])
        d = dict(u=textured, v=_smooth_flow(gen, sizes), w1=_noise(gen, m), w2=_noise(gen, gx), w3=_noise(gen, gy),
                 w4=_noise(gen, P))
    else:
        frames = u.view(case["nt"], case["ny"], case["nx"])
        clean = (_blur(frames) if case["op"] == "blur" else
                 _radon(frames, _angles(case), _bins(case["ny"], case["nx"]))).ravel()
        e = _noise(gen, clean.numel())
        e *= 0.02 * clean.norm() / e.norm()
        # detector readings come in FP32 (which also drops the order of the sums behind `clean`)
        return sizes, dict(b=(clean + e).float().double(), delta=0.02 * float(clean.float().norm()))
    return sizes, {k: x.to(dt) for k, x in d.items()}


def prepare(case, seed):
    sizes, d = _data(case, seed)
    stack = B.Stack(sizes)
    plan = None
    if case["path"] in ("project", "solve"):
        plan = _plan(case, stack)
    elif case["path"] == "edges":
        plan = B.plan_blur(stack, 9, 2.0)
    elif case["path"] == "autograd":
        plan = _plan(dict(case, op="radon"), stack)
    s = State(case, stack=stack, plan=plan, **d)
    if case["path"] == "flow":
        s.v_rev = torch.empty_like(s.v)
    if case["path"] == "gks":
        s.v = torch.empty(2 * stack.n_pair_px, dtype=s.u.dtype, device="cuda")
    return s


# ------------------------------------------------------------------------------- one pass


def run(s):
    c, path = s.case, s.case["path"]
    if path == "project":
        return {"b": B.apply_A(s.plan, s.u), "u": B.apply_At(s.plan, s.r)}
    if path == "edges":
        b = B.apply_A(s.plan, s.u)
        gx, gy = B.apply_grad(s.stack, s.u, wx=s.wx, wy=s.wy)
        return {"b": b, "gx": gx, "gy": gy,
                "u": B.apply_grad(s.stack, gx=s.gx, gy=s.gy, wx=s.wx, wy=s.wy, transpose=True)}
    if path == "motion":
        a = (c["direction"], c["interp"])
        return {"r": B.apply_flow_op(s.stack, _lib.MMOF_FLOW_FWD, *a, s.u, s.v),
                "u": B.apply_flow_op(s.stack, _lib.MMOF_FLOW_ADJ, *a, None, s.v, s.r),
                "dv": B.apply_flow_op(s.stack, _lib.MMOF_FLOW_DV, *a, s.u, s.v, s.r)}
    if path == "flow":
        B.flow_update_scaled(s.stack, s.u, s.v, alpha=0.1, n_sweeps=c["sweeps"], delta_r=c["delta_r"],
                             scale=c["scale"], v_rev=s.v_rev)
        return {"v": s.v, "v_rev": s.v_rev}
    if path == "gks":
        return {"v": B.flow_solve_gks(s.stack, s.u, s.v, ell=c["ell"], n_iter=c["iters"], scale=c["scale"], pq=c["pq"])}
    if path == "krylov":
        GT = B.weighted_gram(s.TV, s.nu, 1e-3)
        GA = B.weighted_gram(s.AV)
        d = B.block_dot(s.AV, s.b)
        b2 = float(torch.dot(s.b, s.b))
        z, lam, d2, status = B.projected_solve(GA, GT, d, b2, 0.01 * b2)
        return {"GT": GT, "GA": GA, "d": d, "z": z, "lam": lam, "status": status, "u": B.block_combine(s.V, z)}
    if path == "autograd":
        u = s.u.detach().requires_grad_(True)
        v = s.v.detach().requires_grad_(True)
        u.grad = v.grad = None
        gx, gy = AG.gradient_op(u, s.stack)
        loss = ((s.w1 * AG.forward_op(u, s.plan)).sum() + (s.w2 * gx).sum() + (s.w3 * gy).sum()
                + (s.w4 * AG.flow_op(u, v, s.stack, 1)).sum())
        loss.backward()
        return {"u": u.grad, "v": v.grad}
    r = B.solve_joint(s.plan, s.b, s.delta, ell=10, k_max=c["iters"], tau=c["tau"], n_sweeps=c["sweeps"], alpha=0.1,
                      op_dtype=c["dtype"], use_flow=c["flow"], reg=c["reg"])
    if c["dtype"] == "f32":
        # FP32 operators determine the frames and lambda to FP32: the program keeps them so
        return {"u": r.u.float(), "lambda": np.asarray(r.lambdas, dtype=np.float32)}
    return {"u": r.u, "v": r.v, "v_rev": r.v_rev, "lambda": np.asarray(r.lambdas), "resid": np.asarray(r.resid)}


# ------------------------------------------------------------------------------- the work


def work(case):
    path, es = case["path"], 4 if case["dtype"] == "f32" else 8
    sizes = _sizes(case)
    n = sum(t * ny * nx for t, ny, nx in sizes)
    P = sum((t - 1) * ny * nx for t, ny, nx in sizes)
    g = sum(t * (2 * ny * nx - ny - nx) for t, ny, nx in sizes)
    m = n if case.get("op", "blur") == "blur" and path != "autograd" else case["nt"] * case["angles"] * _bins(case["ny"], case["nx"])
    proj = 36.0 * n if m == n else 4.0 * n * case.get("angles", 0)   # flops of one application of H
    if path == "project":
        return {"bytes": 2 * es * (n + m), "flops": 2 * proj}
    if path == "edges":
        return {"bytes": es * (2 * n + (n + 2 * g) + (2 * g + n)), "flops": 36.0 * n + 2 * g + 3 * g}
    if path == "motion":
        return {"bytes": es * ((n + 3 * P) + (n + 3 * P) + (n + 5 * P)), "flops": 12.0 * P * 3}
    if path == "flow":
        f = max(1, case["scale"]) ** 2
        return {"bytes": es * (n + 6 * P), "flops": 30.0 * P / f * case["sweeps"]}
    if path == "gks":
        f = 1
        while max(case["ny"], case["nx"]) / f >= 50:
            f *= 2
        K, p = case["ell"] + case["iters"], P / f ** 2
        # the basis read for each new row of the two Gram matrices, the iterate and the orthogonalisation (FP64)
        return {"bytes": es * (n + 2 * P), "flops": sum(2.0 * 2 * p * k * 5 for k in range(1, K))}
    if path == "krylov":
        K, mm = case["cols"], max(n // 8, 2 * case["cols"])
        return {"bytes": es * (g * (K + 1) + mm * K) + 8.0 * n * (K + 1), "flops": float((g + mm) * K * (K + 1) + 2 * n * K)}
    if path == "autograd":
        return {"bytes": es * (2 * (n + m) + 2 * (n + g) + 2 * (n + 3 * P) + (n + 5 * P)), "flops": 2 * proj + 4 * g + 36.0 * P}
    R = g + (P if case["reg"] in ("aniso", "iso") else 0) + (2 * P if case["flow"] else 0)
    by = fl = 0.0
    for k in range(case["iters"]):
        K = 10 + k
        # Theta V for the weighted Gram matrix, V for the iterate and for the new direction, H V for the residual
        by += es * R * (K + 1) + 16.0 * n * K + es * m * K + 2 * es * (n + m) + 2 * es * (n + R)
        fl += float(R) * K * (K + 1) + 4.0 * n * K + 2.0 * m * K + 2 * proj
    by += 10 * (16.0 * (n + m) + 8.0 * n * 10)
    fl += 20 * proj
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------------------- the operators in 64 bits


def _hat(ny, nx, ang, nb):
    """Lower bin and fraction of every pixel at each angle of one frame: [angles, ny * nx]."""
    c = torch.as_tensor([math.cos(a) for a in ang], dtype=torch.float64, device="cuda")
    s = torch.as_tensor([math.sin(a) for a in ang], dtype=torch.float64, device="cuda")
    y = torch.arange(ny, device="cuda", dtype=torch.float64) - (ny - 1) / 2.0
    x = torch.arange(nx, device="cuda", dtype=torch.float64) - (nx - 1) / 2.0
    pos = (x[None, None, :] * c[:, None, None] + y[None, :, None] * s[:, None, None]).reshape(len(ang), -1) + (nb - 1) / 2.0
    j = torch.floor(pos)
    return j.long(), pos - j


def _radon(u, ang, nb):
    """H u of the parallel beam, u [nt, ny, nx] -> [nt, angles, nb] (bins beyond the detector are dropped)."""
    nt, ny, nx = u.shape
    out = torch.zeros(nt, ang.shape[1], nb + 2, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // (ny * nx))
    for t in range(nt):
        flat = u[t].ravel()
        for a in range(0, ang.shape[1], step):
            part = ang[t, a:a + step]
            j, f = _hat(ny, nx, part, nb)
            for off, w in ((0, 1.0 - f), (1, f)):
                k = (j + (off + 1)).clamp_(0, nb + 1)
                out[t, a:a + len(part)].scatter_add_(1, k, w * flat)
    return out[:, :, 1:nb + 1]


def _radon_t(b, ang, ny, nx):
    nt, na, nb = b.shape
    pad = torch.zeros(nt, na, nb + 2, dtype=torch.float64, device="cuda")
    pad[:, :, 1:nb + 1] = b
    out = torch.zeros(nt, ny * nx, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // (ny * nx))
    for t in range(nt):
        for a in range(0, na, step):
            part = ang[t, a:a + step]
            j, f = _hat(ny, nx, part, nb)
            for off, w in ((0, 1.0 - f), (1, f)):
                k = (j + (off + 1)).clamp_(0, nb + 1)
                out[t] += (w * torch.gather(pad[t, a:a + len(part)], 1, k)).sum(0)
    return out.view(nt, ny, nx)


def _fan_entries(ny, nx, theta, nb, geom):
    """Joseph's method: (ray, pixel, weight) of one angle, zero weight outside the frame."""
    dso, dsd, du = geom
    c, s = math.cos(theta), math.sin(theta)
    uj = (torch.arange(nb, device="cuda", dtype=torch.float64) - (nb - 1) / 2.0) * du
    dx, dy = -dsd * s + uj * c, dsd * c + uj * s
    sx, sy = dso * s, -dso * c
    step = torch.hypot(dx, dy)
    for rows, sel in ((True, (dy.abs() >= dx.abs())), (False, (dy.abs() < dx.abs()))):
        k = sel.nonzero().ravel()
        if not k.numel():
            continue
        p, q = (dx[k], dy[k]) if rows else (dy[k], dx[k])
        (s0, s1), (n0, n1) = ((sx, sy), (nx, ny)) if rows else ((sy, sx), (ny, nx))
        line = torch.arange(n1, device="cuda", dtype=torch.float64)[None, :]
        pos = s0 + ((line - (n1 - 1) / 2.0) - s1) * p[:, None] / q[:, None] + (n0 - 1) / 2.0
        i = torch.floor(pos)
        f = pos - i
        for off, w in ((0, 1.0 - f), (1, f)):
            at = i.long() + off
            ok = (at >= 0) & (at < n0)
            at = at.clamp(0, n0 - 1)
            pix = line.long() * nx + at if rows else at * nx + line.long()
            yield k, pix, torch.where(ok, w * (step[k] / q.abs())[:, None], torch.zeros_like(w))


def _fan_pair(u, b, ang, geom):
    nt, ny, nx = u.shape
    nb = b.shape[2]
    out, back = torch.zeros_like(b), torch.zeros(nt, ny * nx, dtype=torch.float64, device="cuda")
    for t in range(nt):
        flat = u[t].ravel()
        for a in range(ang.shape[1]):
            for k, pix, w in _fan_entries(ny, nx, float(ang[t, a]), nb, geom):
                out[t, a, k] += (w * flat[pix]).sum(1)
                back[t].scatter_add_(0, pix.ravel(), (w * b[t, a, k][:, None]).ravel())
    return out, back.view(nt, ny, nx)


def _blur(u):
    i = torch.arange(-4, 5, dtype=torch.float64)
    k = torch.exp(-i * i / 8.0)
    k = (k / k.sum()).tolist()
    nt, ny, nx = u.shape
    p = torch.nn.functional.pad(u, (4, 4, 0, 0))
    h = sum(k[j] * p[:, :, j:j + nx] for j in range(9))
    p = torch.nn.functional.pad(h, (0, 0, 4, 4))
    return sum(k[j] * p[:, j:j + ny, :] for j in range(9))


def _psi_t(gx, gy, nt, ny, nx):
    out = torch.zeros(nt, ny, nx, dtype=torch.float64, device="cuda")
    out[:, :, 1:] += gx
    out[:, :, :-1] -= gx
    out[:, 1:, :] += gy
    out[:, :-1, :] -= gy
    return out


def _cells(v, ny, nx):
    """Corner pixels, fractions and in-range flags of the sample positions p + v(p), v [pairs, 2, ny, nx]."""
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[None, :, None]
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, None, :]
    xr, yr = x + v[:, 0], y + v[:, 1]
    xq, yq = xr.clamp(0, nx - 1.0), yr.clamp(0, ny - 1.0)
    x0, y0 = torch.floor(xq), torch.floor(yq)
    x1, y1 = (x0 + 1).clamp(max=nx - 1).long(), (y0 + 1).clamp(max=ny - 1).long()
    return (x0.long(), y0.long(), x1, y1, xq - x0, yq - y0, (xr >= 0) & (xr <= nx - 1), (yr >= 0) & (yr <= ny - 1))


def _motion(u, v, r, direction, interp):
    """L(v) u, L(v)^T r and (d(L(v)u)/dv)^T r of one sequence."""
    nt, ny, nx = u.shape
    src, base = (u[1:], u[:-1]) if direction > 0 else (u[:-1], u[1:])
    flat = src.reshape(nt - 1, -1)
    take = lambda q: torch.gather(flat, 1, q.reshape(nt - 1, -1)).view(nt - 1, ny, nx)  # noqa: E731
    if interp == 1:
        # the position is the sum in the precision of the call, which decides the pixel
        x = torch.arange(nx, device="cuda")[None, None, :]
        y = torch.arange(ny, device="cuda")[None, :, None]
        xs = torch.round(x + v[:, 0]).clamp(0, nx - 1).long()
        ys = torch.round(y + v[:, 1]).clamp(0, ny - 1).long()
        terms, dv = [(ys * nx + xs, torch.ones(nt - 1, ny, nx, dtype=torch.float64, device="cuda"))], None
    else:
        x0, y0, x1, y1, fx, fy, inx, iny = _cells(v.double(), ny, nx)
        q = [y0 * nx + x0, y0 * nx + x1, y1 * nx + x0, y1 * nx + x1]
        terms = list(zip(q, [(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy]))
        s00, s01, s10, s11 = (take(k) for k in q)
        dv = torch.stack([r * inx * ((1 - fy) * (s01 - s00) + fy * (s11 - s10)),
                          r * iny * ((1 - fx) * (s10 - s00) + fx * (s11 - s01))], dim=1)
    fwd = sum(w * take(k) for k, w in terms) - base
    warp_t = torch.zeros(nt - 1, ny * nx, dtype=torch.float64, device="cuda")
    for k, w in terms:
        warp_t.scatter_add_(1, k.reshape(nt - 1, -1), (w * r).reshape(nt - 1, -1))
    back = torch.zeros_like(u)
    warp_t = warp_t.view(nt - 1, ny, nx)
    if direction > 0:
        back[1:] += warp_t
        back[:-1] -= r
    else:
        back[:-1] += warp_t
        back[1:] -= r
    return fwd, back, torch.zeros_like(v, dtype=torch.float64) if dv is None else dv


def _derivs(u, dr):
    nt, ny, nx = u.shape
    iy = torch.arange(-dr, ny + dr, device="cuda")
    ix = torch.arange(-dr, nx + dr, device="cuda")
    iy = torch.where(iy < 0, -1 - iy, torch.where(iy >= ny, 2 * ny - 1 - iy, iy))
    ix = torch.where(ix < 0, -1 - ix, torch.where(ix >= nx, 2 * nx - 1 - ix, ix))
    p = u[:, iy][:, :, ix]
    box = 2 * dr + 1
    rows = sum(p[:, j:j + ny, :] for j in range(box))
    cols = sum(p[:, :, j:j + nx] for j in range(box))
    Ix = (rows[:, :, 2 * dr:] - rows[:, :, :nx]) / (box * 2 * dr)
    Iy = (cols[:, 2 * dr:, :] - cols[:, :ny, :]) / (box * 2 * dr)
    mean = sum(rows[:, :, j:j + nx] for j in range(box)) / (box * box)
    return Ix[:-1], Iy[:-1], mean[1:] - mean[:-1]


def _block_mean(u, f):
    ny, nx = u.shape[-2:]
    p = torch.nn.functional.pad(u, (0, -nx % f, 0, -ny % f))
    one = torch.nn.functional.pad(torch.ones(ny, nx, dtype=torch.float64, device="cuda"), (0, -nx % f, 0, -ny % f))
    cut = lambda q: q.unflatten(-2, (-1, f)).unflatten(-1, (-1, f)).sum((-3, -1))  # noqa: E731
    return cut(p) / cut(one)


def _up(v, f, ny, nx):
    ny_s, nx_s = v.shape[-2:]
    y = ((torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5) / f - 0.5).clamp(0, ny_s - 1.0)
    x = ((torch.arange(nx, device="cuda", dtype=torch.float64) + 0.5) / f - 0.5).clamp(0, nx_s - 1.0)
    y0, x0 = torch.floor(y).long(), torch.floor(x).long()
    y1, x1 = (y0 + 1).clamp(max=ny_s - 1), (x0 + 1).clamp(max=nx_s - 1)
    fy, fx = (y - y0)[:, None], x - x0
    rows = (1 - fy) * v[..., y0, :] + fy * v[..., y1, :]
    return f * ((1 - fx) * rows[..., x0] + fx * rows[..., x1])


def _sweeps(u, v, gamma, count, dr):
    nt, ny, nx = u.shape
    Ix, Iy, It = _derivs(u, dr)
    d = torch.full((ny, nx), 4.0, dtype=torch.float64, device="cuda")
    d[0] -= 1
    d[-1] -= 1
    d[:, 0] -= 1
    d[:, -1] -= 1
    for _ in range(count):
        p = torch.nn.functional.pad(v, (1, 1, 1, 1))
        m = (p[..., :-2, 1:-1] + p[..., 2:, 1:-1] + p[..., 1:-1, :-2] + p[..., 1:-1, 2:]) / d
        k = (Ix * m[:, 0] + Iy * m[:, 1] + It) / (gamma * d + Ix * Ix + Iy * Iy)
        v = torch.stack([m[:, 0] - Ix * k, m[:, 1] - Iy * k], dim=1)
    return v


def exact(case, seed):
    """What run() returns, in 64 bits; None where there is no such value (iterative solves, roots)."""
    path = case["path"]
    if path in ("gks", "solve"):
        return None
    sizes, d = _data(case, seed)
    raw, d = d, {k: x.double() for k, x in d.items()}
    if path == "krylov":
        w = 1.0 / torch.sqrt(d["nu"] ** 2 + 1e-6)
        GT = torch.zeros(case["cols"], case["cols"], dtype=torch.float64, device="cuda")
        for i in range(0, w.numel(), 1 << 20):
            X = d["TV"][:, i:i + (1 << 20)].contiguous()
            GT += torch.mm(X * w[i:i + (1 << 20)], X.t().contiguous())
        GA = torch.mm(d["AV"], d["AV"].t().contiguous())
        return {"GT": GT, "GA": GA, "d": torch.mv(d["AV"], d["b"]), "z": None, "lam": None, "status": None, "u": None}
    if path == "edges":
        out = {"b": [], "gx": [], "gy": [], "u": []}
        o = ox = oy = 0
        for t, ny, nx in sizes:
            u = d["u"][o:o + t * ny * nx].view(t, ny, nx)
            lx, ly = t * ny * (nx - 1), t * (ny - 1) * nx
            wx, gx = (d[k][ox:ox + lx].view(t, ny, nx - 1) for k in ("wx", "gx"))
            wy, gy = (d[k][oy:oy + ly].view(t, ny - 1, nx) for k in ("wy", "gy"))
            for k, x in (("b", _blur(u)), ("gx", wx * (u[:, :, 1:] - u[:, :, :-1])), ("gy", wy * (u[:, 1:] - u[:, :-1])),
                         ("u", _psi_t(wx * gx, wy * gy, t, ny, nx))):
                out[k].append(x.ravel())
            o, ox, oy = o + t * ny * nx, ox + lx, oy + ly
        return {k: torch.cat(x) for k, x in out.items()}
    nt, ny, nx = sizes[0]
    u = d["u"].view(nt, ny, nx)
    if path == "project":
        if case["op"] == "blur":
            return {"b": _blur(u).ravel(), "u": _blur(d["r"].view(nt, ny, nx)).ravel()}
        r = d["r"].view(nt, case["angles"], -1)
        if case["op"] == "fan":
            b, back = _fan_pair(u, r, _angles(case), _fan(case))
        else:
            b, back = _radon(u, _angles(case), r.shape[2]), _radon_t(r, _angles(case), ny, nx)
        return {"b": b.ravel(), "u": back.ravel()}
    if path == "motion":
        v = raw["v"].view(nt - 1, 2, ny, nx)
        out = _motion(u, v, d["r"].view(nt - 1, ny, nx), case["direction"], case["interp"])
        return dict(zip(("r", "u", "dv"), (x.ravel() for x in out)))
    if path == "flow":
        v, f = d["v"].view(nt - 1, 2, ny, nx), case["scale"]
        if f > 1:
            v = _up(_sweeps(_block_mean(u, f), _block_mean(v, f) / f, 0.01, case["sweeps"], case["delta_r"]), f, ny, nx)
        else:
            v = _sweeps(u, v, 0.01, case["sweeps"], case["delta_r"])
        return {"v": v.ravel(), "v_rev": None}
    ang, P = _angles(case), (nt - 1, ny, nx)
    _, du, dv = _motion(u, raw["v"].view(nt - 1, 2, ny, nx), d["w4"].view(P), 1, 0)
    du = du + _psi_t(d["w2"].view(nt, ny, nx - 1), d["w3"].view(nt, ny - 1, nx), nt, ny, nx)
    du = du + _radon_t(d["w1"].view(nt, case["angles"], -1), ang, ny, nx)
    return {"u": du.ravel(), "v": dv.ravel()}
