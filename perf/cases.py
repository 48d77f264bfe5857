"""Performance cases: what users of the engine have it do, timed through its public entry points.

Six kinds of work, each over the range of sizes it is used at:

* ``cost``      the consistency cost of B motion hypotheses and every pair's term (``Scan.cost``);
* ``grad``      cost and its gradient with respect to every view's motion (``Scan.cost_grad``);
* ``estimate``  one evaluation of the motion-estimation loop: spline nodes -> per-view motion ->
                cost and gradient -> gradient of the nodes (``SplineMotion``, ``Scan.cost_grad``);
* ``served``    a burst of requests over several resident scans (``Server.submit`` / ``wait``);
* ``scan``      a new scan: load the projections, build the Radon-derivative sinograms and read
                them into one host array (``load_scan``, ``build_sinograms``,
                ``ecc_scan_read_sinogram``), as a program does that keeps them beside the scan;
* ``fdk``       the reconstruction of a compensated scan (``Scan.fdk``).

The evaluation kinds install sinograms computed elsewhere (``set_sinograms``): those of ellipsoids,
whose Radon derivative has a closed form.  ``scan`` and ``fdk`` take analytic projections of
ellipsoid phantoms.  All inputs come from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1806_02637_amd import binding, engine, inputs, motion, serve

_ENGINES = {}


def _engine() -> engine.Engine:
    """The program's one engine (a context per process, as a user's program has)."""
    if "gpu" not in _ENGINES:
        _ENGINES["gpu"] = engine.Engine(0)
    return _ENGINES["gpu"]


# ---- cases -----------------------------------------------------------------------------------

_DET_SMALL = dict(W=128, H=128, pitch=2.4, n_alpha=180, n_t=181)
_DET_MID = dict(W=620, H=480, pitch=0.616, n_alpha=360, n_t=512)
_DET_FULL = dict(W=1240, H=960, pitch=0.308, n_alpha=768, n_t=1024)
_EVAL = dict(dtype="f32", geom="f32", kappa="object", c=0.0)  # c = 0: e = d


def listed():
    return [
        # the smallest evaluation: launches and host time count (a check of a few views, a test)
        dict(name="cost_16_views", kind="cost", n_views=16, **_DET_SMALL, K=64, B=1, **_EVAL),
        # the benchmark's step: 32 hypotheses of the 496-view scan
        dict(name="cost_496_views", kind="cost", n_views=496, **_DET_FULL, K=512, B=32, **_EVAL),
        # half the memory per scan (BF16 storage), robust norm on, a mid-size scan
        dict(name="cost_248_bf16", kind="cost", n_views=248, **_DET_MID, K=256, B=32, dtype="bf16", geom="f32",
             kappa="object", c=30.0),
        # odd sizes, FP16 storage, FP64 plane geometry and the detector-bounded plane range
        dict(name="cost_101_detector", kind="cost", n_views=101, W=511, H=389, pitch=0.75, n_alpha=301, n_t=433,
             K=200, B=5, dtype="f16", geom="f64", kappa="detector", c=0.0),
        # gradient of one hypothesis of the mid-size scan, 1488 parameters
        dict(name="grad_248_views", kind="grad", n_views=248, **_DET_MID, K=256, B=1, **_EVAL),
        # gradient of a batch over every view's six parameters (population methods, line searches)
        dict(name="grad_372_views", kind="grad", n_views=372, **_DET_FULL, K=512, B=16, **_EVAL),
        # one evaluation of the motion-estimation experiment: 17 nodes, 496 views
        dict(name="estimate_496_views", kind="estimate", n_views=496, **_DET_FULL, K=512, n_nodes=17, **_EVAL),
        # a burst on a server: three resident scans, half the requests with gradients
        dict(name="served_burst", kind="served", views="60 120 248", **_DET_MID, K=256, B=16, requests=6, **_EVAL),
        # a small scan of the served mix arrives
        dict(name="scan_60_views", kind="scan", n_views=60, **_DET_MID, ds=0.5),
        # a full-size scan arrives
        dict(name="scan_496_views", kind="scan", n_views=496, **_DET_FULL, ds=0.5),
        # a reconstruction with the motion of all six parameters taken out, preview size
        dict(name="fdk_248_moved", kind="fdk", n_views=248, W=620, H=480, pitch=0.616, nx=256, ny=256, nz=256,
             voxel=0.8, moved="all"),
        # the full reconstruction
        dict(name="fdk_496_views", kind="fdk", n_views=496, W=1240, H=960, pitch=0.308, nx=512, ny=512, nz=512,
             voxel=0.4, moved="none"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cost", "cost", "grad", "estimate", "served", "scan", "scan", "fdk", "fdk"])
    W = _log_int(rng, 96, 1240)
    H = max(64, int(W * rng.uniform(0.6, 0.95)))
    det = dict(W=W, H=H, pitch=round(380.0 / W, 4))
    grid = dict(n_alpha=int(80 + W * rng.uniform(0.5, 0.62)), n_t=int(60 + W * rng.uniform(0.75, 0.9)))
    n_views = max(12, min(_log_int(rng, 12, 400), int(1.6e8 / (W * H))))
    K = _log_int(rng, 48, 512)
    opts = dict(dtype=rng.choice(["f32", "f32", "bf16", "f16"]), geom=rng.choice(["f32", "f32", "f32", "f64"]),
                kappa=rng.choice(["object", "object", "object", "detector"]), c=rng.choice([0.0, 0.0, 30.0]))
    if kind in ("cost", "grad"):
        pairs = n_views * (n_views - 1) // 2
        B = max(1, min(_log_int(rng, 1, 32), int(6e8 / (pairs * K))))
        return dict(kind=kind, n_views=n_views, **det, **grid, K=K, B=B, **opts)
    if kind == "estimate":
        opts["geom"] = "f32"
        return dict(kind=kind, n_views=max(n_views, 20), **det, **grid, K=K, n_nodes=rng.randint(5, 17), **opts)
    if kind == "served":
        views = " ".join(str(min(n_views, _log_int(rng, 12, 160))) for _ in range(rng.randint(2, 4)))
        opts["kappa"] = "object"
        return dict(kind=kind, views=views, **det, **grid, K=min(K, 256), B=_log_int(rng, 1, 16),
                    requests=rng.randint(2, 8), **opts)
    if kind == "scan":
        return dict(kind=kind, n_views=n_views, **det, **grid, ds=rng.choice([0.5, 0.5, 0.7]))
    n_views = max(n_views, 40)
    nx, ny = _log_int(rng, 32, 320), _log_int(rng, 32, 320)
    nz = max(8, min(_log_int(rng, 16, 320), int(1.2e10 / (nx * ny * n_views))))
    voxel = round(rng.uniform(120.0, 220.0) / max(nx, ny, nz), 3)
    return dict(kind="fdk", n_views=n_views, **det, nx=nx, ny=ny, nz=nz, voxel=voxel,
                moved=rng.choice(["none", "z", "all"]))


# ---- inputs ----------------------------------------------------------------------------------

def _views(case):
    """View counts of a served case's scans."""
    return [int(n) for n in case["views"].split()]


def _geometry(case, n_views=None) -> inputs.ScanGeometry:
    return inputs.ScanGeometry(case["n_views"] if n_views is None else n_views, case["W"], case["H"], case["pitch"])


def _phantom(geom, seed) -> inputs.Phantom:
    return inputs.random_phantom(seed, 10, contained_radius=0.95 * geom.fov_radius())


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _projections(geom, seed) -> torch.Tensor:
    return inputs.project(geom, _phantom(geom, seed), device=_device(), as_tensor=True)


def _sinograms(geom, n_alpha, n_t, seed) -> torch.Tensor:
    """Radon-derivative sinograms [N, n_alpha + 1, n_t] (FP32) of an ellipsoid phantom.  The plane through
    the source and the detector line (alpha, t) has normal n ~ f cos(alpha) e_u + f sin(alpha) e_v - t e_w; an
    ellipsoid's 3-D Radon transform is rho pi abc (1 - d^2 / h^2) / h with d the plane's distance from its
    centre and h^2 = n^T Q diag(a^2) Q^T n, so its derivative is -2 rho pi abc d / h^3 where |d| < h.  The
    sinogram holds it over 1 + t^2 / f^2, which cancels the normalisation of n."""
    dev = _device()
    ph = _phantom(geom, seed)
    C_all, R_all = geom.frames()
    f = geom.f_px
    t_max = 0.5 * math.hypot(geom.W, geom.H)
    alpha = torch.arange(n_alpha + 1, dtype=torch.float64, device=dev) * (math.pi / n_alpha)
    c, s = f * torch.cos(alpha), f * torch.sin(alpha)
    t = torch.linspace(-t_max, t_max, n_t, dtype=torch.float32, device=dev)[None, None, :]
    out = torch.zeros((geom.n_views, n_alpha + 1, n_t), dtype=torch.float32, device=dev)
    step = max(1, (1 << 24) // ((n_alpha + 1) * n_t))
    for v0 in range(0, geom.n_views, step):
        C = torch.as_tensor(C_all[v0:v0 + step], device=dev)
        R = torch.as_tensor(R_all[v0:v0 + step], device=dev)
        acc = out[v0:v0 + step]
        for e in range(ph.n):
            Q = torch.as_tensor(ph.axes[e], device=dev)
            M = Q @ torch.diag(torch.as_tensor(ph.semi_axes[e] ** 2, device=dev)) @ Q.T
            Mc = R @ M @ R.transpose(1, 2)  # camera axes, [V, 3, 3]
            p = (R @ (C - torch.as_tensor(ph.centers[e], device=dev))[:, :, None])[:, :, 0]
            h0 = c * c * Mc[:, 0, 0, None] + 2 * c * s * Mc[:, 0, 1, None] + s * s * Mc[:, 1, 1, None]
            h1 = -2 * (c * Mc[:, 0, 2, None] + s * Mc[:, 1, 2, None])
            d0 = c * p[:, 0, None] + s * p[:, 1, None]
            h2 = (h0[:, :, None].float() + h1[:, :, None].float() * t) + Mc[:, 2, 2, None, None].float() * t * t
            d = d0[:, :, None].float() - p[:, 2, None, None].float() * t
            k = -2.0 * math.pi * f * f * float(ph.density[e] * np.prod(ph.semi_axes[e]))
            acc += torch.where(d * d < h2, k * d / (h2 * torch.sqrt(h2)), torch.zeros_like(d))
    return out


def _resident(geom, n_alpha, n_t, dtype, seed) -> engine.Scan:
    blank = torch.zeros((geom.n_views, geom.H, geom.W), dtype=torch.float32, device="cuda")
    scan = _engine().load_scan(geom.projection_matrices(), geom.intrinsics(), blank)
    del blank
    scan.set_sinograms(_sinograms(geom, n_alpha, n_t, seed), dtype)
    return scan


def _volume(case):
    return case["nx"], case["ny"], case["nz"], case["voxel"]


def _fdk_motion(case, seed):
    if case["moved"] == "none":
        return None
    params = (5,) if case["moved"] == "z" else (0, 1, 2, 3, 4, 5)
    return inputs.smooth_motion(seed + 1, case["n_views"], 2.0, params)


def _nodes(case, seed) -> np.ndarray:
    """Node values of the out-of-plane translation, as an optimiser meets them half way."""
    nodes = np.zeros((1, 6, case["n_nodes"]))
    nodes[0, 5] = np.random.default_rng(seed + 1).normal(0.0, 1.0, case["n_nodes"])
    return nodes


class _Held:
    """What a program keeps between calls; the scans' memory goes back when it is dropped."""

    def __init__(self, case):
        self.case = case
        self.scans = []
        self.server = None

    def __del__(self):
        try:
            if self.server is not None:
                self.server.close()
            for scan in self.scans:
                scan.free()
        except Exception:
            pass


def prepare(case, seed):
    st = _Held(case)
    kind = case["kind"]
    if kind in ("scan", "fdk"):
        geom = _geometry(case)
        st.images = _projections(geom, seed)
        st.P, st.intr = geom.projection_matrices(), geom.intrinsics()
        if kind == "scan":
            st.sino = np.zeros((case["n_views"], case["n_alpha"] + 1, case["n_t"]), dtype=np.float32)
        else:
            st.scan = _engine().load_scan(st.P, st.intr, st.images)
            st.scans.append(st.scan)
            th = _fdk_motion(case, seed)
            st.theta = None if th is None else torch.as_tensor(th, device="cuda")
        return st
    if kind == "served":
        views = _views(case)
        for i, n in enumerate(views):
            st.scans.append(_resident(_geometry(case, n), case["n_alpha"], case["n_t"], case["dtype"], seed + 10 * i))
        st.R_mm = _geometry(case, 2).default_object_radius()
        st.server = serve.Server(_engine(), n_slots=4, arena_bytes=8 << 30)
        st.requests = []
        for r in range(case["requests"]):
            i = r % len(views)
            st.requests.append((st.scans[i], inputs.random_motion(seed + 100 + r, case["B"], views[i]), r % 2 == 1))
        return st
    geom = _geometry(case)
    st.R_mm = geom.default_object_radius()
    st.c = case["c"] if case["c"] > 0 else math.inf
    st.scan = _resident(geom, case["n_alpha"], case["n_t"], case["dtype"], seed)
    st.scans.append(st.scan)
    if kind == "estimate":
        st.model = motion.SplineMotion(st.scan, case["n_nodes"])
        st.nodes = torch.as_tensor(_nodes(case, seed), device="cuda")
    else:
        st.theta = torch.as_tensor(inputs.random_motion(seed + 1, case["B"], geom.n_views), device="cuda")
    return st


def run(state):
    case = state.case
    kind = case["kind"]
    if kind == "cost":
        return state.scan.cost(state.theta, case["K"], state.R_mm, c=state.c, geom=case["geom"], with_pairs=True,
                               kappa=case["kappa"])
    if kind == "grad":
        return state.scan.cost_grad(state.theta, case["K"], state.R_mm, c=state.c, geom=case["geom"],
                                    kappa=case["kappa"])
    if kind == "estimate":
        theta = state.model.theta(state.nodes)
        cost, grad = state.scan.cost_grad(theta, case["K"], state.R_mm, c=state.c, kappa=case["kappa"])
        return cost, grad, state.model.grad(state.nodes, grad)
    if kind == "served":
        c = case["c"] if case["c"] > 0 else math.inf
        ids = [state.server.submit(scan, theta, case["K"], state.R_mm, grad, c=c, geom=case["geom"],
                                   kappa=case["kappa"]) for scan, theta, grad in state.requests]
        results = [state.server.wait(i) for i in ids]
        return [r.cost for r in results] + [r.grad for r in results if r.grad is not None]
    if kind == "scan":
        scan = _engine().load_scan(state.P, state.intr, state.images)
        scan.build_sinograms(case["n_alpha"], case["n_t"], case["ds"], "f32")
        for v in range(case["n_views"]):
            binding.ecc_scan_read_sinogram(scan.ctx, scan.id, v, state.sino[v].ctypes.data)
        scan.free()
        return state.sino
    return state.scan.fdk(state.images, _volume(case), state.theta)


def work(case):
    kind = case["kind"]
    pixels = case["W"] * case["H"]
    if kind == "scan":
        n, m, k = case["n_views"], case["n_alpha"], case["n_t"]
        # every pixel enters two lines of every angle
        return dict(bytes=4.0 * n * (pixels + (m + 1) * k), flops=4.0 * n * m * pixels)
    if kind == "fdk":
        n, vox = case["n_views"], case["nx"] * case["ny"] * case["nz"]
        length = 2.0 * case["W"]
        ramp = n * case["H"] * 10.0 * length * math.log2(length) / 2.0
        return dict(bytes=4.0 * (n * pixels + vox), flops=16.0 * n * vox + ramp)
    size = 4 if case["dtype"] == "f32" else 2
    cells = (case["n_alpha"] + 1) * case["n_t"]
    views = _views(case) if kind == "served" else [case["n_views"]]
    planes = [n * (n - 1) // 2 * case["K"] for n in views]
    if kind == "served":
        asked = [(r % len(views), r % 2) for r in range(case["requests"])]
        flops = sum(case["B"] * planes[i] * (240.0 if grad else 100.0) for i, grad in asked)
        out = sum(case["B"] * views[i] * (48.0 + 24.0 * grad) for i, grad in asked)
        return dict(bytes=float(size * cells * sum(views)) + out, flops=flops)
    B = case.get("B", 1)
    out = 4.0 * B * planes[0] / case["K"] if kind == "cost" else 24.0 * B * views[0]
    return dict(bytes=size * cells * views[0] + 48.0 * B * views[0] + out,
                flops=B * planes[0] * (100.0 if kind == "cost" else 240.0))


# ---- the same in 64 bits, plain torch --------------------------------------------------------

def _rigid(theta):
    a = torch.deg2rad(theta[:, :3])
    (cx, cy, cz), (sx, sy, sz) = torch.cos(a).T, torch.sin(a).T
    R = torch.stack([cz * cy, cz * sy * sx - sz * cx, cz * sy * cx + sz * sx,
                     sz * cy, sz * sy * sx + cz * cx, sz * sy * cx - cz * sx,
                     -sy, cy * sx, cy * cx], -1).reshape(-1, 3, 3)
    return R, theta[:, 3:]


def _moved(P, theta):
    """P T(theta): the 3x3 part and the source of every view."""
    R, t = _rigid(theta)
    M = P[:, :, :3] @ R
    p4 = P[:, :, 3] + (P[:, :, :3] @ t[:, :, None])[:, :, 0]
    return M, p4, -torch.linalg.solve(M, p4)


def _pair_terms(case, geom, P, sino, theta, ia, ib):
    """e of the pairs (ia, ib) of one hypothesis."""
    K, R_mm = case["K"], geom.default_object_radius()
    M, _, C = _moved(P, theta)
    cof = torch.stack([torch.linalg.cross(M[:, 1], M[:, 2]), torch.linalg.cross(M[:, 2], M[:, 0]),
                       torch.linalg.cross(M[:, 0], M[:, 1])], 1)
    cof = torch.stack([cof[:, 0], cof[:, 1], cof[:, 2] + geom.u0 * cof[:, 0] + geom.v0 * cof[:, 1]], 1)
    bh = torch.nn.functional.normalize(C[ib] - C[ia], dim=1)
    w = (C[ia] * bh).sum(1, keepdim=True) * bh - C[ia]
    h = torch.linalg.norm(w, dim=1)
    u2 = w / h[:, None]
    u1 = torch.linalg.cross(bh, u2)
    k_max = torch.where(h > R_mm, torch.asin((R_mm / h).clamp(max=1.0 - 1e-15)), torch.full_like(h, math.pi / 2))
    u = ((torch.arange(K, dtype=torch.float64, device=h.device) + 0.5) * (2.0 / K) - 1.0)
    kappa = k_max[:, None] * u
    n = torch.cos(kappa)[..., None] * u1[:, None] + torch.sin(kappa)[..., None] * u2[:, None]  # [p, K, 3]
    t_max = 0.5 * math.hypot(geom.W, geom.H)
    dt = 2 * t_max / (case["n_t"] - 1)

    def look_up(i):
        l1, l2, l3 = (n @ cof[i].transpose(1, 2)).unbind(-1)
        fold = (l2 < 0) | ((l2 == 0) & (l1 < 0))
        sign = torch.where(fold, -1.0, 1.0).to(l1.dtype)
        r = torch.sqrt(l1 * l1 + l2 * l2)
        t = -sign * l3 / r
        a = torch.atan2(sign * l2, sign * l1) * (case["n_alpha"] / math.pi)
        hit = l3.abs() <= 0.5 * geom.W * l1.abs() + 0.5 * geom.H * l2.abs()
        m = a.detach().floor().clamp(0, case["n_alpha"] - 1).long()
        tau = (t + t_max) / dt
        k = tau.detach().floor().clamp(-1, case["n_t"]).long()
        fa, ft = a - m, tau - k
        rows = sino.reshape(-1)

        def tap(mm, kk):
            ok = (kk >= 0) & (kk < case["n_t"])
            at = (i[:, None] * (case["n_alpha"] + 1) + mm) * case["n_t"] + kk.clamp(0, case["n_t"] - 1)
            return torch.where(ok, rows[at].double(), torch.zeros((), dtype=torch.float64, device=rows.device))

        top = (1 - ft) * tap(m, k) + ft * tap(m, k + 1)
        bot = (1 - ft) * tap(m + 1, k) + ft * tap(m + 1, k + 1)
        return sign * (1 + t * t / geom.f_px ** 2) * ((1 - fa) * top + fa * bot), hit

    (Sa, hit_a), (Sb, hit_b) = look_up(ia), look_up(ib)
    hit = hit_a & hit_b
    d = torch.where(hit, (Sa - Sb) ** 2, torch.zeros_like(Sa)).sum(1) / hit.sum(1).clamp(min=1)
    return d / (1 + d / case["c"]) if case["c"] > 0 else d


def _evaluate(case, geom, sino, theta, grad):
    """(cost [B], e [B, pairs], gradient [B, N, 6] or None)."""
    dev = sino.device
    P = torch.as_tensor(geom.projection_matrices(), device=dev)
    ia, ib = (torch.as_tensor(x, device=dev) for x in np.triu_indices(geom.n_views, 1))
    step = max(1, (1 << 21) // case["K"])
    e_all = torch.empty((len(theta), len(ia)), dtype=torch.float64, device=dev)
    g_all = torch.zeros((len(theta), geom.n_views, 6), dtype=torch.float64, device=dev) if grad else None
    for b, th in enumerate(theta):
        th = torch.as_tensor(th, device=dev)
        for p in range(0, len(ia), step):
            at = slice(p, p + step)
            x = th.clone().requires_grad_(grad)
            e = _pair_terms(case, geom, P, sino, x, ia[at], ib[at])
            e_all[b, at] = e.detach()
            if grad:
                g_all[b] += torch.autograd.grad(e.sum(), x)[0]
    return e_all.sum(1), e_all, g_all


def _akima(nodes, n_views):
    """Akima 1970 through evenly spaced nodes, at every view index."""
    n = nodes.shape[-1]
    x = torch.linspace(0.0, n_views - 1.0, n, dtype=torch.float64, device=nodes.device)
    m = (nodes[..., 1:] - nodes[..., :-1]) / (x[1:] - x[:-1])
    lo, hi = 2 * m[..., 0] - m[..., 1], 2 * m[..., -1] - m[..., -2]
    m = torch.cat([(2 * lo - m[..., 0])[..., None], lo[..., None], m, hi[..., None],
                   (2 * hi - m[..., -1])[..., None]], -1)
    w_hi, w_lo = (m[..., 3:] - m[..., 2:-1]).abs(), (m[..., 1:-2] - m[..., :-3]).abs()
    flat = w_hi + w_lo == 0
    slope = torch.where(flat, 0.5 * (m[..., 1:-2] + m[..., 2:-1]),
                        (w_hi * m[..., 1:-2] + w_lo * m[..., 2:-1]) / torch.where(flat, 1.0, w_hi + w_lo))
    at = torch.arange(n_views, dtype=torch.float64, device=nodes.device)
    i = (torch.searchsorted(x, at, right=True) - 1).clamp(0, n - 2)
    h = x[i + 1] - x[i]
    s = (at - x[i]) / h
    return ((2 * s ** 3 - 3 * s ** 2 + 1) * nodes[..., i] + (s ** 3 - 2 * s ** 2 + s) * h * slope[..., i]
            + (3 * s ** 2 - 2 * s ** 3) * nodes[..., i + 1] + (s ** 3 - s ** 2) * h * slope[..., i + 1])


def _line_sums(case, geom, images):
    """Sinograms [N, n_alpha + 1, n_t]: t-differences of the weighted images' bilinear line sums."""
    dev = images.device
    N, H, W = images.shape
    n_alpha, n_t, ds = case["n_alpha"], case["n_t"], case["ds"]
    u = torch.arange(W, dtype=torch.float64, device=dev) - geom.u0
    v = torch.arange(H, dtype=torch.float64, device=dev) - geom.v0
    cosw = geom.f_px / torch.sqrt(geom.f_px ** 2 + u[None, :] ** 2 + v[:, None] ** 2)
    pix = torch.zeros((H + 2, W + 2, N), dtype=torch.float64, device=dev)
    pix[1:-1, 1:-1] = (images.double() * cosw).permute(1, 2, 0)
    pix = pix.reshape(-1, N)
    t_max = 0.5 * math.hypot(W, H)
    dt = 2 * t_max / (n_t - 1)
    n_s = 2 * math.ceil(t_max / ds) + 1
    t = -t_max + dt * torch.arange(n_t, dtype=torch.float64, device=dev)
    s = (torch.arange(n_s, dtype=torch.float64, device=dev) - 0.5 * (n_s - 1)) * ds
    G = torch.zeros((n_alpha, n_t, N), dtype=torch.float64, device=dev)
    step = max(1, (1 << 27) // (n_s * N))
    for m in range(n_alpha):
        ca, sa = math.cos(m * math.pi / n_alpha), math.sin(m * math.pi / n_alpha)
        for k in range(0, n_t, step):
            tt = t[k:k + step, None]
            x, y = geom.u0 + tt * ca - s * sa + 1, geom.v0 + tt * sa + s * ca + 1
            inside = (x > 0) & (x < W + 1) & (y > 0) & (y < H + 1)
            line = torch.nonzero(inside)[:, 0]
            x, y = x[inside], y[inside]
            ix, iy = x.floor().long().clamp(0, W), y.floor().long().clamp(0, H)
            fx, fy = (x - ix)[:, None], (y - iy)[:, None]
            at = iy * (W + 2) + ix
            val = ((1 - fy) * ((1 - fx) * pix[at] + fx * pix[at + 1])
                   + fy * ((1 - fx) * pix[at + W + 2] + fx * pix[at + W + 3]))
            G[m, k:k + step].index_add_(0, line, val, alpha=ds)
    pad = torch.nn.functional.pad(G, (0, 0, 1, 1))
    S = (pad[:, 2:] - pad[:, :-2]) / (2 * dt)
    S = torch.cat([S, -S[:1].flip(1)], 0)
    return S.permute(2, 0, 1).contiguous()


def _reconstruct(case, geom, images, theta):
    dev = images.device
    N, H, W = images.shape
    f, D = geom.f_px, geom.sid_mm
    arc = math.radians(geom.arc_deg)
    delta = 0.5 * (arc - math.pi)
    u = torch.arange(W, dtype=torch.float64, device=dev) - geom.u0
    v = torch.arange(H, dtype=torch.float64, device=dev) - geom.v0
    cosw = f / torch.sqrt(f * f + u[None, :] ** 2 + v[:, None] ** 2)
    gamma = -torch.atan(u / f)
    k = torch.arange(-(W - 1), W, dtype=torch.float64, device=dev)
    ramp = torch.where(k.remainder(2) == 1, -1.0 / (math.pi * k) ** 2, torch.zeros_like(k))
    ramp[W - 1] = 0.25
    L = 1 << (3 * W - 2).bit_length()
    ramp_f = torch.fft.rfft(ramp, L)
    M, p4, _ = _moved(torch.as_tensor(geom.projection_matrices(), device=dev),
                      torch.zeros((N, 6), dtype=torch.float64, device=dev) if theta is None
                      else torch.as_tensor(theta, device=dev))
    nx, ny, nz, vox = _volume(case)
    x, y, z = ((torch.arange(n, dtype=torch.float64, device=dev) - 0.5 * (n - 1)) * vox for n in (nx, ny, nz))
    out = torch.zeros((nz, ny, nx), dtype=torch.float64, device=dev)
    for lam in range(N):
        beta = arc * lam / (N - 1)
        w = torch.ones_like(gamma)
        lo, hi = beta < 2 * (delta - gamma), beta > math.pi - 2 * gamma
        w = torch.where(hi, torch.sin(0.25 * math.pi * (math.pi + 2 * delta - beta) / (delta + gamma)) ** 2, w)
        w = torch.where(lo, torch.sin(0.25 * math.pi * beta / (delta - gamma)) ** 2, w)
        q = torch.fft.irfft(torch.fft.rfft(images[lam].double() * cosw * w, L) * ramp_f, L)[:, W - 1:2 * W - 1]
        q = torch.nn.functional.pad(q * (f / D), (2, 2, 2, 2)).reshape(-1)
        a, b, c = (M[lam, i, 2] * z[:, None, None] + M[lam, i, 1] * y[None, :, None]
                   + M[lam, i, 0] * x[None, None, :] + p4[lam, i] for i in range(3))
        pu, pv = (a / c + 2).clamp(0, W + 2), (b / c + 2).clamp(0, H + 2)
        iu, iv = pu.floor().long(), pv.floor().long()
        fu, fv = pu - iu, pv - iv
        at = iv * (W + 4) + iu
        last = len(q) - 1
        val = ((1 - fv) * ((1 - fu) * q[at] + fu * q[(at + 1).clamp(max=last)])
               + fv * ((1 - fu) * q[(at + W + 4).clamp(max=last)] + fu * q[(at + W + 5).clamp(max=last)]))
        out += val * (arc / (N - 1)) * (D / c) ** 2
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "scan":
        length = math.hypot(case["W"], case["H"]) / case["ds"]
        if case["n_views"] * case["n_alpha"] * case["n_t"] * length > 2e10:
            return None
        geom = _geometry(case)
        return _line_sums(case, geom, _projections(geom, seed))
    if kind == "fdk":
        if case["n_views"] * case["nx"] * case["ny"] * case["nz"] > 1e10:
            return None
        geom = _geometry(case)
        return _reconstruct(case, geom, _projections(geom, seed), _fdk_motion(case, seed))
    if case["kappa"] == "detector":  # its plane range has no short form here
        return None
    if kind == "served":
        costs, grads, views = [], [], _views(case)
        sinos = [_sinograms(_geometry(case, n), case["n_alpha"], case["n_t"], seed + 10 * i)
                 for i, n in enumerate(views)]
        for r in range(case["requests"]):
            i = r % len(views)
            cost, _, grad = _evaluate(case, _geometry(case, views[i]), sinos[i],
                                      inputs.random_motion(seed + 100 + r, case["B"], views[i]), r % 2 == 1)
            costs.append(cost)
            grads += [] if grad is None else [grad]
        return costs + grads
    geom = _geometry(case)
    sino = _sinograms(geom, case["n_alpha"], case["n_t"], seed)
    if kind == "estimate":
        nodes = torch.as_tensor(_nodes(case, seed), device=sino.device).requires_grad_(True)
        theta = _akima(nodes, geom.n_views).transpose(1, 2)
        cost, _, grad = _evaluate(case, geom, sino, theta.detach(), True)
        return cost, grad, torch.autograd.grad(theta, nodes, grad)[0]
    theta = inputs.random_motion(seed + 1, case["B"], geom.n_views)
    cost, e, grad = _evaluate(case, geom, sino, theta, kind == "grad")
    return (cost, grad) if kind == "grad" else (cost, e)
