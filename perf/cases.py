"""Work that a user of this framework has it do, as timed cases.

Each case goes through the public Python entry points (binding.Smoother and
warmstart.WarmStartNet) with inputs on the GPU.  The state-space workloads are
the coordinated-turn target with two bearing sensors (nx = 5) and four stacked
targets with eight sensors (nx = 20), simulated from the case's seed; the
smoother starts from a given trajectory (the truth plus noise, one covariance
for every slot), as it does from a learned start or from an earlier solve of
the same track.  The warm-start network runs with its trained weights.

``exact`` evaluates the same calls in 64 bits with plain NumPy / PyTorch: the
sequential Kalman filter and RTS smoother on the linearised model, vectorised
over tracks, and the network as float64 matrix products.
"""
import json
import math
import os

import numpy as np
import torch

from paper_2102_00514_amd import binding, warmstart
from paper_2102_00514_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WEIGHTS = os.path.join(ROOT, "paper_2102_00514_amd", "weights", "warmstart_ieks.npz")

# standard deviations of a given starting trajectory around the truth, per
# state of a target (position, velocity, turn rate)
START_STD = (0.1, 0.1, 0.1, 0.1, 0.05)


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _smooth(name, tracks, t_min, t_max, iters, lin="taylor", precision="f64", targets=1, form="covariance",
            lm=0.0, lanes=0, slots=0):
    c = {"kind": "smooth", "tracks": tracks, "t_min": t_min, "t_max": t_max, "iters": iters, "lin": lin,
         "precision": precision, "targets": targets, "form": form, "lm": lm, "lanes": lanes, "slots": slots}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the paper's experiment at its shortest: one track, ten iterations; launches and latency count
        _smooth("single_T100_ieks_f64", 1, 100, 100, 10),
        # the headline: one long track, ten iterations
        _smooth("single_T32768_ieks_f64", 1, 32768, 32768, 10),
        # one track of an odd length with sigma points, in FP32 (at lengths where FP32 resolves the
        # covariances: longer tracks wander off to where their scan loses digits)
        _smooth("single_T501_cubature_f32", 1, 501, 501, 2, lin="cubature", precision="f32"),
        # the square-root form, for ill-conditioned steps
        _smooth("single_T8191_ieks_sqrt_f64", 1, 8191, 8191, 5, form="sqrt"),
        # hundreds of ragged tracks (two million slots) in one batch, sigma points, the schedule the autotuner finds for them
        _smooth("batch_512_ragged_cubature_f64", 512, 100, 8192, 2, lin="cubature", lanes=64, slots=16),
        # a ragged batch under damping, with the MAP objective of the result
        _smooth("batch_300_ragged_lm_f64", 300, 50, 3000, 3, lm=0.1),
        # filtering pass and marginal likelihood of a batch (model comparison)
        {"name": "filter_256_ragged_f64", "kind": "filter", "tracks": 256, "t_min": 200, "t_max": 4096,
         "lin": "taylor", "precision": "f64"},
        # four stacked targets (nx = 20), sigma points: the long track, a short one, a short one in FP32
        _smooth("stacked_T65536_unscented_f64", 1, 65536, 65536, 1, lin="unscented", targets=4),
        _smooth("stacked_T255_unscented_f64", 1, 255, 255, 5, lin="unscented", targets=4),
        _smooth("stacked_T500_unscented_f32", 1, 500, 500, 1, lin="unscented", precision="f32", targets=4),
        # learned start of 512 tracks, products on the matrix cores
        {"name": "warmstart_512x4096", "kind": "trajectory", "tracks": 512, "t_min": 4096, "t_max": 4096,
         "max_batch": 16384},
        # loss and gradient of one training batch of the warm-start network
        {"name": "warmstart_gradient_1024", "kind": "gradient", "windows": 1024, "data": 4096},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "sqrt", "batch", "lm", "filter", "stacked", "stacked",
                       "trajectory", "gradient"])
    if kind == "single":
        lin = rng.choice(["taylor", "taylor", "cubature"])
        prec = rng.choice(["f64", "f64", "f32"])
        T = _log_uniform(rng, 100, 32768 if prec == "f64" else 600)
        return _smooth("", 1, T, T, rng.choice([3, 5, 10]) if prec == "f64" else rng.choice([1, 2]), lin=lin, precision=prec)
    if kind == "sqrt":
        T = _log_uniform(rng, 500, 16384)
        return _smooth("", 1, T, T, rng.choice([2, 5]), form="sqrt")
    if kind == "batch":
        lo = rng.randint(10, 200)
        return _smooth("", _log_uniform(rng, 32, 512), lo, _log_uniform(rng, 500, 8192), 2,
                       lin=rng.choice(["cubature", "cubature", "taylor"]), lanes=64, slots=rng.choice([4, 8, 16]))
    if kind == "lm":
        return _smooth("", _log_uniform(rng, 20, 400), rng.randint(10, 100), _log_uniform(rng, 500, 4000), 3,
                       lm=rng.choice([0.01, 0.1, 1.0]))
    if kind == "filter":
        return {"kind": "filter", "tracks": _log_uniform(rng, 1, 256), "t_min": rng.randint(100, 400),
                "t_max": _log_uniform(rng, 500, 4096), "lin": rng.choice(["taylor", "cubature"]),
                "precision": "f64"}
    if kind == "stacked":
        prec = rng.choice(["f64", "f64", "f32"])
        T = _log_uniform(rng, 200, 60000) if prec == "f64" else _log_uniform(rng, 100, 600)
        return _smooth("", 1, T, T, 1 if T > 20000 or prec == "f32" else 2, lin=rng.choice(["unscented", "cubature"]),
                       precision=prec, targets=4)
    if kind == "trajectory":
        t = _log_uniform(rng, 200, 4096)
        return {"kind": "trajectory", "tracks": _log_uniform(rng, 8, 512), "t_min": max(1, t - rng.randint(0, 150)),
                "t_max": t, "max_batch": rng.choice([1024, 16384])}
    n = _log_uniform(rng, 16, 1024)
    return {"kind": "gradient", "windows": n, "data": n + rng.randint(0, 2000)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _simulate(rng, T, x0, dt, Lq):
    """States x_0..x_T of one coordinated-turn target: the recursion summed up
    in closed form (turn rate by a cumulative sum, velocity and position as
    cumulative sums in the rotated frame)."""
    e = rng.standard_normal((T, 5)) @ Lq.T
    x = np.empty((T + 1, 5))
    x[0] = x0
    x[1:, 4] = x0[4] + np.cumsum(e[:, 4])
    a = x[:-1, 4] * dt
    theta = np.concatenate([[0.0], np.cumsum(a)])
    turn = np.exp(1j * theta)
    v = turn * (x0[2] + 1j * x0[3] + np.concatenate([[0.0], np.cumsum((e[:, 2] + 1j * e[:, 3]) / turn[1:])]))
    h = 0.5 * a
    small = np.abs(h) < 1e-6
    sinc = np.where(small, 1.0, np.sin(h) / np.where(small, 1.0, h))
    p = x0[0] + 1j * x0[1] + np.cumsum(dt * sinc * np.exp(1j * h) * v[:-1] + e[:, 0] + 1j * e[:, 1])
    x[1:, 0], x[1:, 1] = p.real, p.imag
    x[:, 2], x[:, 3] = v.real, v.imag
    return x


def _problem(case, seed):
    """Problem, starting means [S, nx] and starting covariance [nx, nx]."""
    rng = np.random.default_rng([17, seed])
    nt = case.get("targets", 1)
    n = case["tracks"]
    nx = 5 * nt
    if nt == 1:
        sensors, owner = np.asarray(wl.CT_SENSORS), np.zeros(2, dtype=np.int64)
    else:
        sensors, owner = rng.uniform(-2.0, 2.0, (2 * nt, 2)), np.arange(2 * nt) // 2
    ny = len(sensors)
    Q = wl.ct_process_noise(n_targets=nt)
    Lq = np.linalg.cholesky(wl.ct_process_noise())
    lo, hi = min(case["t_min"], case["t_max"]), case["t_max"]
    # the lengths are the case's, whatever the seed
    lengths = np.random.default_rng([23, n, lo, hi]).integers(lo, hi + 1, n)
    lengths[n // 2] = hi
    states = []
    for T in lengths:
        per = []
        for _ in range(nt):
            if n == 1 and nt == 1:
                x0 = np.asarray(wl.CT_M0)
            else:
                phi = rng.uniform(0.0, 2.0 * np.pi)
                x0 = np.array([*rng.uniform(-1.0, 1.0, 2), np.cos(phi), np.sin(phi), rng.uniform(-1.0, 1.0)])
            per.append(_simulate(rng, int(T), x0, wl.CT_DT, Lq))
        states.append(np.concatenate(per, axis=1))
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    first = offsets[:-1] + np.arange(n)
    truth = np.concatenate(states)
    m0 = truth[first].copy()
    m0[:, 4::5] = 0.0
    keep = np.ones(len(truth), dtype=bool)
    keep[first] = False
    at = truth[keep]
    ang = np.arctan2(at[:, 5 * owner + 1] - sensors[:, 1], at[:, 5 * owner] - sensors[:, 0])
    y = wl.wrap_angle(ang + wl.CT_R_STD * rng.standard_normal(ang.shape))
    std = np.tile(START_STD, nt)
    start = truth + std * rng.standard_normal(truth.shape)
    pb = wl.Problem(nx, ny, wl.MODEL_CT_BEARINGS, wl.ct_params(sensors, owner), Q, wl.CT_R_STD ** 2 * np.eye(ny), m0,
                    np.broadcast_to(np.eye(nx), (n, nx, nx)).copy(), y, offsets, truth)
    return pb, start, np.diag(std ** 2)


def _windows(case, seed):
    """Training windows: bearing features [n, 2 ny, W], labels [n, W, nx], batch indices."""
    rng = np.random.default_rng([19, seed])
    n, W = case["data"], 64
    Lq = np.linalg.cholesky(wl.ct_process_noise())
    sensors = np.asarray(wl.CT_SENSORS)
    T = 1 + W * 16
    runs = []
    for _ in range(-(-n // 16)):
        x0 = np.array([*wl.CT_M0[:4], rng.uniform(-1.0, 1.0)])
        runs.append(_simulate(rng, T, x0, wl.CT_DT, Lq)[1:1 + 16 * W].reshape(16, W, 5))
    lab = np.concatenate(runs)[:n]
    ang = np.arctan2(lab[..., 1:2] - sensors[:, 1], lab[..., 0:1] - sensors[:, 0])
    ang = ang + wl.CT_R_STD * rng.standard_normal(ang.shape)
    x = np.stack([np.sin(ang[..., 0]), np.cos(ang[..., 0]), np.sin(ang[..., 1]), np.cos(ang[..., 1])], axis=1)
    idx = rng.permutation(n)[:case["windows"]].astype(np.int32)
    return x.astype(np.float32), lab.astype(np.float32), idx


def _net_config():
    with np.load(WEIGHTS, allow_pickle=False) as z:
        return json.loads(str(z["config"])), z["params"].copy(), z["mu"].copy(), z["sigma"].copy()


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    stream = torch.cuda.current_stream().cuda_stream
    kind = case["kind"]
    if kind == "gradient":
        x, lab, idx = _windows(case, seed)
        cfg, theta, mu, sigma = _net_config()
        cfg["max_batch"] = max(case["windows"], 16)
        net = warmstart.WarmStartNet(warmstart.config(**cfg), stream=stream, params=theta)
        net.set_normalization(mu, sigma)
        return {"case": case, "net": net, "x": torch.from_numpy(x).cuda(), "lab": torch.from_numpy(lab).cuda(),
                "idx": torch.from_numpy(idx).cuda()}
    pb, start, cov = _problem(case, seed)
    if kind == "trajectory":
        net, _, _ = warmstart.load(WEIGHTS, stream=stream, max_batch=case["max_batch"])
        net.set_tracks(pb.offsets)
        return {"case": case, "net": net, "y": torch.from_numpy(pb.y).cuda(),
                "mean": torch.zeros((pb.n_slots, pb.nx), dtype=torch.float64, device="cuda")}
    dt = torch.float64 if case["precision"] == "f64" else torch.float32
    sm = binding.Smoother(pb, stream=stream, n_iter=case.get("iters", 1), lin=case["lin"],
                          precision=case["precision"], form=case.get("form", "covariance"),
                          lm_lambda=case.get("lm", 0.0), tile_lanes=case.get("lanes", 0),
                          lane_slots=case.get("slots", 0))
    st = {"case": case, "sm": sm, "start": torch.from_numpy(start).to("cuda", dt), "cov0": cov}
    if kind == "filter":
        # the filtering pass linearises at the handle's trajectory
        sm.set_trajectory_device(st["start"].data_ptr(), 0, cov)
    else:
        st["mean"] = torch.empty((pb.n_slots, pb.nx), dtype=dt, device="cuda")
        st["cov"] = torch.empty((pb.n_slots, pb.nx, pb.nx), dtype=dt, device="cuda")
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "gradient":
        grad, loss = state["net"].gradient(state["x"].data_ptr(), state["lab"].data_ptr(), case["data"],
                                           state["idx"].data_ptr(), case["windows"])
        return {"grad": grad, "loss": np.float32(loss)}
    if kind == "trajectory":
        state["net"].trajectory(state["y"].data_ptr(), state["mean"].data_ptr(), mfma=True)
        return state["mean"].float()   # the network's output is FP32, written in double
    sm = state["sm"]
    if kind == "filter":
        return sm.filter(moments=False)[2]
    sm.set_trajectory_device(state["start"].data_ptr(), 0, state["cov0"])
    sm.iterate(case["iters"], want_delta=False)
    sm.result_device(state["mean"].data_ptr(), state["cov"].data_ptr())
    out = {"mean": state["mean"], "cov": state["cov"]}
    if case["lm"] > 0.0:
        out["objective"] = sm.objective()
    return out


def _slots(case):
    lo, hi = min(case["t_min"], case["t_max"]), case["t_max"]
    return case["tracks"] * (0.5 * (lo + hi) + 1.0)


def work(case):
    """Inputs read once, outputs written once; operations of the sequential
    recursion on the linearised model (a Kalman predict, update and RTS step
    per slot and iteration, plus 2 n + 1 sigma-point images under a
    regression) or of the network's products."""
    if case["kind"] == "gradient":
        n = case["windows"]
        params = 201876
        return {"bytes": 4.0 * (n * 64 * (4 + 5) + 2 * params), "flops": 6.0 * n * 16 * params}
    if case["kind"] == "trajectory":
        s = _slots(case)
        return {"bytes": 8.0 * s * (2 + 5) + 4.0 * 201876, "flops": 2.0 * 201876 * s / 4.0}
    nt = case.get("targets", 1)
    n, p = 5.0 * nt, 2.0 * nt
    word = 8.0 if case["precision"] == "f64" else 4.0
    s = _slots(case)
    filt = 2 * (2 * n ** 3) + 2 * (2 * p * n ** 2) + 2 * p ** 2 * n + p ** 3 / 3.0
    smo = n ** 3 / 3.0 + 2 * n ** 3 + 3 * (2 * n ** 3)
    reg = 0.0
    if case["lin"] != "taylor":
        reg = n ** 3 / 3.0 + 2 * n * (2 * n ** 2) + n ** 3 + 2 * n * (2 * p * n)
    if case["kind"] == "filter":
        return {"bytes": s * word * (n + n * n + p) + 8.0 * case["tracks"], "flops": s * (filt + reg)}
    return {"bytes": s * word * (n + p + n + n * n), "flops": case["iters"] * s * (filt + smo + reg)}


# ---------------------------------------------------------------------------
# The same in 64 bits, without the library
# ---------------------------------------------------------------------------

def _ct(x, dt):
    """Transition of stacked coordinated-turn targets and its Jacobian blocks, rows of states."""
    s = x.reshape(*x.shape[:-1], -1, 5)
    vx, vy, w = s[..., 2], s[..., 3], s[..., 4]
    a = w * dt
    small = np.abs(a) < 1e-2
    b = np.where(small, 1.0, a)
    a2 = a * a
    sa, ca = np.sin(a), np.cos(a)
    omc = 2.0 * np.sin(0.5 * a) ** 2
    s1 = dt * np.where(small, 1 - a2 / 6 * (1 - a2 / 20 * (1 - a2 / 42)), sa / b)
    s2 = dt * np.where(small, a / 2 * (1 - a2 / 12 * (1 - a2 / 30 * (1 - a2 / 56))), omc / b)
    d1 = dt * dt * np.where(small, -a / 3 * (1 - a2 / 10 * (1 - a2 / 28 * (1 - a2 / 54))), (a * ca - sa) / (b * b))
    d2 = dt * dt * np.where(small, 0.5 - a2 / 8 * (1 - a2 / 18 * (1 - a2 / 40)), (a * sa - omc) / (b * b))
    out = np.empty_like(s)
    out[..., 0] = s[..., 0] + s1 * vx - s2 * vy
    out[..., 1] = s[..., 1] + s2 * vx + s1 * vy
    out[..., 2] = ca * vx - sa * vy
    out[..., 3] = sa * vx + ca * vy
    out[..., 4] = w
    J = np.zeros(s.shape + (5,))
    for i in (0, 1, 4):
        J[..., i, i] = 1.0
    J[..., 0, 2], J[..., 0, 3], J[..., 0, 4] = s1, -s2, d1 * vx - d2 * vy
    J[..., 1, 2], J[..., 1, 3], J[..., 1, 4] = s2, s1, d2 * vx + d1 * vy
    J[..., 2, 2], J[..., 2, 3], J[..., 2, 4] = ca, -sa, -dt * out[..., 3]
    J[..., 3, 2], J[..., 3, 3], J[..., 3, 4] = sa, ca, dt * out[..., 2]
    return out.reshape(x.shape), J


def _bearings(x, sensors, owner):
    return np.arctan2(x[..., 5 * owner + 1] - sensors[:, 1], x[..., 5 * owner] - sensors[:, 0])


def _regress(lin, x, P, g, center=None):
    """Statistical linear regression of g at N(x, P), rows of slots."""
    n = x.shape[-1]
    L = np.linalg.cholesky(P)
    lam = 0.0 if lin == "cubature" else 1.0     # unscented: alpha = 1, kappa = 1
    gam = math.sqrt(n + lam)
    wj, w0 = 0.5 / (n + lam), lam / (n + lam)
    d = gam * np.swapaxes(L, -1, -2)            # row j = gamma L e_j
    zc = g(x)
    zp, zm = g(x[..., None, :] + d), g(x[..., None, :] - d)
    if center is not None:
        zp, zm = center(zp, zc[..., None, :]), center(zm, zc[..., None, :])
    zb = wj * (zp + zm).sum(-2) + w0 * zc
    D = wj * gam * (zp - zm)                     # rows j
    G = np.swapaxes(np.linalg.solve(np.swapaxes(L, -1, -2), D), -1, -2)
    rp, rm, r0 = zp - zb[..., None, :] - gam * D, zm - zb[..., None, :] + gam * D, zc - zb
    t = lambda r: np.swapaxes(r, -1, -2) @ r  # noqa: E731
    Lam = wj * (t(rp) + t(rm)) + w0 * r0[..., :, None] * r0[..., None, :]
    off = zb - (G @ x[..., None])[..., 0]
    return G, off, Lam


def _sym(A):
    return 0.5 * (A + np.swapaxes(A, -1, -2))


class _Exact:
    """Iterations of the sequential smoother in float64, vectorised over tracks
    (padded to the longest)."""

    def __init__(self, case, seed):
        self.case = case
        self.pb, start, cov = _problem(case, seed)
        if case["precision"] == "f32":
            start = start.astype(np.float32).astype(np.float64)
        pb = self.pb
        self.nt, self.nx, self.ny = pb.n_tracks, pb.nx, pb.ny
        self.len = pb.lengths
        self.Tm = int(self.len.max())
        first = pb.offsets[:-1] + np.arange(self.nt)
        k = np.arange(self.Tm + 1)
        self.valid = k[:, None] <= self.len[None, :]                       # [T+1, tracks]
        self.slot = np.where(self.valid, first[None, :] + k[:, None], first[None, :])
        row = np.where(self.valid, pb.offsets[None, :-1] + np.maximum(k[:, None] - 1, 0), 0)
        self.y = pb.y[row]
        self.x = start[self.slot]
        self.P = np.broadcast_to(cov, self.x.shape + (self.nx,)).copy()
        prm = pb.params[1:].reshape(self.ny, 3)
        self.sensors, self.owner = prm[:, :2], prm[:, 2].astype(np.int64)
        self.dt = pb.params[0]

    def linearise(self):
        pb, x, P = self.pb, self.x, self.P
        nx, ny = self.nx, self.ny
        f = lambda z: _ct(z, self.dt)[0]  # noqa: E731
        h = lambda z: _bearings(z, self.sensors, self.owner)  # noqa: E731
        hx = h(x)
        if self.case["lin"] == "taylor":
            fx, J = _ct(x, self.dt)
            F = np.zeros(x.shape + (nx,))
            for b in range(nx // 5):
                F[..., 5 * b:5 * b + 5, 5 * b:5 * b + 5] = J[..., b, :, :]
            c = fx - (F @ x[..., None])[..., 0]
            Qp = np.broadcast_to(pb.Q, F.shape)
            H = np.zeros(x.shape[:-1] + (ny, nx))
            for s in range(ny):
                o = 5 * self.owner[s]
                dx, dy = x[..., o] - self.sensors[s, 0], x[..., o + 1] - self.sensors[s, 1]
                r2 = dx * dx + dy * dy
                H[..., s, o], H[..., s, o + 1] = -dy / r2, dx / r2
            d = hx - (H @ x[..., None])[..., 0]
            Rp = np.broadcast_to(pb.R, x.shape[:-1] + (ny, ny))
        else:
            F, c, Lam = _regress(self.case["lin"], x, P, f)
            Qp = pb.Q + Lam
            H, d, Om = _regress(self.case["lin"], x, P, h, lambda z, zc: zc + wl.wrap_angle(z - zc))
            Rp = pb.R + Om
        return F, c, Qp, H, d, Rp, hx + wl.wrap_angle(self.y - hx)

    def _damp(self, m, P, k):
        lam = self.case.get("lm", 0.0)
        if not lam > 0.0:
            return m, P
        G = lam * P + np.eye(self.nx)
        m = m + (lam * P @ np.linalg.solve(np.swapaxes(G, -1, -2), (self.x[k] - m)[..., None]))[..., 0]
        return m, _sym(np.linalg.solve(G, P))

    def filter(self):
        F, c, Qp, H, d, Rp, yt = self.lin = self.linearise()
        pb = self.pb
        m, P = self._damp(pb.m0.copy(), pb.P0.copy(), 0)
        fm, fP = np.empty_like(self.x), np.empty(self.x.shape + (self.nx,))
        ll = np.zeros(self.nt)
        fm[0], fP[0] = m, P
        for k in range(1, self.Tm + 1):
            mp = (F[k - 1] @ m[..., None])[..., 0] + c[k - 1]
            Pp = F[k - 1] @ P @ np.swapaxes(F[k - 1], -1, -2) + Qp[k - 1]
            Ht = np.swapaxes(H[k], -1, -2)
            S = H[k] @ Pp @ Ht + Rp[k]
            r = yt[k] - d[k] - (H[k] @ mp[..., None])[..., 0]
            Sr = np.linalg.solve(S, np.concatenate([r[..., None], H[k] @ Pp], axis=-1))
            if self.case["kind"] == "filter":
                one = -0.5 * (np.linalg.slogdet(2.0 * np.pi * S)[1] + (r * Sr[..., 0]).sum(-1))
                ll += np.where(self.valid[k], one, 0.0)
            K = Pp @ Ht
            m = mp + (K @ Sr[..., :1])[..., 0]
            P = _sym(Pp - K @ Sr[..., 1:])
            m, P = self._damp(m, P, k)
            fm[k], fP[k] = m, P
        return fm, fP, ll

    def iterate(self):
        fm, fP, _ = self.filter()
        F, c, Qp = self.lin[:3]
        Pp = F @ fP @ np.swapaxes(F, -1, -2) + Qp
        E = np.swapaxes(np.linalg.solve(Pp, F @ fP), -1, -2)
        g = fm - (E @ ((F @ fm[..., None])[..., 0] + c)[..., None])[..., 0]
        L = _sym(fP - E @ F @ fP)
        xs, Ps = fm.copy(), fP.copy()
        last = self.len
        for k in range(self.Tm - 1, -1, -1):
            live = (k < last)
            x = g[k] + (E[k] @ xs[k + 1][..., None])[..., 0]
            P = L[k] + E[k] @ Ps[k + 1] @ np.swapaxes(E[k], -1, -2)
            xs[k] = np.where(live[:, None], x, fm[k])
            Ps[k] = np.where(live[:, None, None], _sym(P), fP[k])
        self.x, self.P = xs, Ps

    def objective(self):
        pb, x = self.pb, self.x
        d0 = x[0] - pb.m0
        J = 0.5 * (d0 * np.linalg.solve(pb.P0, d0[..., None])[..., 0]).sum(-1)
        fx = _ct(x[:-1], self.dt)[0]
        q = x[1:] - fx
        r = wl.wrap_angle(self.y[1:] - _bearings(x[1:], self.sensors, self.owner))
        t = 0.5 * ((q @ np.linalg.inv(pb.Q) * q).sum(-1) + (r @ np.linalg.inv(pb.R) * r).sum(-1))
        return J + np.where(self.valid[1:], t, 0.0).sum(0)

    def rows(self, a):
        return np.swapaxes(a, 0, 1)[np.swapaxes(self.valid, 0, 1)]


def _exact_net(theta, mu, sigma, x):
    """Normalised network output [n, W, nx] of features x [n, 2 ny, W], torch tensors of one type."""
    n = x.shape[0]
    C, P, H, L = 128, 4, 4, 16
    at = 0

    def take(*shape):
        nonlocal at
        size = math.prod(shape)
        v = theta[at:at + size].reshape(shape)
        at += size
        return v

    w, b = take(C, 4, P), take(C)
    h = torch.relu(torch.einsum("ncjk,ock->noj", x.reshape(n, 4, L, P), w) + b[:, None])
    for layer in range(H):
        w, b = take(C, C, 3), take(C)
        dil = 2 ** layer
        p = torch.nn.functional.pad(h, (dil, dil))
        z = sum(torch.matmul(w[:, :, k].contiguous(), p[:, :, k * dil:k * dil + L].contiguous()) for k in range(3))
        h = h + torch.relu(z + b[:, None])
    w, b = take(P * 5, C), take(P * 5)
    out = torch.matmul(w, h) + b[:, None]                       # [n, P nx, L]
    return out.reshape(n, P, 5, L).permute(0, 3, 1, 2).reshape(n, P * L, 5)


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "gradient":
        x, lab, idx = _windows(case, seed)
        _, theta, mu, sigma = _net_config()
        t = torch.from_numpy(theta).to(dev, torch.float64).requires_grad_(True)
        mu, sigma = (torch.from_numpy(v).to(dev, torch.float64) for v in (mu, sigma))
        out = _exact_net(t, mu, sigma, torch.from_numpy(x[idx]).to(dev, torch.float64))
        loss = ((out - (torch.from_numpy(lab[idx]).to(dev, torch.float64) - mu) / sigma) ** 2).mean()
        (grad,) = torch.autograd.grad(loss, t)
        return {"grad": grad.cpu().numpy(), "loss": np.float64(loss.item())}
    if kind == "trajectory":
        pb, _, _ = _problem(case, seed)
        _, theta, mu, sigma = _net_config()
        theta, mu, sigma = (torch.from_numpy(v).to(dev, torch.float64) for v in (theta, mu, sigma))
        W = 64
        rows, takes, base = [], [], 0    # base: windows of the tracks before
        for i in range(pb.n_tracks):
            T, o = int(pb.lengths[i]), int(pb.offsets[i])
            nw = -(-T // W)
            s = np.minimum(1 + W * np.arange(nw), max(1, T - W + 1))
            rows.append(o + np.minimum(s[:, None] + np.arange(W), T) - 1)
            k = np.maximum(np.arange(T + 1), 1)
            w = np.minimum((k - 1) // W, nw - 1)
            takes.append((base + w) * W + k - s[w])
            base += nw
        ang = torch.from_numpy(pb.y).to(dev)[torch.from_numpy(np.concatenate(rows)).to(dev)]
        x = torch.stack([ang[..., 0].sin(), ang[..., 0].cos(), ang[..., 1].sin(), ang[..., 1].cos()], dim=1)
        out = torch.cat([_exact_net(theta, mu, sigma, v) for v in x.split(4096)])
        states = mu + sigma * out.reshape(-1, 5)
        return states[torch.from_numpy(np.concatenate(takes)).to(dev)].cpu().numpy()
    steps = case.get("iters", 1) * max(case["t_min"], case["t_max"])
    slots = case["tracks"] * max(case["t_min"], case["t_max"])
    if steps * (4 if case.get("targets", 1) > 1 else 1) > 60000 or slots > 1500000:
        return None
    e = _Exact(case, seed)
    if kind == "filter":
        return e.filter()[2]
    for _ in range(case["iters"]):
        e.iterate()
    out = {"mean": e.rows(e.x), "cov": e.rows(e.P)}
    if case["lm"] > 0.0:
        out["objective"] = e.objective()
    return out
