"""Workloads of the planner for timing: the calls that a program built on the library makes, by size and direction.

Every case is one pass through the public entry points: plans of one robot cell (small, ordinary, warm-started in
contact, large), the simulator as a plant, an uneven batch of cells, a box-shaped object, the QP smoothing of samples
and the three kernels of the covariance adaptation.  Scenes, horizons and sample counts are those of the seeded
workloads (``workloads.PLAN``, ``packed_scenes``, ``task_scene``, ``qp_params``); the seed chooses the scene (link
densities, boxes), the start state, the nominal controls and the noise.
"""
import math

import numpy as np
import torch

import paper_2511_21264_amd as mp
import workloads as W

NU, NX = 14, 55
MAX_STEPS = 65536 * 64  # samples x control steps x iterations of the largest listed plan


def listed():
    return [
        # the plant of a closed loop: the simulator runs one state two control steps on; latency only
        dict(name="plant_step", kind="simulate", boxes=3, n=1, H=2),
        # the smallest plan of the workloads (64 samples, no boxes): launches and short dependent kernels
        dict(name="plan_small", kind="plan", boxes=0, K=64, H=20, M=5, coarse=True),
        # the headline workload: one cold plan of 1024 samples over 64 steps, 10 iterations, 3 boxes
        dict(name="plan_main", kind="plan", boxes=3, K=1024, H=64, M=10, coarse=False),
        # a warm-started replan with both pads squeezing the ball (elites, learning rate, best sequence), as a
        # closed loop makes them: arm contacts in every substep
        dict(name="replan_grasp", kind="replan", boxes=3, K=1024, H=64, M=3),
        # the 8-box workload, an odd sample count over a long ragged horizon, one iteration
        dict(name="plan_8box", kind="plan", boxes=8, K=4093, H=100, M=1, coarse=False),
        # throughput: one iteration of 65536 samples
        dict(name="plan_64k", kind="plan", boxes=3, K=65536, H=64, M=1, coarse=False),
        # an uneven batch of 12 cells (K 256..4096, H 32..128, 0..12 boxes), two iterations in packed launches
        dict(name="batch_12", kind="batch", n=12, M=2, mix=0),
        # the tray-moving phase: a box-shaped object with table contacts in every substep, the further cost terms
        dict(name="tray_move", kind="task", task="tray", phase="move", K=1024, H=64, M=1),
        # the QP smoothing of one iteration's samples (60 ADMM iterations)
        dict(name="project", kind="project", K=1024, H=64, iters=60),
        # covariance adaptation over the whole sequence (n = 14 H = 896): update, factor, correlated samples
        dict(name="cov_update", kind="cov_update", K=1024, H=64),
        dict(name="cholesky", kind="cholesky", H=64),
        dict(name="sample_full", kind="sample_full", K=1024, H=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["simulate", "plan", "plan", "plan", "replan", "batch", "task", "project", "project",
                       "cov_update", "cholesky", "sample_full"])
    if kind == "simulate":
        return dict(kind=kind, boxes=rng.randint(0, 12), n=_log(rng, 1, 512), H=rng.randint(1, 16))
    if kind == "plan":
        K = _log(rng, 24, 65536)
        H = rng.randint(8, 100)
        M = max(1, min(rng.randint(1, 6), MAX_STEPS // (K * H)))
        return dict(kind=kind, boxes=rng.randint(0, 12), K=K, H=min(H, max(8, MAX_STEPS // (K * M))), M=M,
                    coarse=rng.random() < 0.25)
    if kind == "replan":
        return dict(kind=kind, boxes=rng.choice([3, 8]), K=_log(rng, 128, 4096), H=rng.randint(16, 100),
                    M=rng.randint(1, 3))
    if kind == "batch":
        return dict(kind=kind, n=rng.randint(2, 12), M=rng.randint(1, 2), mix=rng.randint(1, 9999))
    if kind == "task":
        task, phase = rng.choice([("tray", "pick"), ("tray", "move"), ("handover", "pick"), ("handover", "pass"),
                                  ("handover", "place")])
        return dict(kind=kind, task=task, phase=phase, K=_log(rng, 64, 4096), H=rng.randint(8, 64), M=1)
    if kind == "project":
        return dict(kind=kind, K=_log(rng, 1, 4096), H=rng.choice([64, rng.randint(3, 63), rng.randint(65, 128)]),
                    iters=60)
    if kind == "cov_update":
        return dict(kind=kind, K=_log(rng, 32, 4096), H=rng.randint(4, 100))
    if kind == "cholesky":
        return dict(kind=kind, H=rng.randint(3, 100))
    return dict(kind=kind, K=_log(rng, 8, 4096), H=rng.randint(4, 100))


# ------------------------------------------------------------------------------------------------- inputs


def _dev(a, dtype=torch.float32):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _start(scene, rng, grasp=0.0):
    """A start state near the home pose; grasp > 0: both pads pressed on the ball at its centre's height, the
    commanded position `grasp` metres further in."""
    x = W.initial_state(scene)
    if grasp > 0.0:
        inner = float(scene["ball_r"]) + W.PAD_RAD - 0.001
        x[0:14] = np.tile(_arm_reach(inner), 2)
        x[28:42] = np.tile(_arm_reach(inner - grasp), 2)
    noise = rng.uniform(-1.0, 1.0, 14) * (0.002 if grasp > 0.0 else 0.05)
    x[0:14] += noise
    x[28:42] += noise
    x[14:28] = rng.uniform(-0.05, 0.05, 14)
    return x


def _arm_reach(dx, z=0.09):
    """Joint values that put a pad dx outside the ball's centre line at height z: the planar chain of the arm's
    second, fourth and sixth joints with the wrist as in the home pose, by the law of cosines."""
    L = W.LINK_LEN
    base_x, wrist = abs(W.BASE_POS[0][0]), W.Q_HOME_ARM[5]
    l1 = L[1] + L[2]
    fore = (L[3] + L[4]) + (L[5] + L[6]) * complex(math.cos(wrist), math.sin(wrist))
    tx, tz = base_x - dx, z - L[0]
    r = math.hypot(tx, tz)
    el = math.pi - math.acos((l1 ** 2 + abs(fore) ** 2 - r ** 2) / (2 * l1 * abs(fore)))
    sh = math.atan2(tx, tz) - math.atan2(abs(fore) * math.sin(el), l1 + abs(fore) * math.cos(el))
    q = np.array(W.Q_HOME_ARM, dtype=np.float64)
    q[1], q[3] = sh, el - math.atan2(fore.imag, fore.real)
    return q


def _nominal(rng, H, scale):
    """A smooth nominal: a slow random direction per joint."""
    return scale * rng.normal(size=(1, NU)) * np.linspace(1.0, 0.3, H)[:, None]


def _ball_scene(case, seed, boxes):
    coarse = bool(case.get("coarse"))
    return W.make_scene(2, seed % 997, n_box=boxes, h=0.01 if coarse else 0.002, n_sub=2 if coarse else 5)


def _request(ctx, scene, rng, K, H, M, noise_seed, **kw):
    """The arrays and options of one plan request, on the GPU."""
    return dict(scene=mp.Scene(ctx, scene), x0=_dev(_start(scene, rng, kw.pop("grasp", 0.0))),
                nominal_U=_dev(_nominal(rng, H, 0.05)), K=K, H=H, lam=0.1, sigma=_dev(np.full(NU, 0.3)),
                U_new=torch.zeros((H, NU), device="cuda"), costs=torch.zeros(K, device="cuda"), M=M,
                seed=noise_seed, **kw)


def _batch_sizes(case):
    """(K, H) of every request of an uneven batch: the case's `mix` chooses them."""
    rng = np.random.Generator(np.random.PCG64(77_000 + case["mix"]))
    return [(int(rng.integers(256, 4097)), int(rng.integers(32, 129))) for _ in range(case["n"])]


def _weights(gen, K):
    """Normalised exponential weights with an effective sample size of a tenth of the samples."""
    return torch.softmax(1.5 * torch.randn(K, generator=gen, dtype=torch.float64), 0)


def _covariance(gen, n, rank=64):
    """A covariance as the adaptation leaves it: part of the initial diagonal, a scatter of weighted samples."""
    X = torch.randn(rank, n, generator=gen, dtype=torch.float64) * 0.3
    w = _weights(gen, rank)
    return (0.045 + 1e-4) * torch.eye(n, dtype=torch.float64) + 0.5 * (X * w[:, None]).T @ X


def _cpu_inputs(case, seed):
    """The host-side inputs of the block cases, from the seed alone (numpy or torch, on the CPU)."""
    kind = case["kind"]
    gen = torch.Generator().manual_seed(seed)
    H = case["H"]
    n = NU * H
    if kind == "project":
        scene = W.make_scene(2, seed % 997)
        U = 0.05 * torch.randn(1, 1, NU, generator=gen) + 0.3 * torch.randn(case["K"], H, NU, generator=gen)
        return scene, W.initial_state(scene), U.float()
    if kind == "cov_update":
        nu = 0.1 * torch.randn(n, generator=gen, dtype=torch.float64)
        U = (nu + 0.3 * torch.randn(case["K"], n, generator=gen, dtype=torch.float64)).clamp(-1.5, 1.5).float()
        w = _weights(gen, case["K"])
        nu_new = 0.5 * nu + 0.5 * (w @ U.double())
        return U, w, nu_new, _covariance(gen, n)
    if kind == "cholesky":
        return (_covariance(gen, n),)
    nu = (0.1 * torch.randn(H, NU, generator=gen)).float()
    return nu, torch.linalg.cholesky(_covariance(gen, n)).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    ctx = mp.Context(0)
    rng = np.random.Generator(np.random.PCG64(seed))
    s = dict(kind=kind, ctx=ctx, case=case)
    if kind == "simulate":
        scene = _ball_scene(case, seed, case["boxes"])
        n, H = case["n"], case["H"]
        X = np.stack([_start(scene, rng) for _ in range(n)])
        s.update(scene=mp.Scene(ctx, scene), X=_dev(X), U=_dev(rng.uniform(-0.5, 0.5, (n, H, NU))),
                 costs=torch.zeros(n, device="cuda"), terms=torch.zeros((n, mp.NTERMS), device="cuda"),
                 X_out=torch.zeros((n, NX), device="cuda"))
    elif kind == "plan":
        s["req"] = _request(ctx, _ball_scene(case, seed, case["boxes"]), rng, case["K"], case["H"], case["M"], seed)
    elif kind == "replan":
        s["req"] = _request(ctx, _ball_scene(case, seed, case["boxes"]), rng, case["K"], case["H"], case["M"], seed,
                            grasp=0.02, eta=0.8, n_elite=min(32, case["K"]))
        s["U_best"] = torch.zeros((case["H"], NU), device="cuda")
    elif kind == "batch":
        s["reqs"] = []
        for i, (K, H) in enumerate(_batch_sizes(case)):
            scene = W.make_scene(4, (seed + i) % 997)
            s["reqs"].append(_request(ctx, scene, rng, K, H, case["M"], seed + i))
    elif kind == "task":
        scene = W.task_scene(case["task"], case["phase"], seed % 997)
        s["req"] = _request(ctx, scene, rng, case["K"], case["H"], case["M"], seed)
    elif kind == "project":
        scene, x0, U = _cpu_inputs(case, seed)
        s.update(scene=mp.Scene(ctx, scene), x0=_dev(x0), U=U.cuda(), out=torch.zeros_like(U, device="cuda"),
                 qp=mp.make_qp(W.qp_params(2, iters=case["iters"])))
    elif kind == "cov_update":
        U, w, nu_new, S = _cpu_inputs(case, seed)
        s.update(U=U.cuda(), w=w.cuda(), nu=nu_new.cuda(), S=S.cuda(), out=torch.zeros_like(S, device="cuda"))
    elif kind == "cholesky":
        S, = _cpu_inputs(case, seed)
        s.update(S=S.cuda(), out=torch.zeros_like(S, device="cuda"))
    elif kind == "sample_full":
        nu, L = _cpu_inputs(case, seed)
        s.update(nu=nu.cuda(), L=L.cuda(), seed=seed, out=torch.zeros((case["K"], case["H"], NU), device="cuda"))
    else:
        raise ValueError(kind)
    return s


# -------------------------------------------------------------------------------------------------- one pass


def run(s):
    kind, ctx, case = s["kind"], s["ctx"], s["case"]
    if kind == "simulate":
        mp.mppi_simulate(ctx, s["scene"], s["X"], s["U"], s["costs"], s["terms"], s["X_out"], sync=False)
        return s["costs"], s["terms"], s["X_out"]
    if kind in ("plan", "task"):
        r = s["req"]
        mp.mppi_plan(ctx, r["scene"], r["x0"], r["nominal_U"], r["K"], r["H"], r["lam"], r["sigma"], r["U_new"],
                     r["costs"], M=r["M"], seed=r["seed"], want_stats=False)
        return r["U_new"], r["costs"]
    if kind == "replan":
        r = s["req"]
        mp.mppi_plan_best(ctx, r["scene"], r["x0"], r["nominal_U"], r["K"], r["H"], r["lam"], r["sigma"], r["U_new"],
                          s["U_best"], r["costs"], M=r["M"], seed=r["seed"], eta=r["eta"], n_elite=r["n_elite"],
                          want_stats=False)
        return r["U_new"], s["U_best"], r["costs"]
    if kind == "batch":
        mp.mppi_plan_batch(ctx, s["reqs"])
        return [(r["U_new"], r["costs"]) for r in s["reqs"]]
    if kind == "project":
        mp.mppi_project(ctx, s["scene"], s["x0"], s["U"], s["out"], s["qp"], x0_shared=True, sync=False)
    elif kind == "cov_update":
        mp.mppi_cov_update(ctx, s["U"], s["w"], s["nu"], s["S"], s["out"], 0.5, 1e-4, sync=False)
    elif kind == "cholesky":
        mp.mppi_cholesky(ctx, s["S"], s["out"])
    else:
        mp.mppi_sample_full(ctx, s["nu"], s["L"], s["seed"], 0, case["K"], s["out"], 1.5, sync=False)
    return s["out"]


# ------------------------------------------------------------------------------------------ what it cannot do without


def _rollout_work(steps, n_sub, boxes):
    """Operations of `steps` control steps without contacts: free dynamics and one box test a pair in every substep,
    the stage cost in every step."""
    pairs, cost_pairs = 76 + 15 * boxes, 49 + 14 * boxes
    return steps * (n_sub * (6478 + 6 * pairs) + 596 + 11 * cost_pairs)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        sizes = _batch_sizes(case)
        return dict(bytes=sum(4 * (K + 2 * H * NU + NX + NU) for K, H in sizes),
                    flops=_rollout_work(case["M"] * sum(K * H for K, H in sizes), 5, 6))
    H = case["H"]
    n = NU * H
    if kind == "simulate":
        N = case["n"]
        return dict(bytes=4 * N * (2 * NX + n + 1 + 17), flops=_rollout_work(N * H, 5, case["boxes"]))
    if kind in ("plan", "replan", "task"):
        steps = case["K"] * H * case["M"]
        return dict(bytes=4 * (case["K"] + 2 * n + NX + NU),
                    flops=_rollout_work(steps, 2 if case.get("coarse") else 5, case.get("boxes", 3)))
    if kind == "project":  # the product with the H x H inverse in every iteration of every sequence
        return dict(bytes=8.0 * case["K"] * n, flops=2.0 * case["K"] * NU * case["iters"] * H * H)
    if kind == "cov_update":
        return dict(bytes=4.0 * case["K"] * n + 12.0 * n * n, flops=1.0 * case["K"] * n * (n + 1))
    if kind == "cholesky":
        return dict(bytes=12.0 * n * n, flops=n ** 3 / 3.0)
    return dict(bytes=4.0 * n * n + 4.0 * case["K"] * n, flops=1.0 * case["K"] * n * (n + 1))


# ------------------------------------------------------------------------------------------------ in 64 bits


def _philox_normals(seed, K, H):
    """Philox4x32-10 words of the counters (j, k, q, 0), uniforms in (0, 1] from 24 bits, Box-Muller: [K, H, 14]."""
    j, k, q = (a.astype(np.uint64) for a in np.meshgrid(np.arange(K), np.arange(H), np.arange(4), indexing="ij"))
    c = [j, k, q, np.zeros_like(j)]
    lo = np.uint64(0xFFFFFFFF)
    k0, k1 = np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ k0, b & lo, (a >> np.uint64(32)) ^ c[3] ^ k1, a & lo]
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & lo, (k1 + np.uint64(0xBB67AE85)) & lo
    u = [((w >> np.uint64(8)).astype(np.float64) + 1.0) * 2.0 ** -24 for w in c]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        r = np.sqrt(-2.0 * np.log(a))
        z += [r * np.cos(2.0 * np.pi * b), r * np.sin(2.0 * np.pi * b)]
    return np.stack(z, -1).reshape(K, H, 16)[..., :NU]


def _admm(U, q0, dt, p, u_max):
    """The fixed number of over-relaxed ADMM iterations on A = [I; D1; D2; prefix sums], every joint a QP."""
    K, H, _ = U.shape
    I = torch.eye(H, dtype=torch.float64, device=U.device)
    D1 = (I[1:] - I[:-1])
    D2 = (I[2:] - 2.0 * I[1:-1] + I[:-2])
    A = torch.cat([I, D1, D2, torch.tril(torch.ones_like(I))])
    one = lambda rows, v: torch.full((rows, 1), v, dtype=torch.float64, device=U.device)  # noqa: E731
    P = torch.linalg.inv(I + p["rho"] * A.T @ A)
    out = torch.empty_like(U)
    for d in range(NU):
        edge = torch.cat([one(H, u_max), one(H - 1, p["acc_max"] * dt), one(H - 2, p["jerk_max"] * dt * dt)])
        lo = torch.cat([-edge, one(H, (p["pos_lo"][d] - q0[d]) / dt)])
        hi = torch.cat([edge, one(H, (p["pos_hi"][d] - q0[d]) / dt)])
        v0 = U[:, :, d].T.contiguous()
        v, z = v0, torch.clamp(A @ v0, lo, hi)
        w = torch.zeros_like(z)
        for _ in range(p["iters"]):
            v = P @ (v0 + p["rho"] * (A.T @ (z - w)))
            a = p["alpha"] * (A @ v) + (1.0 - p["alpha"]) * z
            z = torch.clamp(a + w, lo, hi)
            w = w + a - z
        out[:, :, d] = v.clamp(-u_max, u_max).T
    return out


def exact(case, seed):
    """None for the simulator and the plans: hundreds of dependent physics substeps with contacts have no plain
    expression in torch or numpy, and a second simulator in 64 bits takes minutes at these sizes."""
    kind = case["kind"]
    if kind == "project":
        scene, x0, U = _cpu_inputs(case, seed)
        return _admm(U.double().cuda(), x0.astype(np.float32)[28:42].astype(np.float64), scene["h"] * scene["n_sub"],
                     W.qp_params(2, iters=case["iters"]), float(scene["u_max"]))
    if kind == "cov_update":
        U, w, nu, S = (t.cuda() for t in _cpu_inputs(case, seed))
        D = U.double() - nu
        G = (D * w[:, None]).T.contiguous() @ D / w.sum()
        return 0.5 * S + 0.5 * G + 1e-4 * torch.eye(S.shape[0], dtype=torch.float64, device="cuda")
    if kind == "cholesky":
        return torch.linalg.cholesky(_cpu_inputs(case, seed)[0]).cuda()
    if kind == "sample_full":
        nu, L = _cpu_inputs(case, seed)
        Z = torch.tensor(_philox_normals(seed, case["K"], case["H"]).reshape(case["K"], -1), device="cuda")
        U = nu.double().cuda().reshape(1, -1) + Z @ L.T.contiguous().cuda()
        return U.clamp(-1.5, 1.5).reshape(case["K"], case["H"], NU)
    return None
