"""Workloads by which the speed of the library is followed.

Each case is one call pattern of a program that uses the library: batches of
centroidal MPC problems solved through ``Solver`` (single robots, small groups,
training batches, ragged horizons, BF16 operators, hand contacts, long
horizons), the serving loop, the steps before and after a solve, and a whole
control tick of a training loop.  Inputs follow the generator configurations of
``mpcgen`` (same physics and distributions, drawn here on the GPU).  ``exact``
solves the same problems in 64 bits with a plain torch interior point.
"""
import math

import torch

from paper_2606_05687_amd import binding

NX = 13
GRAVITY = 9.81
GAIT = 0.4
HAND_NOMINAL = ((0.35, 0.20, 0.25), (0.35, -0.20, 0.25))
HAND_FRAME = ((0.0, 0.0, -1.0), (0.0, 1.0, 0.0), (1.0, 0.0, 0.0))

# Settings a program passes to Solver.  "default" passes none; the others are
# the schedules the benchmark and the autotuner settle on for the workloads.
SCHEDULES = {
    "default": {},
    "tuned": dict(form=1, iters=3, rho=1.0, refine_passes=12, first_passes=0),
    "packed": dict(form=-1, iters=2, rho=3.0, refine_passes=16, first_passes=0),
    "bf16": dict(form=1, iters=3, rho=10.0, refine_passes=12, first_passes=0, precision=1),
    "hands": dict(form=1, iters=5, rho=10.0),
    "long": dict(form=2, iters=3, rho=1.0, ipm_iters=150, polish_passes=20, kkt_tol=1e-10),
    "long_scan": dict(form=2, iters=3, rho=1.0, ipm_iters=150, polish_passes=20, kkt_tol=1e-10,
                      scan=8),
}


def _solve(name, batch, n, schedule, n_min=0, contacts=2, offsets=False, dt=0.03, duty=0.6,
           push=0.5):
    return dict(name=name, kind="solve", batch=batch, n=n, n_min=n_min or n, schedule=schedule,
                contacts=contacts, offsets=offsets, dt=dt, duty=duty, push=push)


def listed():
    return [
        # one robot's controller: a single problem per control tick, default
        # settings, a tracked input reference and disturbances; latency counts
        _solve("robot_b1_n10", 1, 10, "default", offsets=True, dt=0.04, duty=0.5),
        # a small group of environments (the generator's small_b64_n10)
        _solve("small_b64_n10", 64, 10, "default", dt=0.04, duty=0.5, push=0.0),
        # a training loop's control tick for 4096 environments: stage matrices
        # from compact physics, the solve, the landmark store and the reward
        dict(name="tick_b4096_n10", kind="tick", batch=4096, n=10, n_min=10, schedule="default",
             contacts=2, offsets=False, dt=0.04, duty=0.6, push=0.5, landmarks=5),
        # the benchmark workload (plain_b4096_n20) under its tuned schedule
        _solve("plain_b4096_n20", 4096, 20, "tuned"),
        # ragged horizons of mixed gaits (uneven_b16384's mix at an odd batch)
        _solve("uneven_b3001_n60", 3001, 60, "packed", n_min=10, duty=0.0),
        # BF16 operators (precision_b16384_n30's problems, a quarter of them)
        _solve("bf16_b4096_n30", 4096, 30, "bf16"),
        # loco-manipulation, four contacts (hands_b4096_n20), and a small group
        _solve("hands_b4096_n20", 4096, 20, "hands", contacts=4),
        _solve("hands_b37_n13", 37, 13, "hands", contacts=4, offsets=True),
        # a few long horizons (long_b64_n400's shape at a middle length)
        _solve("long_b24_n160", 24, 160, "long", n_min=80),
        # requests of environment groups through the serving loop, warm start
        dict(name="serving_r16_b64_n60", kind="serving", batch=64, requests=16, n=60, n_min=10,
             schedule="packed", contacts=2, offsets=False, dt=0.03, duty=0.0, push=0.5),
        # stage matrices of the benchmark's batch from compact physics
        dict(name="dynamics_b4096_n20", kind="dynamics", batch=4096, n=20, n_min=20, model="srb",
             dt=0.03),
        # landmark store and reward of one tick
        dict(name="landmarks_e4096_n20", kind="landmarks", batch=4096, n=20, n_min=20,
             landmarks=5, ticks=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("default", "default", "default", "tuned", "tuned", "packed", "bf16",
                       "hands", "hands", "long", "serving", "dynamics", "landmarks", "tick"))
    offsets = rng.random() < 0.5
    duty = rng.choice((0.0, 0.5, 0.6))
    dt = rng.choice((0.03, 0.04))
    if kind == "default":
        n = rng.randint(3, 24)
        n_min = rng.choice((n, max(2, n // 2)))
        return _solve("", _log(rng, 1, 2048), n, "default", n_min=n_min, offsets=offsets, dt=dt,
                      duty=duty)
    if kind == "tuned":
        n = rng.randint(8, 40)
        n_min = rng.choice((n, max(2, n // 2)))
        return _solve("", _log(rng, 64, 82000 // n), n, "tuned", n_min=n_min, offsets=offsets,
                      dt=dt, duty=duty)
    if kind == "packed":
        n = rng.randint(24, 64)
        return _solve("", _log(rng, 64, 3000), n, "packed", n_min=rng.randint(5, 20),
                      offsets=offsets, duty=duty)
    if kind == "bf16":
        n = rng.randint(8, 40)
        return _solve("", _log(rng, 64, 80000 // n), n, "bf16", offsets=offsets, duty=0.6)
    if kind == "hands":
        n = rng.randint(3, 40)
        n_min = rng.choice((n, max(2, n // 2)))
        return _solve("", _log(rng, 4, 40000 // n), n, "hands", n_min=n_min, contacts=4,
                      offsets=offsets, duty=duty)
    if kind == "long":
        n = rng.randint(70, 160)
        return _solve("", rng.randint(2, 24), n, rng.choice(("long", "long_scan")),
                      n_min=rng.choice((n, n // 2)), offsets=offsets, duty=0.6)
    if kind == "serving":
        return dict(kind="serving", batch=_log(rng, 8, 96), requests=rng.randint(2, 16),
                    n=rng.randint(20, 60), n_min=10, schedule="packed", contacts=2,
                    offsets=offsets, dt=0.03, duty=0.0, push=0.5)
    if kind == "tick":
        return dict(kind="tick", batch=_log(rng, 64, 4096), n=rng.randint(5, 10), n_min=5,
                    schedule="default", contacts=2, offsets=False, dt=dt, duty=duty, push=0.5,
                    landmarks=rng.randint(2, 8))
    n = rng.randint(5, 64)
    batch = _log(rng, 16, 160000 // n)
    if kind == "dynamics":
        return dict(kind="dynamics", batch=batch, n=n, n_min=rng.choice((n, max(2, n // 2))),
                    model=rng.choice(("srb", "momentum")), dt=dt)
    return dict(kind="landmarks", batch=batch, n=n, n_min=rng.choice((n, max(2, n // 2))),
                landmarks=rng.randint(1, 12), ticks=rng.randint(1, 6))


# ------------------------------------------------------------------- inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


class _Rng:
    """Draws in float64 on the device, from one seed."""

    def __init__(self, seed):
        self.dev = _device()
        self.g = torch.Generator(device=self.dev).manual_seed(int(seed) % (1 << 62))

    def uni(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=self.g, device=self.dev,
                                           dtype=torch.float64)

    def nrm(self, sd, *shape):
        return sd * torch.randn(shape, generator=self.g, device=self.dev, dtype=torch.float64)

    def ints(self, lo, hi, *shape):
        return torch.randint(lo, hi + 1, shape, generator=self.g, device=self.dev)


def _horizons(r, case):
    N = r.ints(case["n_min"], case["n"], case["batch"])
    N[0] = case["n"]
    return N


def _rotz(psi):
    c, s, o, i = torch.cos(psi), torch.sin(psi), torch.zeros_like(psi), torch.ones_like(psi)
    return torch.stack((c, -s, o, s, c, o, o, o, i), -1).reshape(psi.shape + (3, 3))


def _skew(v):
    x, y, z = v.unbind(-1)
    o = torch.zeros_like(x)
    return torch.stack((o, -z, y, z, o, -x, -y, x, o), -1).reshape(v.shape[:-1] + (3, 3))


def _physics(r, case, N):
    """Compact physics of a batch, float32 device tensors (one yaw per problem,
    the reference moving at a constant speed, the feet where they stand)."""
    B, n, dt = case["batch"], case["n"], case["dt"]
    k = torch.arange(n, device=r.dev)
    valid = k[None, :] < N[:, None]
    yaw = r.uni(-math.pi, math.pi, B)
    Rz = _rotz(yaw)
    vel = Rz[:, :, 0] * r.uni(-1.0, 1.0, B, 1)
    com0 = torch.tensor([0.0, 0.0, 0.8], device=r.dev, dtype=torch.float64)
    cref = com0 + k[None, :, None] * dt * vel[:, None, :]
    side = torch.tensor([0.10, -0.10], device=r.dev, dtype=torch.float64)
    feet = Rz[:, None, :, 1] * side[None, :, None] + r.nrm(0.1, B, 2, 3)
    ph = dict(N=N.to(torch.int32), yaw_k=yaw[:, None] * valid, c_ref=cref * valid[..., None],
              feet=feet[:, None] * valid[:, :, None, None], mass=r.uni(30.0, 60.0, B),
              inertia=r.uni(1.0, 4.0, B, 3),
              dt=torch.full((B,), float(dt), device=r.dev, dtype=torch.float64))
    f32 = {key: v if key == "N" else v.to(torch.float32).contiguous() for key, v in ph.items()}
    return f32, dict(yaw=yaw, vel=vel, com0=com0, valid=valid)


def _matrices(ph, model="srb"):
    """A, B, e in float64 from compact physics (the formulas of the header)."""
    d = {k: v.double() for k, v in ph.items() if k != "N"}
    Bn, n = d["yaw_k"].shape
    dev = d["yaw_k"].device
    z = dict(device=dev, dtype=torch.float64)
    valid = (torch.arange(n, device=dev)[None, :] < ph["N"][:, None])[:, :, None, None]
    eye3 = torch.eye(3, **z)
    dt = d["dt"][:, None, None, None]
    mass = d["mass"][:, None, None, None]
    A = torch.eye(NX, **z).repeat(Bn, n, 1, 1)
    B = torch.zeros(Bn, n, NX, 12, **z)
    e = torch.zeros(Bn, n, NX, **z)
    arm = _skew(d["feet"] - d["c_ref"][:, :, None, :])          # [B, n, 2, 3, 3]
    if model == "momentum":
        A[:, :, 0:3, 3:6] = dt / mass * eye3
        for i in range(2):
            B[:, :, 3:6, 6 * i:6 * i + 3] = dt * eye3
            B[:, :, 6:9, 6 * i:6 * i + 3] = dt * arm[:, :, i]
            B[:, :, 6:9, 6 * i + 3:6 * i + 6] = dt * eye3
        e[:, :, 5] = -(d["dt"] * d["mass"])[:, None] * GRAVITY
    else:
        Rz = _rotz(d["yaw_k"])
        Iw = Rz @ ((1.0 / d["inertia"])[:, None, :, None] * Rz.transpose(-1, -2))
        A[:, :, 0:3, 6:9] = dt * Rz.transpose(-1, -2)
        A[:, :, 3:6, 9:12] = dt * eye3
        A[:, :, 11, 12] = d["dt"][:, None]
        for i in range(2):
            B[:, :, 6:9, 6 * i:6 * i + 3] = dt * (Iw @ arm[:, :, i])
            B[:, :, 6:9, 6 * i + 3:6 * i + 6] = dt * Iw
            B[:, :, 9:12, 6 * i:6 * i + 3] = dt / mass * eye3
    A = torch.where(valid, A, torch.eye(NX, **z))
    return A, B * valid, e * valid[..., 0]


def _problems(case, seed):
    """A batch of problems as float32 device tensors (the layout Solver takes)
    and the compact physics of its feet."""
    r = _Rng(seed)
    B, n, dt, nc = case["batch"], case["n"], case["dt"], case["contacts"]
    m = 6 * nc
    N = _horizons(r, case)
    ph, aux = _physics(r, case, N)
    valid, vel, yaw = aux["valid"], aux["vel"], aux["yaw"]
    k = torch.arange(n, device=r.dev)
    A, Bm, _ = _matrices(ph)
    z = dict(device=r.dev, dtype=torch.float64)
    mass = ph["mass"].double()
    xr = torch.zeros(B, n + 1, NX, **z)
    xr[:, :, 2] = yaw[:, None]
    xr[:, :, 3:6] = aux["com0"] + torch.arange(n + 1, **z)[None, :, None] * dt * vel[:, None, :]
    xr[:, :, 9:12] = vel[:, None, :]
    xr[:, :, 12] = -GRAVITY
    x0 = xr[:, 0].clone()
    x0[:, 9:12] += r.nrm(case["push"], B, 3)
    duty = r.uni(0.35, 0.65, B) if case["duty"] == 0.0 else torch.full((B,), case["duty"], **z)
    frac = (r.uni(0.0, 1.0, B)[:, None, None] + k[None, :, None] * dt / GAIT
            + torch.arange(2, **z) / 2) % 1.0
    contact = (frac < duty[:, None, None]) & valid[..., None]
    R = torch.full((B, m), 1e-5, **z)
    u_ref = torch.zeros(B, n, m, **z)
    u_prev = torch.zeros(B, m, **z)
    e = torch.zeros(B, n, NX, **z)
    if nc == 4:
        # both hands on one push cycle, a reference normal force each
        Rz = _rotz(yaw)
        frame = Rz @ torch.tensor(HAND_FRAME, **z)
        inv = Rz @ ((1.0 / ph["inertia"].double())[:, :, None] * Rz.transpose(-1, -2))
        hand = (r.uni(0.0, 1.0, B)[:, None] + k[None, :] * dt / (2 * GAIT)) % 1.0
        hand = (hand < r.uni(0.5, 1.0, B)[:, None]) & valid
        contact = torch.cat((contact, hand[..., None], hand[..., None]), -1)
        force = r.uni(40.0, 120.0, B, 2)
        off = r.nrm(0.05, B, 2, 3)
        Bh = torch.zeros(B, n, NX, 12, **z)
        for h in range(2):
            arm = Rz @ torch.tensor(HAND_NOMINAL[h], **z) + off[:, h]
            Bh[:, :, 6:9, 6 * h:6 * h + 3] = (dt * inv @ _skew(arm) @ frame)[:, None]
            Bh[:, :, 6:9, 6 * h + 3:6 * h + 6] = (dt * inv @ frame)[:, None]
            Bh[:, :, 9:12, 6 * h:6 * h + 3] = (dt * frame / mass[:, None, None])[:, None]
            u_ref[:, :, 12 + 6 * h + 2] = torch.where(hand, force[:, h, None], 0.0)
            R[:, 12 + 6 * h:15 + 6 * h] = 1e-3
        Bm = torch.cat((Bm, Bh * valid[:, :, None, None]), -1)
    if case["offsets"]:
        sd = torch.tensor([2e-3] * 6 + [0.02] * 6 + [1e-3], **z)
        e = r.nrm(1.0, B, n, NX) * sd * valid[..., None]
        for i in range(nc):
            sdf = torch.tensor([20.0, 20.0, 30.0, 5.0, 5.0, 5.0], **z)
            ref = r.nrm(1.0, B, n, 6) * sdf
            ref[..., 2] += 0.5 * mass[:, None] * GRAVITY if i < 2 else 0.0
            u_ref[:, :, 6 * i:6 * i + 6] += ref * valid[..., None]
            u_prev[:, 6 * i:6 * i + 3] = r.nrm(50.0, B, 3)
            u_prev[:, 6 * i + 3:6 * i + 6] = r.nrm(5.0, B, 3)
    dev = dict(A=A, B=Bm, e=e, x0=x0, u_prev=u_prev, x_ref=xr[:, 1:] * valid[..., None],
               u_ref=u_ref, Q=r.uni(1.0, 100.0, B, NX), R=R, mu=r.uni(0.3, 0.9, B),
               fz_max=torch.full((B,), 1000.0, **z), tau_max=torch.full((B,), 50.0, **z),
               weight=mass * GRAVITY)
    dev = {key: v.to(torch.float32).contiguous() for key, v in dev.items()}
    dev["N"] = N.to(torch.int32)
    dev["contact"] = contact.to(torch.uint8).contiguous()
    return dev, ph


def _landmark_inputs(case, seed):
    """Trajectories of a solve, the realised CoM, and the reward's weights."""
    r = _Rng(seed)
    B, n, L = case["batch"], case["n"], case["landmarks"]
    N = _horizons(r, case).to(torch.int32)
    x = r.nrm(0.3, B, n + 1, NX).to(torch.float32)
    past = r.nrm(0.3, L, B, n + 1, NX).to(torch.float32)
    com = r.nrm(0.3, B, 3).to(torch.float32)
    alpha = r.uni(0.2, 1.0, L).to(torch.float32)
    qc = torch.tensor([1.0, 1.0, 2.0], device=r.dev)
    return N, x, past, com, alpha, qc


def _offsets_of(N, L):
    """Landmark offsets n_l = 1 + floor(l (N - 1) / (L - 1)) per environment."""
    ls = torch.arange(L, device=N.device)
    return 1 + (ls[None, :] * (N.long()[:, None] - 1)) // max(1, L - 1) if L > 1 else \
        torch.ones(N.shape[0], 1, dtype=torch.long, device=N.device)


SIGMA = 0.5


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("solve", "tick"):
        dev, ph = _problems(case, seed)
        solver = binding.Solver(0, **SCHEDULES[case["schedule"]])
        state = dict(kind=kind, dev=dev, solver=solver, out=solver.alloc_out(dev))
        if kind == "tick":
            # the matrices are built each tick from the physics
            dev["A"], dev["B"] = torch.empty_like(dev["A"]), torch.empty_like(dev["B"])
            L, n = case["landmarks"], case["n"]
            r = _Rng(seed + 1)
            state.update(ph=ph, tick=n, com=(dev["x0"][:, 3:6] + 0.02).contiguous(),
                         ring=binding.LandmarkRing(case["batch"], L, n + 1),
                         alpha=r.uni(0.2, 1.0, L).to(torch.float32),
                         qc=torch.tensor([1.0, 1.0, 2.0], device=r.dev))
            # the previous tick's predictions, from the reference
            x = torch.cat((dev["x0"][:, None], dev["x_ref"]), 1).contiguous()
            state["ring"].push(x, dev["N"], state["tick"] - 1)
        return state
    if kind == "serving":
        reqs = []
        for q in range(case["requests"]):
            dev, _ = _problems(case, seed * 64 + q)
            reqs.append(dev)
        total = case["batch"] * case["requests"]
        server = binding.Server(0, lanes=2, capacity=max(64, total // 2), warm_slots=total,
                                **SCHEDULES[case["schedule"]])
        outs = [binding.Solver.alloc_out(None, d) for d in reqs]
        return dict(kind=kind, reqs=reqs, outs=outs, server=server, batch=case["batch"])
    if kind == "dynamics":
        r = _Rng(seed)
        N = _horizons(r, case)
        ph, _ = _physics(r, case, N)
        z = dict(device=r.dev, dtype=torch.float32)
        B, n = case["batch"], case["n"]
        return dict(kind=kind, ph=ph, model=case["model"], A=torch.empty(B, n, NX, NX, **z),
                    B=torch.empty(B, n, NX, 12, **z),
                    e=torch.empty(B, n, NX, **z) if case["model"] == "momentum" else None)
    N, x, past, com, alpha, qc = _landmark_inputs(case, seed)
    ring = binding.LandmarkRing(case["batch"], case["landmarks"],
                                case["n"] * case["ticks"] + 1, case["ticks"])
    tick = case["n"] * case["ticks"]
    # solves of earlier ticks whose predictions reach this tick: their l-th
    # landmark of the longest horizon
    offs = _offsets_of(torch.tensor([case["n"]], device=N.device), case["landmarks"])[0].tolist()
    for l, o in enumerate(offs):
        ring.push(past[l], N, tick - o * case["ticks"])
    return dict(kind=kind, ring=ring, x=x, N=N, com=com, alpha=alpha, qc=qc, tick=tick)


def run(s):
    kind = s["kind"]
    if kind == "solve":
        out = s["solver"].solve(s["dev"], s["out"])
        return {k: out[k] for k in ("u", "x", "status")}
    if kind == "tick":
        binding.build_dynamics(s["ph"], s["dev"]["A"], s["dev"]["B"])
        out = s["solver"].solve(s["dev"], s["out"])
        reward, used = s["ring"].reward(s["com"], s["tick"], s["alpha"], s["qc"], SIGMA)
        s["ring"].push(out["x"], s["dev"]["N"], s["tick"])
        return {"u": out["u"], "x": out["x"], "status": out["status"], "reward": reward,
                "used": used}
    if kind == "serving":
        tickets = [s["server"].submit(d, o, warm_base=q * s["batch"])
                   for q, (d, o) in enumerate(zip(s["reqs"], s["outs"]))]
        for t in tickets:
            s["server"].wait(t)
        return [{k: o[k] for k in ("u", "x", "status")} for o in s["outs"]]
    if kind == "dynamics":
        A, B, e = binding.build_dynamics(s["ph"], s["A"], s["B"], s["e"], model=s["model"])
        return {"A": A, "B": B} if e is None else {"A": A, "B": B, "e": e}
    reward, used = s["ring"].reward(s["com"], s["tick"], s["alpha"], s["qc"], SIGMA)
    s["ring"].push(s["x"], s["N"], s["tick"])
    return {"reward": reward, "used": used, "com": s["ring"].com, "tag": s["ring"].tag}


# --------------------------------------------------------------------- work


def work(case):
    """Bytes: every input read once, every output written once.  Flops of a
    solve: the sweeps the schedule asks for and one LQ solve of the horizon
    (backward recursion, rollout, costates), which no certified solve can do
    without; with four contacts one Newton step of the interior point."""
    B, n, kind = case["batch"], case["n"], case["kind"]
    S = B * (n + case["n_min"]) // 2          # stages
    if kind == "dynamics":
        out = 4 * (169 + 156 + (13 if case["model"] == "momentum" else 0))
        return {"bytes": B * n * (out + 40) + 24 * B, "flops": S * 250}
    if kind == "landmarks":
        L = case["landmarks"]
        return {"bytes": B * (L * (12 + 12 + 4) + L * 16 + 12 + 8 + 4), "flops": B * L * 12}
    m = 6 * case["contacts"]
    s = SCHEDULES[case["schedule"]]
    if kind == "serving":
        B, S = B * case["requests"], S * case["requests"]
    per_in = 4 * (169 + 13 * m + 13 + (13 + m if case["offsets"] else 0)) + case["contacts"]
    per_out = 4 * (m + 13)
    lift = 13 + m
    setup = 2 * (13 * lift * lift // 2 + lift ** 3 // 3)
    sweep = 2 * (lift * lift + 4 * 13 * 13 + 3 * 13 * m + m * m) + 20 * lift
    lq = 2 * (13 * 13 * 13 * 2 + 3 * 13 * 13 * m + 13 * m * m + m * m * (13 + m)) + 6 * 13 * lift
    flops = S * (setup + s.get("iters", 100) * sweep + lq)
    nbytes = S * (per_in + per_out) + B * 4 * (13 * 3 + 2 * m + 8)
    if kind == "tick":
        nbytes += S * 40 + B * case["landmarks"] * 44
    return {"bytes": nbytes, "flops": flops}


# -------------------------------------------------------------------- exact


def _rows(mu):
    """Wrench rows [B, 11, 6] of one contact: the friction pyramid, the normal
    force bound, the moment box."""
    B = mu.shape[0]
    G = torch.zeros(B, 11, 6, device=mu.device, dtype=torch.float64)
    for i, (j, sg) in enumerate(((0, 1), (0, -1), (1, 1), (1, -1))):
        G[:, i, j] = sg
        G[:, i, 2] = -mu
    G[:, 4, 2] = 1.0
    for a in range(3):
        G[:, 5 + a, 3 + a] = 1.0
        G[:, 8 + a, 3 + a] = -1.0
    return G


def _inverse(H):
    """Inverse of a batch of SPD matrices (Gauss-Jordan, no pivoting)."""
    m = H.shape[-1]
    M = torch.cat((H, torch.eye(m, device=H.device, dtype=H.dtype).expand_as(H)), -1).clone()
    for p in range(m):
        t = M[:, p] / M[:, p, p, None]
        M = torch.addcmul(M, M[:, :, p, None], t[:, None, :], value=-1.0)
        M[:, p] = t
    return M[:, :, m:]


def _optimum(dev, cap=100):
    """The optimum of every problem in 64 bits: a primal-dual interior point
    with Mehrotra's corrector, Newton steps by the Riccati recursion.  Returns
    u [B, n, m] and x [B, n + 1, 13], zero on padding."""
    d = {k: v.double() for k, v in dev.items() if k not in ("N", "contact")}
    A, Bm, e = d["A"], d["B"], d["e"]
    Bn, n, _, m = Bm.shape
    nc = m // 6
    valid = torch.arange(n, device=A.device)[None, :] < dev["N"][:, None]
    st = (dev["contact"] != 0) & valid[..., None]               # [B, n, nc]
    on = st.repeat_interleave(6, -1).double()                    # [B, n, m]
    Bm = Bm * on[:, :, None, :] * valid[:, :, None, None]
    A = torch.where(valid[:, :, None, None], A, torch.eye(NX, device=A.device, dtype=A.dtype))
    e = e * valid[..., None]
    Q = d["Q"][:, None, :] * valid[..., None]                    # per stage
    R = d["R"][:, None, :].expand(Bn, n, m)
    mg, tm = d["weight"], d["tau_max"]
    sc = torch.cat((mg[:, None].repeat(1, 5), tm[:, None].repeat(1, 6)), 1)
    G = _rows(d["mu"]) / sc[:, :, None]                          # scaled rows
    h = torch.zeros_like(sc)
    h[:, 4] = d["fz_max"]
    h[:, 5:] = tm[:, None]
    h = h / sc
    rows = st[..., None].double().expand(Bn, n, nc, 11)
    count = rows.sum((1, 2, 3)).clamp(min=1.0)
    Gb, hb = G[:, None, None], h[:, None, None]

    def g_of(u):                                                 # G u, [B, n, nc, 11]
        return (Gb @ u.view(Bn, n, nc, 6, 1))[..., 0]

    def gt_of(z):                                                # G^T z, [B, n, m]
        return (Gb.transpose(-1, -2) @ z[..., None])[..., 0].reshape(Bn, n, m)

    def roll(u, first, aff):
        x = [first]
        for k in range(n):
            y = (A[:, k] @ x[-1][:, :, None] + Bm[:, k] @ u[:, k, :, None])[:, :, 0]
            x.append(y + aff[:, k] if aff is not None else y)
        return torch.stack(x, 1)

    ns = st.sum(-1).clamp(min=1).double()
    u = torch.zeros(Bn, n, nc, 6, device=A.device, dtype=torch.float64)
    u[..., 2] = 0.5 * mg[:, None, None] / ns[..., None] * st
    u = u.reshape(Bn, n, m)
    x = roll(u, d["x0"], e)
    s = (hb - g_of(u)).clamp(min=1.0) * rows + (1 - rows)
    z = rows.clone()
    ur, xr = d["u_ref"], d["x_ref"]

    def per_problem(v):
        return v[:, None, None, None]

    left = torch.ones(Bn, device=A.device, dtype=torch.float64)
    best, least = u.clone(), torch.full_like(left, math.inf)
    for _ in range(cap):
        rp = (g_of(u) - hb + s) * rows
        mu = (s * z * rows).sum((1, 2, 3)) / count
        better = (mu < least) & (left < 1e-9)
        best = torch.where(better[:, None, None], u, best)
        least = torch.where(better, mu, least)
        # the linear residuals shrink by 1 - a per step; beyond this point only
        # the multipliers of active rows lose digits, the inputs gain none
        live = (mu > 1e-12) | (rp.abs().amax((1, 2, 3)) > 1e-11) | (left > 1e-11)
        if not bool(live.any()):
            break
        w = z / s * rows
        RR = torch.diag_embed(R.reshape(Bn, n, nc, 6)) + Gb.transpose(-1, -2) @ (w[..., None] * Gb)
        # factor
        S = torch.zeros(Bn, NX, NX, device=A.device, dtype=torch.float64)
        HI, K = [None] * n, [None] * n
        eye = torch.eye(m, device=A.device, dtype=torch.float64)
        for k in range(n - 1, -1, -1):
            W = S + torch.diag_embed(Q[:, k])
            WB, WA = W @ Bm[:, k], W @ A[:, k]
            H = Bm[:, k].transpose(-1, -2) @ WB
            for i in range(nc):
                H[:, 6 * i:6 * i + 6, 6 * i:6 * i + 6] += RR[:, k, i]
            H = H * on[:, k, :, None] * on[:, k, None, :] + eye * (1 - on[:, k])[:, None, :]
            HI[k] = _inverse(H)
            hx = (WB.transpose(-1, -2) @ A[:, k]) * on[:, k, :, None]
            K[k] = -HI[k] @ hx
            S = A[:, k].transpose(-1, -2) @ WA + hx.transpose(-1, -2) @ K[k]
            S = 0.5 * (S + S.transpose(-1, -2))

        def newton(target):
            cr = (z + (-target + z * rp) / s) * rows             # row coefficients
            rho = (R * (u - ur) + gt_of(cr)) * on
            lam = torch.zeros(Bn, NX, device=A.device, dtype=torch.float64)
            kap = [None] * n
            for k in range(n - 1, -1, -1):
                q = Q[:, k] * (x[:, k + 1] - xr[:, k]) + lam
                hw = (Bm[:, k].transpose(-1, -2) @ q[:, :, None])[:, :, 0] + rho[:, k]
                kap[k] = -(HI[k] @ hw[:, :, None])[:, :, 0]
                lam = (A[:, k].transpose(-1, -2) @ q[:, :, None]
                       + K[k].transpose(-1, -2) @ hw[:, :, None])[:, :, 0]
            dx = torch.zeros(Bn, NX, device=A.device, dtype=torch.float64)
            du = []
            for k in range(n):
                du.append((K[k] @ dx[:, :, None])[:, :, 0] + kap[k])
                dx = (A[:, k] @ dx[:, :, None] + Bm[:, k] @ du[-1][:, :, None])[:, :, 0]
            du = torch.stack(du, 1) * on
            ds = (-rp - g_of(du)) * rows
            dz = (-target - z * ds) / s * rows
            return du, ds, dz

        def limit(v, dv):
            r = torch.where((dv < 0) & (rows > 0), -v / dv, torch.full_like(v, math.inf))
            return r.amin((1, 2, 3)).clamp(max=1.0)

        du, ds, dz = newton(s * z)
        a = per_problem(torch.minimum(limit(s, ds), limit(z, dz)))
        mua = ((s + a * ds) * (z + a * dz) * rows).sum((1, 2, 3)) / count
        # centred well inside, short of the boundary: degenerate problems
        # otherwise stall with a few products far below the others
        sig = (mua / mu.clamp(min=1e-300)).clamp(min=0.45, max=1.0) ** 3
        du, ds, dz = newton(s * z + ds * dz - per_problem(sig * mu))
        a = 0.9 * torch.minimum(limit(s, ds), limit(z, dz))
        ok = live & torch.isfinite(du).all(-1).all(-1)
        a = torch.where(ok, a.clamp(max=1.0), torch.zeros_like(a))
        left = left * (1.0 - a)
        u = torch.where(ok[:, None, None], u + a[:, None, None] * du, u)
        s = torch.where(per_problem(ok), s + per_problem(a) * ds, s)
        z = torch.where(per_problem(ok), z + per_problem(a) * dz, z)
        x = roll(u, d["x0"], e)
    u = best
    x = roll(u, d["x0"], e)
    k1 = torch.arange(n + 1, device=A.device)[None, :] <= dev["N"][:, None]
    return u * on, x * k1[..., None]


def exact(case, seed):
    kind = case["kind"]
    if kind == "dynamics":
        r = _Rng(seed)
        N = _horizons(r, case)
        ph, _ = _physics(r, case, N)
        A, B, e = _matrices(ph, case["model"])
        return {"A": A, "B": B, "e": e} if case["model"] == "momentum" else {"A": A, "B": B}
    if kind == "landmarks":
        N, x, past, com, alpha, qc = _landmark_inputs(case, seed)
        L, d, n, B = case["landmarks"], case["ticks"], case["n"], case["batch"]
        tick, ring = n * d, n * d + 1
        store = torch.zeros(B, ring, L, 3, device=N.device, dtype=torch.float64)
        tag = torch.full((B, ring, L), -1, device=N.device, dtype=torch.long)
        offs, ls = _offsets_of(N, L), torch.arange(L, device=N.device)
        env = torch.arange(B, device=N.device)[:, None]

        def push(traj, t):
            at = (t + offs * d) % ring
            store[env, at, ls[None, :]] = traj[env, offs, 3:6].double()
            tag[env, at, ls[None, :]] = t + offs * d

        for l, o in enumerate(_offsets_of(torch.tensor([n], device=N.device), L)[0].tolist()):
            push(past[l], tick - o * d)
        # run() rewards a tick, then pushes its own solve
        hit = (tag[:, tick % ring] == tick).double()
        err = com.double()[:, None] - store[:, tick % ring]
        cost = (err * err * qc.double()).sum(-1) * alpha.double() * hit
        reward = torch.exp(-cost.sum(-1) / SIGMA ** 2)
        push(x, tick)
        return {"reward": reward, "used": None, "com": store, "tag": None}
    if kind == "serving":
        got = []
        for q in range(case["requests"]):
            dev, _ = _problems(case, seed * 64 + q)
            got.append(dev)
        u, x = _optimum({k: torch.cat([g[k] for g in got]) for k in got[0]})
        B = case["batch"]
        return [{"u": u[q * B:(q + 1) * B], "x": x[q * B:(q + 1) * B], "status": None}
                for q in range(case["requests"])]
    dev, ph = _problems(case, seed)
    if kind == "solve":
        u, x = _optimum(dev)
        return {"u": u, "x": x, "status": None}
    A, B, _ = _matrices(ph)
    u, x = _optimum(dict(dev, A=A, B=B))
    r = _Rng(seed + 1)
    L = case["landmarks"]
    alpha = r.uni(0.2, 1.0, L).to(torch.float32).double()
    qc = torch.tensor([1.0, 1.0, 2.0], device=r.dev, dtype=torch.float64)
    com = (dev["x0"][:, 3:6] + 0.02).double()
    # predictions of the previous tick that reach this one: offset 1
    offs = _offsets_of(dev["N"], L)
    err = com - dev["x_ref"][:, 0, 3:6].double()
    cost = ((offs == 1).double() * alpha).sum(-1) * (err * err * qc).sum(-1)
    return {"u": u, "x": x, "status": None, "reward": torch.exp(-cost / SIGMA ** 2),
            "used": None}
