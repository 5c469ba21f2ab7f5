"""Performance cases: what programs that use the swarm stepper ask of it.

Four kinds of call, each through the Python binding as a user's program makes
it:

  step   one control step of a simulation loop: step_observe, or
         step_observe_reward in a reinforcement-learning loop; or a replay of
         a HIP graph that such calls were captured in
  diff   one training step through the differentiable rollout: forward, and
         backward to the initial state, the actions and the parameters
  vjp    the vector-Jacobian product of one control step (step_backward), as
         a program calls it that keeps its own trajectory
  reset  the end of an episode: new parameters and states for some of the
         environments, an observation of all, and a snapshot of the state

``exact`` gives the same results from plain float64 torch operations.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.utils.checkpoint

from paper_2306_09537_amd import workloads as W
from paper_2306_09537_amd.quadswarm import QuadSwarm, rollout

EPISODE = 1000  # substeps after which a simulation loop starts over
ACTION_SETS = 16
SENSOR_ROW = 18

PLAIN = 0
FREE = W.SWARM_FLAGS & ~W.QS_COLLIDE
SWARM = W.SWARM_FLAGS


def listed():
    step = dict(kind="step", sizes="same", reward=False, sensor=False, downwash=False,
                tuned=False, graph=0)
    diff = dict(kind="diff", sizes="same", ckpt=20, substeps=1, beta=100.0)
    return [
        # the smallest batch, latency alone: single quads without a room, as
        # a controller is tried out on
        dict(step, name="plain_64x1", envs=64, n=1, k=0, phys="plain", substeps=1),
        # a reinforcement-learning loop with every option on: 100 Hz control
        # over 200 Hz physics, reward, sensor noise and downwash, few neighbours
        dict(step, name="rl_1024x8_k3", envs=1024, n=8, k=3, phys="swarm", substeps=2,
             reward=True, sensor=True, downwash=True),
        # the ordinary batch of swarms of 8
        dict(step, name="swarm_4096x8", envs=4096, n=8, k=6, phys="swarm", substeps=1),
        # a swarm size that is no power of two
        dict(step, name="odd_4096x12", envs=4096, n=12, k=6, phys="swarm", substeps=2,
             reward=True),
        # the largest batches: dense swarms, and single quads
        dict(step, name="scale_32768x32", envs=32768, n=32, k=6, phys="swarm", substeps=1),
        dict(step, name="scale_1048576x1", envs=1048576, n=1, k=0, phys="free", substeps=1),
        # environments of 1 to 32 quads together, ten substeps per call, ten
        # calls captured in one graph
        dict(step, name="uneven_16384", envs=16384, n=32, sizes="powers", k=6, phys="swarm",
             substeps=10, tuned=True, graph=10),
        # trajectory optimisation through the simulator: the ordinary batch,
        # the largest, and environments of different sizes
        dict(diff, name="diff_1024x8", envs=1024, n=8, calls=200, phys="swarm"),
        dict(diff, name="diff_32768x32", envs=32768, n=32, calls=100, phys="swarm"),
        dict(diff, name="diff_uneven_2048", envs=2048, n=16, sizes="range", calls=50, substeps=2,
             ckpt=10, phys="swarm"),
        # one control step differentiated inside a program's own graph
        dict(kind="vjp", name="vjp_4096x8", envs=4096, n=8, sizes="same", substeps=2,
             phys="swarm"),
        # the end of an episode for one environment in eight
        dict(kind="reset", name="reset_16384x8", envs=16384, n=8, sizes="same", k=6,
             phys="swarm", every=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "diff", "diff", "vjp", "reset"))
    n = rng.choice((1, 2, 4, 8, 16, 32, _log_int(rng, 1, 48), _log_int(rng, 3, 48)))
    sizes = rng.choice(("same", "same", "range")) if n > 1 else "same"
    phys = "free" if n == 1 else "swarm"
    mean = n if sizes == "same" else (n + 1) / 2
    if kind == "step":
        substeps = rng.choice((1, 2, 2, 4, 10))
        quads = _log_int(rng, 64, 1048576 / substeps)
        graph = rng.choice((0, 0, 0, 4))
        return dict(kind=kind, envs=max(1, int(quads / mean)), n=n, sizes=sizes,
                    k=rng.choice((0, 1, 2, 3, 4, 6, 6, 8)) if n > 1 else 0, phys=phys,
                    substeps=substeps, reward=rng.random() < 0.4, sensor=rng.random() < 0.3,
                    downwash=n > 1 and rng.random() < 0.25, tuned=rng.random() < 0.3, graph=graph)
    if kind == "diff":
        substeps = rng.choice((1, 1, 2))
        calls = _log_int(rng, 10, 100)
        quads = _log_int(rng, 256, 262144 / substeps)
        return dict(kind=kind, envs=max(1, int(quads / mean)), n=n, sizes=sizes, calls=calls,
                    substeps=substeps, ckpt=rng.choice((5, 10, 20)),
                    beta=rng.choice((100.0, 100.0, 50.0, 0.0)) if n > 1 else 0.0, phys=phys)
    quads = _log_int(rng, 64, 262144)
    if kind == "vjp":
        return dict(kind=kind, envs=max(1, int(quads / mean)), n=n, sizes=sizes,
                    substeps=rng.choice((1, 2, 4)), phys=phys)
    return dict(kind=kind, envs=max(1, int(quads / mean)), n=n, sizes=sizes,
                k=rng.choice((0, 3, 6)) if n > 1 else 0, phys=phys, every=rng.choice((1, 2, 8)))


# ---- inputs -----------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _sizes(case):
    """Swarm size of each environment (of the case alone, not of the seed)."""
    if case["sizes"] == "same":
        return np.full(case["envs"], case["n"], dtype=np.int32)
    r = np.random.RandomState(case["envs"] % 65521)
    if case["sizes"] == "powers":
        powers = [1 << i for i in range(int(math.log2(case["n"])) + 1)]
        return r.choice(np.array(powers), size=case["envs"]).astype(np.int32)
    return r.randint(1, case["n"] + 1, size=case["envs"]).astype(np.int32)


def _flags(case):
    f = {"plain": PLAIN, "free": FREE, "swarm": SWARM}[case["phys"]]
    f |= W.QS_SENSOR_NOISE if case.get("sensor") else 0
    f |= W.QS_DOWNWASH if case.get("downwash") else 0
    return f


def _states(g, params):
    """Start states as the workloads draw them: positions U([-2,2]^2 x
    [0.5,2.5]), velocities and rates N(0, 0.5^2), attitude within 30 degrees
    of upright, motors at the hover command."""
    q, dev = params.shape[0], params.device
    f64 = dict(dtype=torch.float64, device=dev, generator=g)
    s = torch.zeros(q, 27, dtype=torch.float64, device=dev)
    s[:, 0:3] = torch.rand(q, 3, **f64) * torch.tensor([4.0, 4.0, 2.0], device=dev)
    s[:, 0:3] += torch.tensor([-2.0, -2.0, 0.5], device=dev)
    s[:, 3:6] = 0.5 * torch.randn(q, 3, **f64)
    phi, psi, c = (torch.rand(q, **f64) for _ in range(3))
    phi, psi = 2 * math.pi * phi, 2 * math.pi * psi
    c = math.cos(math.radians(30.0)) * (1 - c) + c
    sn = torch.sqrt(1 - c * c)
    x, y, o = torch.cos(phi), torch.sin(phi), torch.zeros_like(c)
    tilt = torch.stack([c + x * x * (1 - c), x * y * (1 - c), y * sn,
                        x * y * (1 - c), c + y * y * (1 - c), -x * sn,
                        -y * sn, x * sn, c], 1).view(q, 3, 3)
    cz, sz = torch.cos(psi), torch.sin(psi)
    yaw = torch.stack([cz, -sz, o, sz, cz, o, o, o, o + 1], 1).view(q, 3, 3)
    s[:, 6:15] = (tilt.unsqueeze(3) * yaw.unsqueeze(1)).sum(2).reshape(q, 9)
    s[:, 15:18] = 0.5 * torch.randn(q, 3, **f64)
    s[:, 18:22] = torch.sqrt(1.0 / params[:, 4:5].double())
    return s.float()


def _params(g, q, randomise, dev):
    nominal = torch.tensor([W.NOMINAL[k] for k in ("mass", "ixx", "iyy", "izz",
                                                   "thrust_to_weight", "motor_tau")],
                           dtype=torch.float64, device=dev)
    width = torch.tensor([0.2] * 5 + [0.3], dtype=torch.float64, device=dev)
    u = 2 * torch.rand(q, 6, dtype=torch.float64, device=dev, generator=g) - 1
    return (nominal * (1 + (width * u if randomise else 0 * u))).float()


def _key(seed):
    return (0x9E3779B97F4A7C15 * (seed + 1)) & 0xFFFFFFFFFFFFFFFF


def _inputs(case, seed):
    """Everything the call gets, as tensors."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    q = int(_sizes(case).sum())

    def uniform(*shape):
        return torch.rand(*shape, device=dev, generator=g)

    d = dict(params=_params(g, q, case["phys"] != "plain", dev))
    d["state"] = _states(g, d["params"])
    if case["kind"] in ("step", "reset"):
        d["goals"] = uniform(q, 3) * torch.tensor([6.0, 6.0, 2.0], device=dev)
        d["goals"] += torch.tensor([-3.0, -3.0, 1.0], device=dev)
    if case["kind"] == "step":
        # fresh actions for every call; a second half that mirrors the first
        # keeps a long loop from spinning the quads up
        n_sets = case["graph"] or ACTION_SETS
        acts = []
        for _ in range(0, n_sets, 2):
            a = uniform(q, 4)
            acts += [a, 1.0 - a]
        d["actions"] = acts[:n_sets]
    elif case["kind"] == "diff":
        d["actions"] = uniform(case["calls"], q, 4)
        d["g_state"] = torch.randn(q, 27, device=dev, generator=g)
        d["g_pen"] = uniform(q)
    elif case["kind"] == "vjp":
        d["actions"] = uniform(q, 4)
        d["g_state"] = torch.randn(q, 27, device=dev, generator=g)
    else:
        d["new_params"] = _params(g, q, True, dev)
        d["new_state"] = _states(g, d["new_params"])
        first = seed % case["every"]
        mask = torch.zeros(case["envs"], dtype=torch.uint8, device=dev)
        mask[first::case["every"]] = 1
        d["mask"] = mask
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    offsets = np.concatenate([[0], np.cumsum(_sizes(case))]).astype(np.int32)
    sim = QuadSwarm(offsets, W.BASE_CONSTS, d["params"].cpu().numpy(), d["state"].cpu().numpy(),
                    case.get("k", 0), _flags(case), _key(seed))
    q = sim.n_quads
    s = dict(d, case=case, sim=sim)
    dev = d["state"].device
    if case["kind"] in ("step", "reset"):
        s["obs"] = torch.empty(q, sim.obs_dim, device=dev)
    if case["kind"] == "step":
        s["calls"] = 0
        if case["reward"]:
            sim.set_reward_weights(W.REWARD_WEIGHTS)
            s["r"] = torch.empty(q, device=dev)
        if case["tuned"]:
            sim.autotune(d["actions"][0], case["substeps"], d["goals"], s["obs"])
        if case["graph"]:
            sim.set_graph_mode(True)
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):  # warm up outside the capture
                _control_step(s, 0)
            torch.cuda.current_stream().wait_stream(side)
            sim.set_state(d["state"], 0)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                for k in range(case["graph"]):
                    _control_step(s, k)
    elif case["kind"] == "vjp":
        s["out"] = (torch.empty_like(d["state"]), torch.empty_like(d["actions"]),
                    torch.zeros(q, 6, device=dev))
    elif case["kind"] == "reset":
        s["snapshot"] = torch.empty(q, 27, device=dev)
    return s


def _control_step(s, k):
    case, sim = s["case"], s["sim"]
    if case["reward"]:
        sim.step_observe_reward(s["actions"][k], case["substeps"], s["goals"], s["obs"], s["r"])
    else:
        sim.step_observe(s["actions"][k], case["substeps"], s["goals"], s["obs"])


def run(s):
    case, sim = s["case"], s["sim"]
    if case["kind"] == "step":
        per_pass = case["substeps"] * (case["graph"] or 1)
        k = s["calls"]
        if k and k % max(1, EPISODE // per_pass) == 0:  # a new episode
            sim.set_state(s["state"], 0)
        s["calls"] = k + 1
        if case["graph"]:
            s["graph"].replay()
        else:
            _control_step(s, k % ACTION_SETS)
        return (s["obs"], s["r"]) if case["reward"] else s["obs"]
    if case["kind"] == "diff":
        leaves = [s[k].detach().requires_grad_(True) for k in ("state", "actions", "params")]
        end, pen = rollout(sim, *leaves, case["substeps"], case["ckpt"], case["beta"])
        if case["beta"] > 0:
            grads = torch.autograd.grad((end, pen), leaves, (s["g_state"], s["g_pen"]))
        else:
            grads = torch.autograd.grad(end, leaves, s["g_state"])
        return (end.detach(), pen.detach()) + tuple(grads)
    if case["kind"] == "vjp":
        sim.step_backward(s["state"], s["actions"], case["substeps"], 0, s["g_state"], *s["out"])
        return s["out"]
    sim.set_params(s["new_params"], s["mask"])
    sim.set_state(s["new_state"], 0, s["mask"])
    obs = sim.observe(s["goals"], s["obs"])
    state, _ = sim.get_state(s["snapshot"])
    return obs, state


def work(case):
    """Operations as the plain definition counts them (add, multiply, divide,
    square root and transcendental one each): a substep of a quad 247 and 4
    per swarm-mate, an observation 11, 8 per swarm-mate and 6 per slot, a
    differentiated substep 877 and 25.5 per swarm-mate."""
    sz = _sizes(case).astype(np.float64)
    q, mates = sz.sum(), (sz * (sz - 1)).sum()
    k = case.get("k", 0)
    row = 4.0 * (SENSOR_ROW + 6 * k)
    observe = 11 * q + 8 * (mates if k else 0) + 6 * k * q
    if case["kind"] == "step":
        calls = case["graph"] or 1
        # a graph keeps the state between its calls on the device as well
        per_call = q * (2 * 108 + 24 + 16 + 12 + row + (4 if case["reward"] else 0))
        flops = case["substeps"] * (247 * q + 4 * mates) + observe
        return {"bytes": calls * per_call, "flops": calls * flops}
    if case["kind"] == "diff":
        steps = case["calls"] * case["substeps"]
        return {"bytes": q * (4 * 108 + 2 * 24 + 8 + 32.0 * case["calls"]),
                "flops": steps * (877 * q + 25.5 * mates)}
    if case["kind"] == "vjp":
        return {"bytes": q * (3 * 108 + 2 * 16 + 3 * 24.0),
                "flops": case["substeps"] * (877 * q + 13.0 * mates)}
    part = q / case["every"]
    return {"bytes": part * (2 * 108 + 24 + 32) + q * (2 * 108 + 60 + 12 + row), "flops": observe}


# ---- the same in float64, from plain torch operations -----------------------
def _f32(v):
    return float(np.float32(v))


C = {k: (tuple(_f32(x) for x in v) if isinstance(v, tuple) else _f32(v))
     for k, v in W.BASE_CONSTS.items()}
ARM = C["arm_length"] / math.sqrt(2.0)
NOISE = C["motor_noise_std"] * math.sqrt(1.0 - C["motor_noise_decay"] ** 2)


def _mulhilo(a, m):
    """High and low words of the 64-bit product of 32-bit a (int64) and m."""
    lo = a * (m & 0xFFFF)
    hi = a * (m >> 16) + (lo >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def _words(case, seed, q, t, stream, number):
    """Philox4x32-10 (Salmon et al., SC'11) at (quad, t, stream << 8 | draw)."""
    key = _key(seed)
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    c0 = torch.arange(q, device=_device())
    c1 = torch.full_like(c0, t & 0xFFFFFFFF)
    c2 = torch.full_like(c0, t >> 32)
    c3 = torch.full_like(c0, stream << 8 | number)
    for _ in range(10):
        h0, l0 = _mulhilo(c0, 0xD2511F53)
        h1, l1 = _mulhilo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return torch.stack([c0, c1, c2, c3], 1)


def _uniforms(*a):
    return (2 * (_words(*a) >> 9) + 1).double() / 2.0 ** 24


def _normals(*a):
    u = _uniforms(*a)
    r, w = torch.sqrt(-2 * torch.log(u[:, 0::2])), 2 * math.pi * u[:, 1::2]
    return torch.stack([r * torch.cos(w), r * torch.sin(w)], 2).view(-1, 4)


def _norm(v):
    """Lengths, with derivative zero at zero."""
    n2 = (v * v).sum(-1)
    some = n2 > 0
    return torch.where(some, torch.sqrt(torch.where(some, n2, torch.ones_like(n2))), 0 * n2)


def _unit(v):
    n = _norm(v)
    return v / torch.where(n > 0, n, torch.ones_like(n)).unsqueeze(-1)


class _Swarms:
    """Quads of the environments side by side: [E][n_max] with a mask."""

    def __init__(self, case):
        sz = torch.from_numpy(_sizes(case).astype(np.int64)).to(_device())
        off = torch.cumsum(sz, 0) - sz
        lane = torch.arange(int(sz.max()), device=sz.device)
        self.there = lane < sz[:, None]
        self.index = torch.where(self.there, off[:, None] + lane, off[:, None])
        self.at = self.there.nonzero(as_tuple=True)
        self.mates = (self.there[:, :, None] & self.there[:, None, :]
                      & (lane[:, None] != lane[None, :]))

    def wide(self, v):
        return v[self.index]

    def flat(self, v):
        return v[self.at]


def _substep(case, seed, sw, P, s, uhat, t, beta=0.0):
    """One substep of every quad.  s: x, v, R [Q][3][3], w, u, e, fl; returns
    the new s, the penalty's increment and the interaction events."""
    flags, dt, g = _flags(case), C["dt"], C["gravity"]
    x, v, R, w, u, e, fl = s
    m, J = P[:, 0], P[:, 1:4]
    f_max = 0.25 * m * g * P[:, 4]
    lag = 1.0 - torch.exp(-dt / P[:, 5])
    u = u + lag[:, None] * (uhat - u)
    if flags & W.QS_MOTOR_NOISE:
        z = _normals(case, seed, x.shape[0], t, 0, 0)
        e = C["motor_noise_decay"] * e + NOISE * f_max[:, None] * z
    f = f_max[:, None] * u * u + e
    f0, f1, f2, f3 = f.unbind(1)
    T = f.sum(1)
    tau = torch.stack([ARM * (f2 + f3 - f0 - f1), ARM * (f1 + f2 - f0 - f3),
                       C["k_tau"] * (f0 + f2 - f1 - f3)], 1)
    F = T[:, None] * R[:, :, 2]
    # free flight
    grav = torch.tensor([0.0, 0.0, -g], dtype=x.dtype, device=x.device)
    v1 = v + dt * ((F - C["drag_coef"] * v) / m[:, None] + grav)
    x1 = x + dt * v1
    w1 = w + dt * (tau - torch.linalg.cross(w, J * w)) / J
    r0, r1, r2 = R.unbind(2)
    c0 = _unit(r0 + dt * (r1 * w1[:, 2:3] - r2 * w1[:, 1:2]))
    c1 = r1 + dt * (r2 * w1[:, 0:1] - r0 * w1[:, 2:3])
    c1 = _unit(c1 - (c0 * c1).sum(1, keepdim=True) * c0)
    R1 = torch.stack([c0, c1, torch.linalg.cross(c0, c1)], 2)
    rest = torch.zeros_like(fl, dtype=torch.bool)
    ev = {k: rest for k in ("hit", "wall", "ceiling", "quad")}
    if flags & W.QS_FLOOR:
        # resting on the floor: friction in the plane, nothing else moves
        rest = (fl != 0) & (F[:, 2] <= m * g)
        n_f = C["floor_mu"] * (m * g - F[:, 2])
        still = (v[:, 0] == 0) & (v[:, 1] == 0)
        Fh, vh = F[:, :2], v[:, :2]
        held = _unit(Fh) * torch.clamp(_norm(Fh) - n_f, min=0.0)[:, None]
        fr = torch.where(still[:, None], held, Fh - n_f[:, None] * _unit(vh))
        vr = vh + dt * (fr - C["drag_coef"] * vh) / m[:, None]
        vr = torch.where(((vr * vh).sum(1) < 0)[:, None], 0 * vr, vr)
        vr = torch.cat([vr, 0 * vr[:, :1]], 1)
        x1 = torch.where(rest[:, None], x + dt * vr, x1)
        v1 = torch.where(rest[:, None], vr, v1)
        w1 = torch.where(rest[:, None], 0 * w1, w1)
        R1 = torch.where(rest[:, None, None], R, R1)
    fl = torch.where(rest, fl, torch.zeros_like(fl))
    x, v, w, R = x1, v1, w1, R1
    if flags & W.QS_ROOM:
        lo = torch.tensor([C["room_min"][0], C["room_min"][1], -math.inf], dtype=x.dtype,
                          device=x.device)
        hi = torch.tensor(C["room_max"], dtype=x.dtype, device=x.device)
        flip = ((x < lo) & (v < 0)) | ((x > hi) & (v > 0))
        x = torch.where(x < lo, lo, torch.where(x > hi, hi, x))
        v = torch.where(flip, -C["wall_restitution"] * v, v)
        v = torch.where(flip.any(1)[:, None], C["col_decay"] * v, v)
        ev["wall"], ev["ceiling"] = flip[:, :2].any(1), flip[:, 2]
    if flags & W.QS_FLOOR:
        hit = x[:, 2] < C["room_min"][2]
        ev["hit"] = hit
        x = torch.where(hit[:, None] & torch.tensor([False, False, True], device=x.device),
                        torch.full_like(x, C["room_min"][2]), x)
        v = torch.where(hit[:, None], 0 * v, v)
        w = torch.where(hit[:, None], 0 * w, w)
        fl = torch.where(hit, torch.ones_like(fl), fl)
        a = _unit(R[:, :2, 0])
        o = 0 * a[:, 0]
        level = torch.stack([a[:, 0], -a[:, 1], o, a[:, 1], a[:, 0], o, o, o, o + 1], 1)
        R = torch.where(hit[:, None, None], level.view(-1, 3, 3), R)
    pen = 0 * x[:, 0]
    if flags & W.QS_COLLIDE and case["n"] > 1:
        xe, ve = sw.wide(x), sw.wide(v)
        d = xe[:, :, None] - xe[:, None]  # from j to i
        d2 = (d * d).sum(3)
        safe = torch.where(sw.mates, d2, torch.ones_like(d2))
        dist = torch.sqrt(safe)
        touch = sw.mates & (d2 < C["col_dist"] ** 2)
        nrm = d / dist.unsqueeze(3)
        sp = ((ve[:, None] - ve[:, :, None]) * nrm).sum(3)
        act = touch & (sp > 0)
        dv = (torch.where(act, sp, 0 * sp).unsqueeze(3) * nrm).sum(2)
        hit = sw.flat(act.any(2))
        v = torch.where(hit[:, None], C["col_decay"] * (v + sw.flat(dv)), v)
        ev["quad"] = hit
        if beta > 0:
            p = 0.5 * torch.nn.functional.softplus(beta * (C["col_dist"] - dist), threshold=60.0)
            pen = sw.flat((torch.where(sw.mates, p, 0 * p) / beta).sum(2))
        if flags & W.QS_DOWNWASH:
            up = -d[..., 2]  # how far j is above i
            over = (sw.mates & (d[..., 0] ** 2 + d[..., 1] ** 2 < C["dw_radius"] ** 2)
                    & (up > 0) & (up < C["dw_height"]) & (sw.wide(fl) == 0)[:, :, None])
            acc = -C["dw_k1"] * (C["dw_k2"] * up + C["dw_b1"])
            kick = dt * sw.flat(torch.where(over, acc, 0 * acc).sum(2))
            v = torch.cat([v[:, :2], v[:, 2:] + kick[:, None]], 1)
    return (x, v, R, w, u, e, fl), pen, ev


def _split(state):
    q = state.shape[0]
    return (state[:, 0:3], state[:, 3:6], state[:, 6:15].reshape(q, 3, 3), state[:, 15:18],
            state[:, 18:22], state[:, 22:26], state[:, 26].detach())


def _join(s):
    x, v, R, w, u, e, fl = s
    return torch.cat([x, v, R.reshape(-1, 9), w, u, e, fl[:, None]], 1)


def _command(a):
    return torch.sqrt(0.5 * (torch.clamp(a, -1.0, 1.0) + 1.0))


def _observe(case, seed, sw, s, goals, t):
    x, v, R, w = s[:4]
    q, k, n = x.shape[0], case["k"], sw.there.shape[1]
    off = x - goals
    near = torch.zeros(q, k, 6, dtype=x.dtype, device=x.device)
    real = torch.zeros(q, k, dtype=torch.bool, device=x.device)
    if k and n > 1:
        xe, ve = sw.wide(x), sw.wide(v)
        d2 = ((xe[:, None] - xe[:, :, None]) ** 2).sum(3)
        d2 = torch.where(sw.mates, d2, torch.full_like(d2, math.inf))
        top = min(k, n)
        val, j = torch.sort(d2, dim=2, stable=True)
        val, j = val[:, :, :top], j[:, :, :top]
        e = torch.arange(j.shape[0], device=x.device)[:, None, None]
        rel = torch.cat([xe[e, j] - xe[:, :, None], ve[e, j] - ve[:, :, None]], 3)
        ok = val < math.inf
        near[:, :top] = sw.flat(torch.where(ok.unsqueeze(3), rel, 0 * rel))
        real[:, :top] = sw.flat(ok)
    own = [off, v, R.reshape(q, 9), w]
    if _flags(case) & W.QS_SENSOR_NOISE:
        def u(number):
            return 2 * _uniforms(case, seed, q, t, 4, number)[:, :3] - 1

        own = [off + C["sn_x"] * u(0), v + C["sn_v"] * u(1), R.reshape(q, 9),
               w + C["sn_w"] * _normals(case, seed, q, t, 4, 2)[:, :3]]
    return torch.cat(own + [near.reshape(q, 6 * k)], 1), off, near, real


def _reward(P, s, thrust0, off, near, real, ev):
    x, v, R, w, u, e, fl = s
    f_max = 0.25 * P[:, 0] * C["gravity"] * P[:, 4]
    f = f_max[:, None] * u * u + e
    a = [_f32(z) for z in W.REWARD_WEIGHTS]
    trace = R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2]
    r = (a[0] * _norm(off) + a[1] * _norm(v) + a[2] * R[:, 2, 2] + a[3] * _norm(w)
         + a[4] * _norm(f) + a[5] * _norm(f - thrust0) + a[6] * (trace - 1) / 2
         + a[7] * R[:, 0, 0] + a[8] * ev["hit"] + a[9] * (fl != 0) + a[10] * ev["wall"]
         + a[11] * ev["ceiling"] + a[12] * ev["quad"])
    close = torch.clamp(1 - _norm(near[..., :3]) / a[14], min=0.0)
    return r + a[13] * (close * real).sum(1)


def _pairs(case):
    sz = _sizes(case)
    return float(sz.shape[0]) * float(sz.max()) ** 2


def exact(case, seed):
    d = _inputs(case, seed)
    sw = _Swarms(case)
    P, state = d["params"].double(), d["state"].double()
    if case["kind"] == "step":
        s = _split(state)
        t, calls = 0, case["graph"] or 1
        for k in range(calls):
            uhat = _command(d["actions"][k].double())
            f_max = 0.25 * P[:, 0] * C["gravity"] * P[:, 4]
            thrust0 = f_max[:, None] * s[4] * s[4] + s[5]
            ev = None
            for _ in range(case["substeps"]):
                s, _, now = _substep(case, seed, sw, P, s, uhat, t)
                ev = now if ev is None else {n: ev[n] | now[n] for n in ev}
                t += 1
        obs, off, near, real = _observe(case, seed, sw, s, d["goals"].double(), t)
        return (obs, _reward(P, s, thrust0, off, near, real, ev)) if case["reward"] else obs
    if case["kind"] == "reset":
        pick = torch.repeat_interleave(d["mask"].bool(), torch.from_numpy(
            _sizes(case).astype(np.int64)).to(state.device))
        state = torch.where(pick[:, None], d["new_state"].double(), state)
        obs = _observe(case, seed, sw, _split(state), d["goals"].double(), 0)[0]
        return obs, state
    calls = case.get("calls", 1)
    # minutes in float64 where the swarms are both large and many
    if _pairs(case) * calls * case["substeps"] > 4e8:
        return None
    acts = d["actions"].double().view(calls, -1, 4)
    leaves = [z.requires_grad_(True) for z in (state, acts, P)]
    beta = case.get("beta", 0.0)

    def control_step(k, pen, *s):
        uhat = _command(leaves[1][k])
        for i in range(case["substeps"]):
            s, p, _ = _substep(case, seed, sw, leaves[2], s, uhat, k * case["substeps"] + i, beta)
            pen = pen + p
        return (pen,) + tuple(s)

    s = _split(leaves[0])
    pen = 0 * leaves[0][:, 0]
    for k in range(calls):
        if calls > 1:
            pen, *s = torch.utils.checkpoint.checkpoint(control_step, k, pen, *s,
                                                        use_reentrant=False)
        else:
            pen, *s = control_step(k, pen, *s)
    end = _join(s)
    loss = (end * d["g_state"].double()).sum()
    if beta > 0:
        loss = loss + (pen * d["g_pen"].double()).sum()
    gs, ga, gp = torch.autograd.grad(loss, leaves, allow_unused=True)
    if case["kind"] == "vjp":
        return gs, ga.view(-1, 4), gp
    return end.detach(), pen.detach(), gs, ga, gp
