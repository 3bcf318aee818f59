"""Workloads of the MPPI library, timed through its public entry points.

A case is a dict of plain values; its "path" says which call it stands for:

  step     Controller.step: one MPC step, the warm-start knots and the state given
  tick     Controller.run_tick: prediction over the delay, warm-start shift, step
  fleet    step_batch, or a captured Graph of it: one round of many robots
  predict  Controller.predict and shift_knots: what a tick does before its step
  update   update_noalloc: weights and knot update of given costs and samples

The robots, sizes, noise and costs are those of paper_2511_19204_amd.synth; the
states are small perturbations of a robot's stance and the warm starts jittered
stance knots, as a controller meets them between ticks.  exact() is the same
method in 64 bits with numpy.  Rollouts with ground contact over a whole horizon
have no such value: rounding decides contact events, and a float rollout and a
double one part ways within some tens of steps, so exact() covers the arms'
steps, the prediction and the update.
"""
import math

import numpy as np
import torch

from paper_2511_19204_amd import mppi, synth

MODELS = {"arm": synth.chain_model, "ytree": synth.ytree_model, "quadruped": synth.quadruped_model,
          "hexapod": synth.hexapod_model, "humanoid": synth.humanoid_model}
DOF = {"arm": 3, "ytree": 6, "quadruped": 18, "hexapod": 24, "humanoid": 27}
NU = {"arm": 3, "ytree": 6, "quadruped": 12, "hexapod": 18, "humanoid": 21}
# arithmetic of one control step of one rollout (non-trivial operations of the
# plain method, profiles/flops_per_rollout_step.txt; the hexapod's and the
# branching arm's by their degrees of freedom)
STEP_FLOPS = {"arm": 664.0, "ytree": 1328.0, "quadruped": 8404.0, "hexapod": 11200.0, "humanoid": 14946.0}
DT = {"arm": 0.01, "ytree": 0.01, "quadruped": 0.005, "hexapod": 0.005, "humanoid": 0.004}


def listed():
    return [
        # the smallest controller: the planar arm, ten iterations of two wavefronts
        {"name": "arm_step", "path": "step", "model": "arm", "samples": 32, "horizon": 50, "knots": 4, "iters": 10,
         "noise": "linear"},
        # a quadruped at the paper's real-time sample count, one full control tick
        {"name": "quadruped_tick", "path": "tick", "model": "quadruped", "samples": 64, "horizon": 100, "knots": 8,
         "iters": 3, "noise": "exp", "delay": 1},
        # the same robot planning further ahead, from few to many samples
        {"name": "quadruped_k256", "path": "step", "model": "quadruped", "samples": 256, "horizon": 200, "knots": 8,
         "iters": 1, "noise": "linear"},
        {"name": "quadruped_k4096", "path": "step", "model": "quadruped", "samples": 4096, "horizon": 200, "knots": 8,
         "iters": 1, "noise": "linear"},
        {"name": "quadruped_k16384", "path": "step", "model": "quadruped", "samples": 16384, "horizon": 200, "knots": 8,
         "iters": 1, "noise": "linear"},
        # spline ablation: natural cubic knots (samples stored, not drawn again), odd sizes
        {"name": "quadruped_spline", "path": "step", "model": "quadruped", "samples": 333, "horizon": 77, "knots": 7,
         "iters": 3, "noise": "exp", "spline": 1},
        # a tree of another shape, ragged last wavefront
        {"name": "hexapod_step", "path": "step", "model": "hexapod", "samples": 97, "horizon": 83, "knots": 8,
         "iters": 3, "noise": "exp"},
        # a humanoid's control tick, and its task preset at many samples
        {"name": "humanoid_tick", "path": "tick", "model": "humanoid", "samples": 256, "horizon": 150, "knots": 10,
         "iters": 3, "noise": "exp", "delay": 2},
        {"name": "humanoid_k1024", "path": "step", "model": "humanoid", "samples": 1024, "horizon": 150, "knots": 10,
         "iters": 3, "noise": "task"},
        # mixed robots stepped together: a small fleet replayed as a graph, a large one as batches
        {"name": "fleet16_graph", "path": "fleet", "robots": 16, "graph": True},
        {"name": "fleet64", "path": "fleet", "robots": 64, "graph": False},
        # the weighted update on given samples, without allocation, many slices
        {"name": "update_20000", "path": "update", "samples": 20000, "knots": 8, "nu": 12, "raw": False},
    ]


def draw(rng):
    """One more case of the listed ranges (sizes over their logarithm, odd ones among them)."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(("step", "step", "step", "tick", "tick", "fleet", "update", "predict"))
    if path == "fleet":
        return {"path": path, "robots": size(2, 60), "graph": rng.random() < 0.5}
    if path == "update":
        return {"path": path, "samples": size(50, 60000), "knots": rng.randint(4, 12), "nu": rng.choice((3, 6, 12, 18, 21)),
                "raw": rng.random() < 0.3}
    model = rng.choice(("arm", "ytree", "quadruped", "quadruped", "hexapod", "humanoid"))
    case = {"path": path, "model": model, "samples": 0, "horizon": rng.randint(40, 200), "knots": rng.randint(4, 12),
            "iters": rng.randint(1, 4), "noise": rng.choice(("linear", "exp", "task"))}
    # no more arithmetic than the 64-robot round
    most = 6e10 / (STEP_FLOPS[model] * case["horizon"] * case["iters"])
    case["samples"] = size(20, min(16384, most))
    if path != "step":
        case["delay"] = rng.randint(1, 6)
    if rng.random() < 0.25:
        case["spline"] = rng.choice((1, 2))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _problem(case, seed):
    """(model, params, noise seed, state, warm-start knots) of a single-robot case."""
    name = case["model"]
    m = MODELS[name](seed % 10)
    noise = {"linear": ("linear", 0.1, 0.3) if not m["floating_base"] else ("linear", 0.05, 0.4),
             "exp": ("exp", 0.4, 1.0, 1.0), "task": ("exp", 0.1, 1.0, 1.0)}[case["noise"]]
    cost = "ee" if not m["floating_base"] else ("bipedal" if name == "humanoid" else "walking")
    p = synth.params(m, case["samples"], case["horizon"], DT[name], case["knots"], case["iters"], noise, cost,
                     lam=synth.TASK_SAMPLING["lambda"] if case["noise"] == "task" else 1.0)
    p["spline_mode"] = case.get("spline", 0)
    x = synth.perturbed_states(m, 1, seed, 0.005)[0]
    rng = np.random.default_rng(seed + 1)
    kn = synth.nominal_knots(m, p["n_knots"])
    half = kn.size // 2
    kn[:half] += rng.normal(0, 0.02, half)
    kn[half:] += rng.normal(0, 0.1, half) if p["spline_mode"] == 0 else 0.0
    return m, p, 1000 + seed, x, synth.f32(kn)


def _gpu(a, dtype=torch.float32):
    return torch.tensor(np.asarray(a), dtype=dtype, device="cuda")


def _info(t):
    """A step's info words as its float (lowest cost) and its whole values."""
    return {"S_best": t[:1].view(torch.float32), "counts": t[1:]}


def _update_inputs(case, seed):
    """Costs and samples as rollouts leave them: a spread of costs, a few of them infinite."""
    n, e = case["samples"], 2 * case["knots"] * case["nu"]
    rng = np.random.default_rng(seed)
    nom = synth.f32(rng.normal(0, 0.5, e))
    costs = synth.f32(1e3 * np.exp(rng.normal(0, 0.5, n)))
    costs[rng.random(n) < 0.01] = np.inf
    costs[0] = np.float32(900.0)
    samples = (nom[None, :] + 0.3 * rng.standard_normal((n, e), dtype=np.float32)).astype(np.float32)
    return costs, samples, nom


def prepare(case, seed):
    path = case["path"]
    if path == "update":
        costs, samples, nom = _update_inputs(case, seed)
        return {"case": case, "costs": _gpu(costs), "samples": _gpu(samples), "nom": _gpu(nom),
                "out": torch.empty(nom.size, device="cuda"), "weights": torch.empty(costs.size, device="cuda")}
    if path == "fleet":
        # another seed is another fleet state; the robots' sizes stay the workload's
        s = {"case": case, "ctrls": [], "x": [], "kin": [], "kout": [], "best": [], "info": []}
        for r, (m, p, nseed) in enumerate(synth.serving_mix(case["robots"], 0)):
            x = synth.perturbed_states(m, 1, 1000 * seed + r, 0.005)[0]
            kn = synth.nominal_knots(m, p["n_knots"])
            s["ctrls"].append(mppi.Controller(mppi.Model(m), p, nseed + 100 * seed))
            s["x"].append(_gpu(x))
            s["kin"].append(_gpu(kn))
            s["kout"].append(torch.empty(kn.size, device="cuda"))
            s["best"].append(torch.empty(kn.size, device="cuda"))
            s["info"].append(torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda"))
        if case["graph"]:
            s["graph"] = mppi.Graph(s["ctrls"], s["x"], s["kin"], s["kout"], s["best"], s["info"])
        return s
    m, p, nseed, x, kn = _problem(case, seed)
    s = {"case": case, "ctrl": mppi.Controller(mppi.Model(m), p, nseed), "x": _gpu(x), "kin": _gpu(kn),
         "kout": torch.empty(kn.size, device="cuda"), "best": _gpu(kn),
         "info": torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda"), "xp": torch.empty(x.size, device="cuda")}
    if path == "step":
        s["costs"] = torch.empty((p["n_iters"], p["n_samples"]), device="cuda")
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "step":
        s["ctrl"].step(s["x"], s["kin"], s["kout"], s["best"], s["info"], s["costs"])
        return {"knots": s["kout"], "best": s["best"], "info": _info(s["info"]), "costs": s["costs"]}
    if path == "tick":
        s["ctrl"].run_tick(s["x"], case["delay"], s["best"], s["kout"], s["info"], s["xp"])
        return {"knots": s["kout"], "best": s["best"], "info": _info(s["info"]), "state": s["xp"]}
    if path == "predict":
        s["ctrl"].predict(s["x"], s["kin"], case["delay"], s["xp"])
        s["ctrl"].shift_knots(s["kin"], case["delay"], s["kout"])
        return {"state": s["xp"], "knots": s["kout"]}
    if path == "update":
        mppi.update_noalloc(case["samples"], 2 * case["knots"] * case["nu"], 1.0 if not case["raw"] else 300.0,
                            1 if case["raw"] else 0, s["costs"], s["samples"], s["nom"], s["out"], s["weights"])
        return {"knots": s["out"], "weights": s["weights"]}
    if case["graph"]:
        s["graph"].launch()
    else:
        mppi.step_batch(s["ctrls"], s["x"], s["kin"], s["kout"], s["best"], s["info"])
    return {"knots": torch.cat(s["kout"]), "best": torch.cat(s["best"]),
            "info": [_info(i) for i in s["info"]][:15]}


def _step_work(name, samples, horizon, iters, knots):
    """Bytes (state, knots in and out, costs) and operations of a step."""
    e = 2 * knots * NU[name]
    return 4.0 * (2 * DOF[name] + 1 + 3 * e + iters * samples), STEP_FLOPS[name] * samples * horizon * iters


def work(case):
    path = case["path"]
    if path == "update":
        n, e = case["samples"], 2 * case["knots"] * case["nu"]
        return {"bytes": 4.0 * (n * e + 2 * n + 2 * e), "flops": 2.0 * n * e}
    if path == "fleet":
        b = f = 0.0
        for m, p, _ in synth.serving_mix(case["robots"], 0):
            name = {3: "arm", 12: "quadruped", 21: "humanoid"}[m["n_u"]]
            db, df = _step_work(name, p["n_samples"], p["horizon"], p["n_iters"], p["n_knots"])
            b, f = b + db, f + df
        return {"bytes": b, "flops": f}
    if path == "predict":
        return {"bytes": 4.0 * (4 * DOF[case["model"]] + 4 * case["knots"] * NU[case["model"]]),
                "flops": STEP_FLOPS[case["model"]] * case["delay"]}
    b, f = _step_work(case["model"], case["samples"], case["horizon"], case["iters"], case["knots"])
    return {"bytes": b, "flops": f + STEP_FLOPS[case["model"]] * case.get("delay", 0)}


# ---------------------------------------------------------------------------
# the method in 64 bits
# ---------------------------------------------------------------------------
def _skew(a):
    z = np.zeros(a.shape[:-1])
    return np.stack([np.stack([z, -a[..., 2], a[..., 1]], -1), np.stack([a[..., 2], z, -a[..., 0]], -1),
                     np.stack([-a[..., 1], a[..., 0], z], -1)], -2)


def _quat_R(q):
    w, x, y, z = np.moveaxis(q, -1, 0)
    return np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], -1),
                     np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], -1),
                     np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1)], -2)


def _mv(a, x):
    return (a @ x[..., None])[..., 0]


def _bodies(m, q):
    """World rotations and origins of every body at the configurations q [n, nq]."""
    n, off = q.shape[0], 7 if m["floating_base"] else 0
    R, P, j = [], [], 0
    for b, par in enumerate(m["parent"]):
        if m["floating_base"] and b == 0:
            R.append(_quat_R(q[:, 3:7]))
            P.append(q[:, :3])
            continue
        k = _skew(m["axis"][b])
        c, s = np.cos(q[:, off + j])[:, None, None], np.sin(q[:, off + j])[:, None, None]
        Rj = m["R_tree"][b] @ (np.eye(3) + s * k + (1 - c) * (k @ k))
        Rp = R[par] if par >= 0 else np.broadcast_to(np.eye(3), (n, 3, 3))
        R.append(Rp @ Rj)
        P.append((P[par] if par >= 0 else 0.0) + Rp @ m["p_tree"][b])
        j += 1
    return R, P


def _control_step(m, q, v, qref, vref, dt):
    """One linearly implicit control step of n states; also the clipped torques."""
    n, nv, fb = q.shape[0], m["n_v"], m["floating_base"]
    qj, vj = q[:, 7 if fb else 0:], v[:, 6 if fb else 0:]
    t = m["kp"] * (qref - qj) + m["kd"] * (vref - vj)
    tau = np.clip(t, -m["tau_max"], m["tau_max"])
    gain = np.where(np.abs(t) < m["tau_max"], dt * (m["kd"] + dt * m["kp"]), 0.0)
    R, P = _bodies(m, q)
    J, V, A = [], [], []  # body Jacobians, twists and velocity-product accelerations about the world origin
    M, C = np.zeros((n, nv, nv)), np.zeros((n, nv))
    g = np.array([0, 0, 0, 0, 0, -m["gravity"]])
    j = 0
    for b, par in enumerate(m["parent"]):
        Jb = np.zeros((n, 6, nv)) if par < 0 else J[par].copy()
        Ab = np.zeros((n, 6)) if par < 0 else A[par]
        if fb and b == 0:
            Jb[:, :3, :3] = R[0]
            Jb[:, 3:, :3] = _skew(P[0]) @ R[0]
            Jb[:, 3:, 3:6] = R[0]
            Vb = _mv(Jb, v)
        else:
            col = (6 if fb else 0) + j
            ax = R[b] @ m["axis"][b]
            Jb[:, :3, col], Jb[:, 3:, col] = ax, np.cross(P[b], ax)
            Vb = _mv(Jb, v)
            s = Jb[:, :, col] * v[:, col:col + 1]
            Ab = Ab + np.concatenate([np.cross(Vb[:, :3], s[:, :3]),
                                      np.cross(Vb[:, :3], s[:, 3:]) + np.cross(Vb[:, 3:], s[:, :3])], 1)
            j += 1
        xx, yy, zz, xy, xz, yz = m["inertia"][b]
        Ic = R[b] @ np.array([[xx, xy, xz], [xy, yy, yz], [xz, yz, zz]]) @ np.swapaxes(R[b], 1, 2)
        cx = _skew(P[b] + R[b] @ m["com"][b])
        mass = m["mass"][b]
        I6 = np.zeros((n, 6, 6))
        I6[:, :3, :3] = Ic + mass * cx @ np.swapaxes(cx, 1, 2)
        I6[:, :3, 3:], I6[:, 3:, :3] = mass * cx, mass * np.swapaxes(cx, 1, 2)
        I6[:, 3:, 3:] = mass * np.eye(3)
        h = _mv(I6, Vb)
        f = _mv(I6, Ab - g) + np.concatenate([np.cross(Vb[:, :3], h[:, :3]) + np.cross(Vb[:, 3:], h[:, 3:]),
                                              np.cross(Vb[:, :3], h[:, 3:])], 1)
        Jt = np.swapaxes(Jb, 1, 2)
        M += Jt @ I6 @ Jb
        C += _mv(Jt, f)
        J.append(Jb)
        V.append(Vb)
        A.append(Ab)
    rhs = -C
    rhs[:, nv - m["n_u"]:] += tau
    M[:, range(nv - m["n_u"], nv), range(nv - m["n_u"], nv)] += m["armature"] + gain
    for body, pos in zip(m["contact_body"], m["contact_pos"]):
        x = P[body] + R[body] @ pos
        Jc = J[body][:, 3:] - _skew(x) @ J[body][:, :3]
        vc = _mv(Jc, v)
        fn = np.where(x[:, 2] < 0, np.maximum(0.0, -m["k_contact"] * x[:, 2] - m["d_contact"] * vc[:, 2]), 0.0)
        nrm = np.sqrt(vc[:, 0] ** 2 + vc[:, 1] ** 2 + m["eps_fric"] ** 2)
        a = m["mu"] * fn / nrm
        rhs += _mv(np.swapaxes(Jc, 1, 2), np.stack([-a * vc[:, 0], -a * vc[:, 1], fn], 1))
        w = np.stack([vc[:, 0] / nrm, vc[:, 1] / nrm, 0 * nrm], 1)
        z = np.array([0.0, 0.0, 1.0])
        D = a[:, None, None] * (np.eye(3) - z[:, None] * z - w[:, :, None] * w[:, None, :]) + m["d_contact"] * z[:, None] * z
        M += np.where(fn > 0, dt, 0.0)[:, None, None] * (np.swapaxes(Jc, 1, 2) @ D @ Jc)
    v = v + dt * np.linalg.solve(M, rhs[..., None])[..., 0]
    q = q.copy()
    q[:, 7 if fb else 0:] += dt * v[:, 6 if fb else 0:]
    if fb:
        q[:, :3] += dt * _mv(R[0], v[:, 3:6])
        w = v[:, :3]
        th = 0.5 * dt * np.linalg.norm(w, axis=1, keepdims=True)
        e0, e = np.cos(th), 0.5 * dt * np.sinc(th / np.pi) * w
        a0, a = q[:, 3:4], q[:, 4:7]
        r = np.concatenate([a0 * e0 - np.sum(a * e, 1, keepdims=True), a0 * e + e0 * a + np.cross(a, e)], 1)
        q[:, 3:7] = r / np.linalg.norm(r, axis=1, keepdims=True)
    return q, v, tau


def _spline(p, kn, nu, m, F):
    """Position and velocity at the integer time m of F per horizon ((K - 1) m / F knots in)."""
    K = p["n_knots"]
    kn = kn.reshape(-1, 2, K, nu)
    delta = p["horizon"] * p["dt"] / (K - 1)
    seg = min(m // F, K - 2)
    s = min((m - seg * F) / F, 1.0)
    q0, q1, m0, m1 = kn[..., 0, seg, :], kn[..., 0, seg + 1, :], delta * kn[..., 1, seg, :], delta * kn[..., 1, seg + 1, :]
    qr = (2 * s**3 - 3 * s**2 + 1) * q0 + (s**3 - 2 * s**2 + s) * m0 + (3 * s**2 - 2 * s**3) * q1 + (s**3 - s**2) * m1
    vr = ((6 * s**2 - 6 * s) * q0 + (3 * s**2 - 4 * s + 1) * m0 + (6 * s - 6 * s**2) * q1 + (3 * s**2 - 2 * s) * m1) / delta
    return qr, vr


def _slopes(p, pos):
    """Knot slopes of the position-only splines through pos [..., K, nu]."""
    K = p["n_knots"]
    delta = p["horizon"] * p["dt"] / (K - 1)
    if p["spline_mode"] == 2:
        out = [np.zeros(pos[..., 0, :].shape)]
        for k in range(K - 1):
            out.append(2 * (pos[..., k + 1, :] - pos[..., k, :]) / delta - out[-1])
        return np.stack(out, -2)
    A = 4 * np.eye(K) + np.eye(K, k=1) + np.eye(K, k=-1)
    A[0, 0] = A[-1, -1] = 2
    up = np.concatenate([pos[..., 1:, :], pos[..., -1:, :]], -2)
    dn = np.concatenate([pos[..., :1, :], pos[..., :-1, :]], -2)
    return np.linalg.solve(A, 3 * (up - dn) / delta)


def _philox(ctr, key):
    """Philox4x32-10 of the counters ctr [n, 4] (uint64 arrays of 32-bit words)."""
    c = [ctr[:, k].astype(np.uint64) for k in range(4)]
    k0, k1 = np.uint64(key & 0xffffffff), np.uint64(key >> 32)
    low = np.uint64(0xffffffff)
    for r in range(10):
        if r:
            k0, k1 = (k0 + np.uint64(0x9E3779B9)) & low, (k1 + np.uint64(0xBB67AE85)) & low
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ k0, p1 & low, (p0 >> np.uint64(32)) ^ c[3] ^ k1, p0 & low]
    return np.stack(c, 1)


def _samples(m, p, nseed, nominal, it):
    """Perturbed, clipped and clamped knots [N, 2, K, nu] of iteration `it` of a first call."""
    N, K, nu = p["n_samples"], p["n_knots"], m["n_u"]
    ku = K * nu
    blocks = (ku + 1) // 2
    ctr = np.zeros((N * blocks, 4), np.uint64)
    ctr[:, 0] = np.tile(np.arange(blocks), N)
    ctr[:, 1] = np.repeat(np.arange(N), blocks)
    ctr[:, 2] = it
    u = ((_philox(ctr, nseed) >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0**-23
    u = u.reshape(N, blocks * 2, 2)[:, :ku]
    r = np.sqrt(-2 * np.log(u[..., 0]))
    zq, zv = (r * f(2 * np.pi * u[..., 1]) for f in (np.cos, np.sin))
    zq[0] = zv[0] = 0
    k = np.arange(K)
    I = p["n_iters"]
    if p["noise_mode"] == 0:
        sig = p["scale_q"] * np.exp(-(I - it) / (p["beta1"] * I) - (K - k) / (p["beta2"] * K))
    else:
        sig = p["sigma_lo"] + (p["sigma_hi"] - p["sigma_lo"]) * k / (K - 1)
    sig = sig[:, None]
    nom = nominal.reshape(2, K, nu)
    delta = p["horizon"] * p["dt"] / (K - 1)
    q = np.clip(nom[0] + sig * zq.reshape(N, K, nu), m["q_min"], m["q_max"])
    if p["spline_mode"] != 0:
        return np.stack([q, _slopes(p, q)], 1)
    lim = 2 * np.minimum(m["q_max"] - q, q - m["q_min"]) / delta
    v = np.clip(nom[1] + sig / delta * zv.reshape(N, K, nu), -lim, lim)
    return np.stack([q, v], 1)


def _weights(costs, raw, lam):
    fine = np.isfinite(costs)
    lo, hi = costs[fine].min(), costs[fine].max()
    s = costs - lo if raw else (costs - lo) / (hi - lo if hi > lo else 1.0)
    w = np.where(fine, np.exp(-np.where(fine, s, 0.0) / lam), 0.0)
    return w / w.sum()


def _arm_step(case, seed):
    """A step of a fixed-base arm: every sample's cost, the nominal and the best sample."""
    m, p, nseed, x, nom = _problem(case, seed)
    N, H, nu, K = p["n_samples"], p["horizon"], m["n_u"], p["n_knots"]
    all_costs, best, s_best = [], nom, np.inf
    for it in range(p["n_iters"]):
        th = _samples(m, p, nseed, nom, it)
        q, v = np.tile(x[:nu], (N, 1)), np.tile(x[nu:], (N, 1))
        cost = np.zeros(N)

        def height(q):
            R, P = _bodies(m, q)
            return (P[m["ee_body"]] + R[m["ee_body"]] @ m["ee_pos"])[:, 2] - p["z_des"]

        for h in range(H):
            qr, vr = _spline(p, th, nu, h * (K - 1), H)
            cost += p["w_ee"] * height(q) ** 2
            q, v, tau = _control_step(m, q, v, qr, vr if p["spline_mode"] == 0 else 0.0 * vr, p["dt"])
            cost += p["w_tau"] * np.sum(tau ** 2, 1)
        cost += p["w_ee"] * height(q) ** 2
        th = th.reshape(N, -1)
        all_costs.append(cost)
        if cost.min() < s_best:
            s_best, best = cost.min(), th[int(np.argmin(cost))]
        nom = _weights(cost, p["weight_mode"] == 1, p["lambda"]) @ th
    return {"knots": nom, "best": best, "info": {"S_best": np.array([s_best]), "counts": None}, "costs": np.stack(all_costs)}


def exact(case, seed):
    if case["path"] == "update":
        costs, samples, nom = _update_inputs(case, seed)
        w = _weights(costs, case["raw"], 300.0 if case["raw"] else 1.0)
        return {"knots": w @ samples.astype(np.float64), "weights": w}
    if case["path"] == "predict":
        m, p, _, x, kn = _problem(case, seed)
        nu, K, F = m["n_u"], p["n_knots"], p["horizon"]
        q, v = x[None, :m["n_q"]], x[None, m["n_q"]:]
        for h in range(case["delay"]):
            qr, vr = _spline(p, kn, nu, h * (K - 1), F)
            q, v, _ = _control_step(m, q, v, qr, vr if p["spline_mode"] == 0 else 0.0 * vr, p["dt"])
        at = [_spline(p, kn, nu, k * F + case["delay"] * (K - 1), F) for k in range(K)]
        pos, vel = np.concatenate([a[0] for a in at]), np.concatenate([a[1] for a in at])
        if p["spline_mode"] != 0:
            vel = _slopes(p, pos)
        return {"state": np.concatenate([q[0], v[0]]), "knots": np.concatenate([pos.reshape(-1), vel.reshape(-1)])}
    if case["path"] == "step" and case["model"] in ("arm", "ytree") and case["samples"] * case["horizon"] * case["iters"] < 300000:
        return _arm_step(case, seed)
    return None
