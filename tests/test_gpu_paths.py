"""The path kernel (a quad of lanes, or one lane, per root-to-leaf path of the
tree) against the body schedule's kernel, bit for bit: the body schedule at its default lane
count takes it, at any other lane count it does not, and a step's results do
not depend on the lane count.  Trees of every kind the kernel is compiled for
(path counts, path lengths, fixed and floating bases, bodies that several paths
share, contacts on inner bodies and on the base), at the sample counts where a
wavefront is partly filled."""
import numpy as np
import pytest

from paper_2511_19204_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2511_19204_amd import mppi


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    mppi.lib()


def _tree(name, floating, legs, fork=None, seed=3):
    """A tree of serial legs (their lengths in `legs`) on a floating base or on the
    world; every leaf has a contact point.
    fork = (leg, body of the leg, lengths): further legs that hang off that body."""
    rng = np.random.default_rng(seed)
    t = synth._Tree()
    axes = [(1, 0, 0), (0, 1, 0), (0, 1, 0), (0, 0, 1)]
    if floating:
        t.body(-1, (0, 0, 1), (0, 0, 0), 8.0, (0.01, 0.02, -0.01), (0.4, 0.3, 0.1))
    leaves, body_of = [], {}

    def leg(k, root, n):
        par = root
        for i in range(n):
            p = (0.2 * np.cos(k), 0.2 * np.sin(k), 0.0) if i == 0 else (0.02, 0.01, -0.15)
            par = t.body(par, axes[i % 4], p, rng.uniform(0.5, 1.5), tuple(rng.uniform(-0.05, 0.05, 3)), (0.05, 0.04, 0.15),
                         joint=(-1.5, 1.5, 30.0, 60.0, 2.0, float(rng.uniform(-0.3, 0.3))))
            body_of[(k, i)] = par
        leaves.append(par)

    # depth first: a fork's legs follow the leg they hang off
    for k, n in enumerate(legs):
        if fork and fork[0] == k:
            leg(k, 0 if floating else -1, fork[1] + 1)
            leaves.pop()
            root = body_of[(k, fork[1])]
            for f, nf in enumerate(fork[2]):
                leg(10 + f, root, nf)
        else:
            leg(k, 0 if floating else -1, n)
    cb, cp = list(leaves), [(0.0, 0.0, -0.15)] * len(leaves)
    if floating:
        cb += [leaves[0], leaves[0], 0, body_of[(0, 0)]]
        cp += [(0.03, 0.0, -0.15), (-0.03, 0.01, -0.15), (0.1, 0.0, -0.05), (0.0, 0.0, -0.1)]
    m = t.finish(name, floating, cb if floating else [], cp if floating else np.zeros((0, 3)), ee_body=leaves[-1],
                 ee_pos=(0, 0, -0.1))
    m["n_substeps"] = 1
    m["armature"] = synth.f32(np.full(m["n_u"], 0.1))
    m["k_contact"], m["d_contact"] = 2e3, 50.0
    q = np.zeros(m["n_q"])
    if floating:
        q[2], q[3] = 0.12, 1.0  # some of the points start in the ground
    m["x0"] = synth.f32(np.concatenate([q, rng.normal(0, 0.2, m["n_v"])]))
    return m


TREES = {
    "arm": lambda: synth.chain_model(1),
    "ytree": lambda: synth.ytree_model(1),
    "three_arms": lambda: _tree("three_arms", False, [3, 2, 1]),
    "long_arm": lambda: _tree("long_arm", False, [6]),
    "forked_arm": lambda: _tree("forked_arm", False, [2], fork=(0, 1, [2, 3, 1])),
    "seven_arms": lambda: _tree("seven_arms", False, [2, 1, 3, 2, 1, 2, 3]),
    "monopod": lambda: _tree("monopod", True, [3]),
    "monopod5": lambda: _tree("monopod5", True, [5]),
    "biped": lambda: _tree("biped", True, [3, 2]),
    "biped6": lambda: _tree("biped6", True, [6, 4]),
    "tripod": lambda: _tree("tripod", True, [3, 3, 1]),
    "quadruped": lambda: synth.quadruped_model(2),
    "hexapod": lambda: synth.hexapod_model(2),
    "hexapod4": lambda: _tree("hexapod4", True, [4, 4, 3, 4, 2, 4]),
    "humanoid": lambda: synth.humanoid_model(2),
    "forked_legs": lambda: _tree("forked_legs", True, [3, 2, 4], fork=(1, 1, [3, 4])),
}


def _params(m, n, horizon=24, knots=5, iters=2, cost=None, **more):
    cost = cost or ("walking" if m["floating_base"] else "ee")
    p = synth.params(m, n, horizon, 0.005, knots, iters, ("exp", 0.4, 1.0, 1.0), cost)
    p.update(more)
    return p


def _step(c, m, p, seed=0):
    rng = np.random.default_rng(seed)
    kn = synth.nominal_knots(m, p["n_knots"])
    kn = kn + (rng.normal(0, 0.05, kn.size) if p.get("spline_mode", 0) == 0 else 0.0)
    dev = lambda a: torch.tensor(np.asarray(a, np.float32), device="cuda")  # noqa: E731
    out = {"knots": torch.zeros(c.E, device="cuda"), "best": torch.zeros(c.E, device="cuda"),
           "info": torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda"),
           "costs": torch.zeros((p["n_iters"], p["n_samples"]), device="cuda")}
    c.step(dev(m["x0"]), dev(kn), out["knots"], out["best"], out["info"], out["costs"])
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def _both(m, p, seed=77):
    """The step through the path kernel and through the body schedule's kernel."""
    model = mppi.Model(m)
    c = mppi.Controller(model, p, seed)
    other = mppi.Controller(model, p, seed, lanes=2 * c.lanes)
    assert other.lanes == 2 * c.lanes
    return _step(c, m, p), _step(other, m, p)


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), (what, k)


@pytest.mark.parametrize("name", sorted(TREES))
@pytest.mark.parametrize("n", [1, 5, 67])
def test_path_kernel_equals_body_schedule(name, n):
    m = TREES[name]()
    a, b = _both(m, _params(m, n))
    print(f"{name} N={n}: costs[0][:3] {a['costs'][0][:3]}")
    assert np.any(np.isfinite(a["costs"]))
    _same(a, b, (name, n))


def _past_one_turn(m):
    """Just more samples than the quad form's wavefronts of one turn of the device
    (four SIMDs per compute unit) hold: the one-lane form's range begins."""
    leaves = len(set(range(len(m["parent"]))) - set(int(p) for p in m["parent"]) - ({0} if m["floating_base"] else set()))
    lanes = 4 * (1 if leaves <= 1 else 2 if leaves <= 2 else 4 if leaves <= 4 else 8)
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count * (64 // lanes) + 37


@pytest.mark.parametrize("name", sorted(TREES))
def test_one_lane_form_equals_body_schedule(name):
    m = TREES[name]()
    n = _past_one_turn(m)
    a, b = _both(m, _params(m, n, horizon=7, iters=1))
    print(f"{name} N={n}: costs[0][:3] {a['costs'][0][:3]}")
    assert np.any(np.isfinite(a["costs"]))
    _same(a, b, (name, n))


@pytest.mark.parametrize("more", [dict(spline_mode=1), dict(spline_mode=2, knots=4), dict(substeps=3),
                                  dict(weight_mode=1, horizon=1), dict(q_des=[0.96, 0.0, 0.28, 0.0]), dict(knots=40)])
def test_one_lane_form_options(more):
    more = dict(more)
    m = dict(TREES["quadruped"]())
    m["n_substeps"] = more.pop("substeps", 1)
    a, b = _both(m, _params(m, _past_one_turn(m), **{"horizon": 7, "iters": 1, **more}))
    _same(a, b, more)


@pytest.mark.parametrize("name", ["arm", "quadruped", "humanoid", "forked_legs"])
@pytest.mark.parametrize("more", [dict(spline_mode=1), dict(spline_mode=2, knots=4), dict(substeps=3),
                                  dict(weight_mode=1, horizon=1), dict(q_des=[0.96, 0.0, 0.28, 0.0])])
def test_options(name, more):
    more = dict(more)
    m = dict(TREES[name]())
    m["n_substeps"] = more.pop("substeps", 1)
    a, b = _both(m, _params(m, 21, **more))
    _same(a, b, (name, more))


@pytest.mark.parametrize("name", ["biped", "hexapod4"])
def test_end_effector_cost_on_a_floating_tree(name):
    m = TREES[name]()
    a, b = _both(m, _params(m, 9, cost="ee"))
    _same(a, b, name)


def test_end_effector_on_the_base_keeps_the_body_kernel():
    m = dict(TREES["biped"](), ee_body=0)
    a, b = _both(m, _params(m, 9, cost="ee"))
    _same(a, b, "base")


@pytest.mark.parametrize("name", ["ytree", "biped6", "quadruped", "hexapod", "humanoid"])
def test_prediction_equals_the_traced_rollout(name):
    """The state predicted n steps ahead is the state the body schedule's traced
    rollout of the same trajectory (sample 0, the nominal) has there."""
    m = TREES[name]()
    p = _params(m, 3, horizon=12)
    c = mppi.Controller(mppi.Model(m), p, 5)
    kn = torch.tensor(synth.nominal_knots(m, p["n_knots"]), dtype=torch.float32, device="cuda")
    x = torch.tensor(m["x0"], dtype=torch.float32, device="cuda")
    nx, rec = m["n_q"] + m["n_v"], m["n_q"] + 2 * m["n_v"] + 2
    tmap = torch.tensor([0, -1, -1], dtype=torch.int32, device="cuda")
    trace = torch.zeros((1, 13, rec), device="cuda")
    c.trace(x, kn, 0, 0, tmap, trace, torch.zeros((3, c.E), device="cuda"), torch.zeros(3, device="cuda"),
            torch.zeros((3, 12), dtype=torch.int32, device="cuda"))
    for n in (0, 1, 7, 12):
        out = torch.zeros(nx, device="cuda")
        c.predict(x, kn, n, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), trace[0, n, :nx].cpu().numpy()), (name, n)


@pytest.mark.parametrize("scale", [1, 40])
def test_mixed_batch_equals_plain_steps(scale):
    """scale 1: the batch fits the device at once (quad form); 40: it does not (both
    forms in one launch)."""
    names = ["arm", "quadruped", "humanoid", "ytree", "hexapod", "quadruped"]
    ms = [TREES[n]() for n in names]
    ps = [_params(m, 11 * scale + 6 * i, horizon=15 + i * i, iters=1 + i % 3) for i, m in enumerate(ms)]
    models = [mppi.Model(m) for m in ms]
    plain = [_step(mppi.Controller(md, p, 9 + i), m, p) for i, (md, m, p) in enumerate(zip(models, ms, ps))]
    ctrls = [mppi.Controller(md, p, 9 + i) for i, (md, p) in enumerate(zip(models, ps))]
    dev = lambda a: torch.tensor(np.asarray(a, np.float32), device="cuda")  # noqa: E731
    kin = []
    for m, p in zip(ms, ps):
        kn = synth.nominal_knots(m, p["n_knots"])
        kin.append(dev(kn + np.random.default_rng(0).normal(0, 0.05, kn.size)))
    xs = [dev(m["x0"]) for m in ms]
    ko = [torch.zeros(c.E, device="cuda") for c in ctrls]
    best = [torch.zeros(c.E, device="cuda") for c in ctrls]
    info = [torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda") for _ in ctrls]
    mppi.step_batch(ctrls, xs, kin, ko, best, info)
    torch.cuda.synchronize()
    for i, a in enumerate(plain):
        for k, t in (("knots", ko[i]), ("best", best[i]), ("info", info[i])):
            assert np.array_equal(a[k], t.cpu().numpy(), equal_nan=True), (names[i], k)


@pytest.mark.parametrize("copies,sizes", [(8, (1, 15, 16, 17, 63, 64, 65, 1008, 1024, 1025)), (2, (1000, 1023, 1025, 4097))])
@pytest.mark.parametrize("name,knots", [("arm", 4), ("arm", 5), ("hexapod", 4)])
def test_update_forms_agree(copies, sizes, name, knots):
    """The update's parts spread over workgroups of a few element blocks (an instance
    alone) and whole (a launch of more than 1024 parts): sizes around a slice of 16 samples, the
    last slice and the width's limit of 1024 samples, an odd and an even number of
    knot elements (stored samples and samples drawn again), a last tile that is not full."""
    m = TREES[name]()
    ps = [_params(m, n, horizon=2, knots=knots, iters=2) for n in sizes] * copies
    parts = sum((p["n_samples"] + 15) // 16 for p in ps if p["n_samples"] <= 1024)
    model = mppi.Model(m)
    x = torch.tensor(np.asarray(m["x0"], np.float32), device="cuda")
    ctrls = [mppi.Controller(model, p, 3 + i) for i, p in enumerate(ps)]
    kn = torch.tensor(np.asarray(synth.nominal_knots(m, knots), np.float32), device="cuda")
    out = {}
    for form in ("alone", "batch"):
        ko = [torch.zeros(c.E, device="cuda") for c in ctrls]
        best = [torch.zeros(c.E, device="cuda") for c in ctrls]
        info = [torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda") for _ in ctrls]
        for c in ctrls:
            c.tick = 0
        if form == "alone":
            for i, c in enumerate(ctrls):
                c.step(x, kn, ko[i], best[i], info[i])
        else:
            mppi.step_batch(ctrls, [x] * len(ctrls), [kn] * len(ctrls), ko, best, info)
        torch.cuda.synchronize()
        out[form] = [[t.cpu().numpy() for t in ts] for ts in zip(ko, best, info)]
    assert (parts > 1024) == (copies == 8), parts
    for p, a, b in zip(ps, out["alone"], out["batch"]):
        for s, t in zip(a, b):
            assert np.array_equal(s, t, equal_nan=True), p["n_samples"]
