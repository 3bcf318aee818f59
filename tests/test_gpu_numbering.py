"""Trees whose bodies are not numbered depth first: a model only asks that a parent
comes before its children.  Every schedule and form of a launch sweeps them as the
FP64 oracle does."""
import numpy as np
import pytest

import oracle as O
from paper_2511_19204_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2511_19204_amd import mppi


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    mppi.lib()


PARENTS = {
    # the first leaf hangs off the base's second child
    "two_legs": [-1, 0, 0, 1],
    "three_reversed": [-1, 0, 0, 0, 3, 2, 1],
    "four_ragged": [-1, 0, 0, 0, 0, 1, 3, 4, 6],
    # eight legs of one to three bodies, level by level
    "eight_ragged": [-1, 0, 0, 0, 0, 0, 0, 0, 0, 8, 1, 6, 3, 10, 9],
    "six_of_four": [-1] + [0] * 6 + list(range(1, 19)),
    # the bodies several paths share are numbered before and after other legs
    "forked": [-1, 0, 0, 2, 1, 3, 1, 2, 6, 4, 5],
    "forked_fixed": [-1, -1, 0, 1, 0, 1, 3, 2, 4],
}


def _model(name, seed=3):
    par = PARENTS[name]
    floating = "fixed" not in name
    rng = np.random.default_rng(seed)
    t = synth._Tree()
    axes = [(1, 0, 0), (0, 1, 0), (0, 1, 0), (0, 0, 1)]
    for b, p in enumerate(par):
        if floating and b == 0:
            t.body(-1, (0, 0, 1), (0, 0, 0), 8.0, (0.01, 0.02, -0.01), (0.4, 0.3, 0.1))
            continue
        at = (0.2 * np.cos(b), 0.2 * np.sin(b), 0.0) if p <= 0 else (0.02, 0.01, -0.15)
        t.body(p, axes[b % 4], at, rng.uniform(0.5, 1.5), tuple(rng.uniform(-0.05, 0.05, 3)), (0.05, 0.04, 0.15),
               joint=(-1.5, 1.5, 30.0, 60.0, 2.0, float(rng.uniform(-0.3, 0.3))))
    leaves = sorted(set(range(len(par))) - set(par))
    cb, cp = (leaves, [(0.0, 0.0, -0.15)] * len(leaves)) if floating else ([], np.zeros((0, 3)))
    m = t.finish(name, floating, cb, cp, ee_body=leaves[0], ee_pos=(0, 0, -0.1))
    m["n_substeps"] = 1
    m["armature"] = synth.f32(np.full(m["n_u"], 0.1))
    m["k_contact"], m["d_contact"] = 2e3, 50.0
    q = np.zeros(m["n_q"])
    if floating:
        q[2], q[3] = 0.12, 1.0  # some of the points start in the ground
    m["x0"] = synth.f32(np.concatenate([q, rng.normal(0, 0.2, m["n_v"])]))
    return m


def _params(m, n, horizon, iters=1):
    return synth.params(m, n, horizon, 0.005, 5, iters, ("exp", 0.4, 1.0, 1.0), "walking" if m["floating_base"] else "ee")


def _dev(a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda")


def _knots(m, p):
    kn = synth.nominal_knots(m, p["n_knots"])
    return kn + np.random.default_rng(0).normal(0, 0.05, kn.size)


def _step(c, m, p):
    out = {"knots": torch.zeros(c.E, device="cuda"), "best": torch.zeros(c.E, device="cuda"),
           "info": torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda"),
           "costs": torch.zeros((p["n_iters"], p["n_samples"]), device="cuda")}
    c.step(_dev(m["x0"]), _dev(_knots(m, p)), out["knots"], out["best"], out["info"], out["costs"])
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("how", ["lanes", "more_lanes", "chain", "team"])
@pytest.mark.parametrize("name", sorted(PARENTS))
def test_rollout_costs_match_oracle(name, how):
    """Within 1e-3 relative over a horizon too short for contacts to amplify rounding,
    or 4 times the oracle's own FP32 error where that is larger."""
    m = _model(name)
    p = _params(m, 24, 10)
    c = mppi.Controller(mppi.Model(m), p, 7)
    if how == "more_lanes":
        c.set_lanes(2 * c.lanes)
    elif how != "lanes":
        c.set_schedule(how)
    kn = _knots(m, p)
    smp = np.stack([synth.f32(O.sample_knots(m, p, kn, 7, 0, 0, k)) for k in range(24)])
    costs = torch.zeros(24, device="cuda")
    c.rollouts(_dev(m["x0"]), _dev(smp), costs, None)
    torch.cuda.synchronize()
    ref = np.array([O.rollout(m, p, m["x0"], s) for s in smp])
    f32 = np.array([O.rollout_f32(m, p, m["x0"], s)[0] for s in smp])
    rel, rel32 = np.abs(costs.cpu().numpy() - ref) / np.abs(ref), np.abs(f32 - ref) / np.abs(ref)
    print(f"{name} {how}: max rel err {rel.max():.2e} (oracle-f32 {rel32.max():.2e})")
    assert rel.max() <= max(1e-3, 4 * rel32.max())


@pytest.mark.parametrize("name", sorted(PARENTS))
def test_schedules_and_persistent_launches_agree(name):
    """The body schedule at two lane counts above its default, the chain schedule and
    the persistent form of a batch: the same bits."""
    m = _model(name)
    p = _params(m, 67, 30, iters=2)
    model = mppi.Model(m)
    c = mppi.Controller(model, p, 77)
    a = _step(mppi.Controller(model, p, 77, lanes=2 * c.lanes), m, p)
    assert np.all(np.isfinite(a["costs"]))
    others = {"chain": _step(mppi.Controller(model, p, 77, schedule="chain"), m, p)}
    if 4 * c.lanes <= 64:
        others["lanes"] = _step(mppi.Controller(model, p, 77, lanes=4 * c.lanes), m, p)
    out = [torch.zeros(c.E, device="cuda"), torch.zeros(c.E, device="cuda")]
    mppi.set_batch_options(True)
    try:
        mppi.step_batch([c], [_dev(m["x0"])], [_dev(_knots(m, p))], [out[0]], [out[1]])
    finally:
        mppi.set_batch_options(False)
    torch.cuda.synchronize()
    others["persistent"] = {"knots": out[0].cpu().numpy(), "best": out[1].cpu().numpy()}
    for how, b in others.items():
        for k in b:
            assert np.array_equal(a[k], b[k]), (name, how, k)


def test_traced_states_match_oracle():
    """A traced rollout's states against the oracle's, within 1e-3 of the largest
    component or 4 times the oracle's own FP32 error where that is larger."""
    m = _model("four_ragged")
    p = _params(m, 3, 8)
    c = mppi.Controller(mppi.Model(m), p, 5)
    nq, nv, H = m["n_q"], m["n_v"], p["horizon"]
    kn = synth.f32(synth.nominal_knots(m, p["n_knots"]))
    trace = torch.zeros((1, H + 1, nq + 2 * nv + 2), device="cuda")
    c.trace(_dev(m["x0"]), _dev(kn), 0, 0, torch.tensor([0, -1, -1], dtype=torch.int32, device="cuda"), trace,
            torch.zeros((3, c.E), device="cuda"), torch.zeros(3, device="cuda"),
            torch.zeros((3, H), dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    got = trace.cpu().numpy()[0, :, :nq + nv]
    for h in (1, 4, 8):
        ref = O.predict(m, p, m["x0"], kn, h)
        scale = max(1.0, np.abs(ref).max())
        f32 = np.abs(O.predict_f32(m, p, m["x0"], kn, h) - ref).max() / scale
        err = np.abs(got[h] - ref).max() / scale
        print(f"step {h}: {err:.2e} (oracle-f32 {f32:.2e})")
        assert err <= max(1e-3, 4 * f32), h


@pytest.mark.parametrize("form", ["quad", "lane"])
@pytest.mark.parametrize("name", sorted(PARENTS))
def test_path_kernel_adds_children_in_body_order(name, form):
    """The default lane count (the path kernel) against another one, bit for bit: the
    paths that bring the base's children are added in the children's order."""
    m = _model(name)
    # the one-lane form's range begins past the quad form's wavefronts of one turn of the device
    n = 67 if form == "quad" else 64 * torch.cuda.get_device_properties(0).multi_processor_count + 5
    p = _params(m, n, 40 if form == "quad" else 20)
    model = mppi.Model(m)
    c = mppi.Controller(model, p, 77)
    a, b = _step(c, m, p), _step(mppi.Controller(model, p, 77, lanes=2 * c.lanes), m, p)
    assert np.all(np.isfinite(a["costs"]))
    for k in a:
        assert np.array_equal(a[k], b[k]), (name, k, int(np.sum(a[k] != b[k])))


@pytest.mark.parametrize("name", sorted(PARENTS))
def test_prediction_equals_the_traced_rollout(name):
    m = _model(name)
    p = _params(m, 3, 12)
    c = mppi.Controller(mppi.Model(m), p, 5)
    kn, x = _dev(synth.nominal_knots(m, p["n_knots"])), _dev(m["x0"])
    nx, rec = m["n_q"] + m["n_v"], m["n_q"] + 2 * m["n_v"] + 2
    trace = torch.zeros((1, 13, rec), device="cuda")
    c.trace(x, kn, 0, 0, torch.tensor([0, -1, -1], dtype=torch.int32, device="cuda"), trace,
            torch.zeros((3, c.E), device="cuda"), torch.zeros(3, device="cuda"),
            torch.zeros((3, 12), dtype=torch.int32, device="cuda"))
    for n in (1, 7, 12):
        out = torch.zeros(nx, device="cuda")
        c.predict(x, kn, n, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), trace[0, n, :nx].cpu().numpy()), n
