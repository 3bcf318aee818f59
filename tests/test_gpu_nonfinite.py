"""Rollouts that overflow or start from values that are not finite: the path kernel's
forms and its prediction against the body schedule's kernel.  Past a path's end the
path kernel walks massless bodies, which multiply what may be infinite by zero."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2511_19204_amd import mppi, synth
    from test_gpu_paths import TREES, _params, _past_one_turn, _step


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    mppi.lib()


NAMES = ["arm", "three_arms", "seven_arms", "forked_arm", "monopod", "biped", "quadruped", "hexapod4", "humanoid"]
# (state component from the end, value): the last joint's velocity and angle, the base's
STARTS = {"fast": ("v", -1, 1e19), "faster": ("v", -1, 3e38), "first_joint": ("v", "first", 3e38), "inf": ("v", -1, np.inf),
          "nan": ("v", -1, np.nan), "far": ("q", -1, 1e30), "base": ("v", 0, 1e25)}


def _model(name, start):
    m = dict(TREES[name]())
    x = np.array(m["x0"], np.float32)
    what, i, value = STARTS[start]
    if i == "first":
        i = 6 if m["floating_base"] else 0
    at = (m["n_q"] if what == "v" else 0) + (i if i >= 0 else (m["n_v"] if what == "v" else m["n_q"]) + i)
    x[at] = value
    m["x0"] = x
    return m


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), (what, k)


@pytest.mark.parametrize("start", sorted(STARTS))
@pytest.mark.parametrize("name", NAMES)
def test_starts_that_overflow(name, start):
    m = _model(name, start)
    model = mppi.Model(m)
    for p in (_params(m, 67, horizon=6, iters=2), _params(m, _past_one_turn(m), horizon=3, iters=1)):
        c = mppi.Controller(model, p, 77)
        a, b = _step(c, m, p), _step(mppi.Controller(model, p, 77, lanes=2 * c.lanes), m, p)
        print(f"{name} {start} N={p['n_samples']} {mppi.launch_forms([c])}: {np.isinf(a['costs']).mean():.2f} of the costs infinite")
        assert not np.any(np.isnan(a["costs"]))
        _same(a, b, (name, start, p["n_samples"]))


@pytest.mark.parametrize("name", NAMES)
def test_some_samples_diverge(name):
    """Gains that throw some of the samples off: their costs are infinite, the others' stay."""
    m = dict(TREES[name]())
    m["d_contact"], m["k_contact"], m["armature"] = 0.0, 1e9, synth.f32(np.full(m["n_u"], 1e-4))
    m["kd"], m["tau_max"] = synth.f32(np.full(m["n_u"], -40.0)), synth.f32(np.full(m["n_u"], 1e30))
    model = mppi.Model(m)
    for p in (_params(m, 67, horizon=60, iters=1), _params(m, _past_one_turn(m), horizon=60, iters=1)):
        c = mppi.Controller(model, p, 77)
        a, b = _step(c, m, p), _step(mppi.Controller(model, p, 77, lanes=2 * c.lanes), m, p)
        print(f"{name} N={p['n_samples']}: {np.isinf(a['costs']).mean():.2f} of the costs infinite")
        _same(a, b, (name, p["n_samples"]))


@pytest.mark.parametrize("start", sorted(STARTS))
@pytest.mark.parametrize("name", NAMES)
def test_prediction_of_starts_that_overflow(name, start):
    """The predicted state is finite where the traced rollout's is, and the same there."""
    m = _model(name, start)
    p = _params(m, 3, horizon=4)
    c = mppi.Controller(mppi.Model(m), p, 5)
    kn = torch.tensor(synth.nominal_knots(m, p["n_knots"]), dtype=torch.float32, device="cuda")
    x = torch.tensor(m["x0"], dtype=torch.float32, device="cuda")
    nx, rec = m["n_q"] + m["n_v"], m["n_q"] + 2 * m["n_v"] + 2
    trace = torch.zeros((1, 5, rec), device="cuda")
    c.trace(x, kn, 0, 0, torch.tensor([0, -1, -1], dtype=torch.int32, device="cuda"), trace,
            torch.zeros((3, c.E), device="cuda"), torch.zeros(3, device="cuda"),
            torch.zeros((3, 4), dtype=torch.int32, device="cuda"))
    for n in (1, 2, 4):
        out = torch.zeros(nx, device="cuda")
        c.predict(x, kn, n, out)
        torch.cuda.synchronize()
        a, b = out.cpu().numpy(), trace[0, n, :nx].cpu().numpy()
        ok = np.isfinite(b)
        assert np.array_equal(np.isfinite(a), ok), (n, a, b)
        assert np.array_equal(a[ok], b[ok]), (n, a, b)
