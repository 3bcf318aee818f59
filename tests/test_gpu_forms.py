"""Launches in every kernel form, checked to be in it: both forms of the path kernel in
one launch, and body kernels beside them, against the body schedule's kernel (any
other lane count), bit for bit."""
import numpy as np
import pytest

from paper_2511_19204_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2511_19204_amd import mppi
    from test_gpu_numbering import PARENTS, _model
    from test_gpu_paths import TREES, _params, _past_one_turn, _step, _tree


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    mppi.lib()


def _dev(a):
    return torch.tensor(np.asarray(a, np.float32), device="cuda")


def _fleet(ms, ps):
    return [mppi.Controller(mppi.Model(m), p, 9 + i) for i, (m, p) in enumerate(zip(ms, ps))]


def _round(ctrls, ms, ps, how):
    xs = [_dev(m["x0"]) for m in ms]
    kin = []
    for m, p in zip(ms, ps):
        kn = synth.nominal_knots(m, p["n_knots"])
        kin.append(_dev(kn + np.random.default_rng(0).normal(0, 0.05, kn.size)))
    ko = [torch.zeros(c.E, device="cuda") for c in ctrls]
    best = [torch.zeros(c.E, device="cuda") for c in ctrls]
    info = [torch.zeros(mppi.INFO_INTS, dtype=torch.int32, device="cuda") for _ in ctrls]
    for c in ctrls:
        c.tick = 0
    if how == "graph":
        g = mppi.Graph(ctrls, xs, kin, ko, best, info)
        g.launch()
        torch.cuda.synchronize()
        g.close()
    else:
        mppi.step_batch(ctrls, xs, kin, ko, best, info)
    torch.cuda.synchronize()
    return [{"knots": a.cpu().numpy(), "best": b.cpu().numpy(), "info": c.cpu().numpy()} for a, b, c in zip(ko, best, info)]


@pytest.mark.parametrize("how", ["batch", "graph"])
@pytest.mark.parametrize("kind", ["both", "with_body"])
def test_mixed_launch_equals_the_body_schedule(kind, how):
    """both: long rollouts in the quad form beside one-lane ones, in one work table.
    with_body: trees that the body kernel takes in the same batch."""
    wide = _tree("eight_joints", False, [1] * 8)
    trees = {k: f() for k, f in TREES.items()}
    if kind == "both":
        # few long rollouts of deep trees, many short ones of all kinds
        names = [("humanoid", 37, 60), ("biped6", 21, 60), ("arm", 700, 9), ("quadruped", 610, 7), ("humanoid", 330, 5), ("ytree", 415, 8),
                 ("hexapod", 290, 6), ("forked_legs", 203, 6), ("long_arm", 333, 9)]
        ms = [trees[n] for n, _, _ in names]
    else:
        names = [("quadruped", 605, 20), ("wide", 2049, 24), ("humanoid", 301, 16), ("wide", 4100, 21), ("arm", 333, 30)]
        ms = [wide if n == "wide" else trees[n] for n, _, _ in names]
    want = {"both": {"quad", "lane"}, "with_body": {"schedule"}}[kind]
    # samples by the size of the device, until its SIMDs do not hold the launch at once
    for scale in (1, 2, 4, 8, 16):
        ps = [_params(m, n * (1 if h == 60 else scale) + i, horizon=h, iters=1 + i % 2) for i, (m, (_, n, h)) in enumerate(zip(ms, names))]
        ctrls = _fleet(ms, ps)
        forms = mppi.launch_forms(ctrls)
        if want <= set(forms) and len(set(forms)) > 1:
            break
    print(kind, scale, list(zip([n for n, _, _ in names], forms)))
    assert want <= set(forms) and len(set(forms)) > 1
    got = _round(ctrls, ms, ps, how)
    for i, (m, p, c) in enumerate(zip(ms, ps, ctrls)):
        other = mppi.Controller(mppi.Model(m), p, 9 + i, lanes=2 * c.lanes)
        assert mppi.launch_forms([other]) == ["schedule"]
        ref = _step(other, m, p)
        for k in got[i]:
            assert np.array_equal(got[i][k], ref[k], equal_nan=True), (names[i], forms[i], k)


# trees that are as fast or faster in the body kernel past one turn of the device: the
# one-lane form takes their kinds where the numbering keeps them off the depth-specialised
# body kernels (PARENTS: two legs, fixed bodies that paths share, six legs of four, ...)
BODY_PAST_ONE_TURN = {"biped", "forked_arm", "hexapod4", "tripod"}


@pytest.mark.parametrize("name", sorted(TREES) if torch.cuda.is_available() else [])
def test_forms_by_size(name):
    """The sizes of the tests of each form are in it."""
    m = TREES[name]()
    model = mppi.Model(m)
    assert mppi.launch_forms([mppi.Controller(model, _params(m, 67), 1)]) == ["quad"]
    many = mppi.Controller(model, _params(m, _past_one_turn(m), horizon=7, iters=1), 1)
    assert mppi.launch_forms([many]) == ["schedule" if name in BODY_PAST_ONE_TURN else "lane"]
    assert mppi.launch_forms([mppi.Controller(model, _params(m, 67), 1, schedule="chain")]) == ["schedule"]


@pytest.mark.parametrize("name", sorted(PARENTS) if torch.cuda.is_available() else [])
def test_forms_of_other_numberings(name):
    m = _model(name)
    model = mppi.Model(m)
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + 5
    assert mppi.launch_forms([mppi.Controller(model, _params(m, 67), 1)]) == ["quad"]
    got = mppi.launch_forms([mppi.Controller(model, _params(m, n), 1)])
    # (the numbering of "three_reversed" is one that the depth-specialised body kernels take)
    assert got == ["schedule" if name == "three_reversed" else "lane"], got


@pytest.mark.parametrize("legs,floating,n", [([1] * 8, False, 8200), ([1] * 4, True, 8200), ([2] * 6, True, 16400)])
def test_wide_shallow_trees_in_the_body_kernel(legs, floating, n):
    m = _tree("wide", floating, legs)
    p = _params(m, n, horizon=9, iters=2)
    model = mppi.Model(m)
    c = mppi.Controller(model, p, 77)
    assert mppi.launch_forms([c]) == ["schedule"]
    a, b = _step(c, m, p), _step(mppi.Controller(model, p, 77, lanes=2 * c.lanes), m, p)
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k


def test_launch_forms_arguments():
    with pytest.raises(mppi.MppiError):
        mppi.launch_forms([])
