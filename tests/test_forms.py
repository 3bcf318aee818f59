"""Choice of a launch's kernel forms (csrc/mppi_forms.hpp), on the CPU: against step
times measured on the MI355X, and the linear split against a plain search."""
import ctypes as C
import os
import random
import subprocess

import numpy as np
import pytest

from paper_2511_19204_amd import build

BODY, QUAD, LANE = 0, 1, 2
FIELDS = ("path", "folds", "floating", "serial", "shared", "depth", "path_len", "path_lanes", "body_key", "base_children",
          "contacts_max", "contacts_path", "samples", "steps", "quad_lds", "lane_lds", "body_lds")
SIMDS = 1024  # 256 compute units
SHIM = """
#include "mppi_forms.hpp"
extern "C" void forms(int n, const double* f, int simds, int* out) {
  std::vector<mppi::FormDesc> list(n);
  for (int i = 0; i < n; ++i) {
    mppi::FormDesc& d = list[i];
    const double* x = f + 17 * i;
    d.path = x[0]; d.folds = x[1]; d.floating = x[2]; d.serial = x[3]; d.shared = x[4]; d.depth = x[5];
    d.path_len = x[6]; d.path_lanes = x[7]; d.body_key = x[8]; d.base_children = x[9]; d.contacts_max = x[10];
    d.contacts_path = x[11]; d.samples = x[12]; d.steps = x[13]; d.quad_lds = x[14]; d.lane_lds = x[15]; d.body_lds = x[16];
  }
  const std::vector<mppi::Form> r = mppi::choose_forms(list, simds);
  for (int i = 0; i < n; ++i) out[i] = r[i];
}
"""

# tree: floating, serial, shared bodies, depth, bodies per path of the kernel, lanes per
# rollout of the quad form and of the body kernel, the base's children, contacts
# of a body, contacts along a path.  cN: a chain; wABC: fixed arms of A, B, C
# bodies; fABC: such legs on a floating base; fork: bodies that paths share.
TREES = {
    "c1": (0, 1, 0, 1, 3, 4, 4, 0, 0, 0),
    "c2": (0, 1, 0, 2, 3, 4, 4, 0, 0, 0),
    "c3": (0, 1, 0, 3, 3, 4, 4, 0, 0, 0),
    "c6": (0, 1, 0, 6, 6, 4, 8, 0, 0, 0),
    "w1111": (0, 0, 0, 1, 3, 16, 4, 0, 0, 0),
    "w11111111": (0, 0, 0, 1, 3, 32, 8, 0, 0, 0),
    "w2222": (0, 0, 0, 2, 3, 16, 8, 0, 0, 0),
    "w22222222": (0, 0, 0, 2, 3, 32, 16, 0, 0, 0),
    "w33333333": (0, 0, 0, 3, 3, 32, 32, 0, 0, 0),
    "f1": (1, 0, 0, 1, 3, 4, 4, 1, 1, 1),
    "f1111": (1, 0, 0, 1, 3, 16, 8, 4, 1, 1),
    "f11111111": (1, 0, 0, 1, 3, 32, 16, 8, 1, 1),
    "f222222": (1, 0, 0, 2, 3, 32, 16, 6, 1, 1),
    "f33333333": (1, 0, 0, 3, 3, 32, 32, 8, 1, 1),
    "f6666": (1, 0, 0, 6, 6, 16, 32, 4, 1, 1),
    "f61111111": (1, 0, 0, 6, 6, 32, 16, 8, 1, 2),
    "fork_8x1": (0, 0, 1, 2, 4, 16, 8, 0, 0, 0),
    "quadruped": (1, 0, 0, 3, 3, 16, 16, 4, 1, 1),
    "hexapod": (1, 0, 0, 3, 3, 32, 32, 6, 1, 1),
    "humanoid": (1, 0, 1, 6, 6, 16, 32, 3, 4, 5),
}
# (tree, samples, microseconds a step in the body kernel, in the better form of the path kernel)
MEASURED = [
    ("c1", 1024, 1.68, 1.72), ("c1", 8192, 1.67, 1.77), ("c1", 16384, 1.63, 1.86), ("c1", 32768, 2.11, 3.03), ("c1", 65536, 4.07, 2.96),
    ("c2", 1024, 2.27, 1.71), ("c2", 8192, 2.09, 1.79), ("c2", 16384, 2.11, 1.85), ("c2", 32768, 3.05, 3.01), ("c2", 65536, 5.85, 2.99),
    ("c3", 1024, 2.66, 1.69), ("c3", 8192, 2.56, 1.79), ("c3", 16384, 2.53, 1.81), ("c3", 32768, 3.76, 3.05), ("c3", 65536, 7.31, 2.97),
    ("c6", 8192, 5.48, 3.73), ("c6", 16384, 7.29, 3.65), ("c6", 32768, 14.49, 6.96), ("c6", 65536, 28.19, 6.72),
    ("w1111", 8192, 2.17, 3.00), ("w1111", 16384, 2.04, 2.95), ("w1111", 32768, 2.72, 5.91), ("w1111", 65536, 5.26, 11.78),
    ("w11111111", 8192, 2.10, 2.94), ("w11111111", 16384, 2.71, 5.92), ("w11111111", 32768, 5.28, 11.86), ("w11111111", 65536, 10.19, 23.57),
    ("w2222", 8192, 2.64, 3.03), ("w2222", 16384, 3.35, 2.95), ("w2222", 32768, 6.58, 5.93), ("w2222", 65536, 12.78, 11.80),
    ("w22222222", 4096, 2.67, 3.02), ("w22222222", 8192, 3.39, 3.00), ("w22222222", 16384, 6.65, 5.98), ("w22222222", 32768, 12.96, 11.92), ("w22222222", 65536, 25.31, 23.53),
    ("w33333333", 2048, 3.41, 1.82), ("w33333333", 4096, 4.16, 3.05), ("w33333333", 8192, 8.22, 3.01), ("w33333333", 16384, 16.04, 5.97), ("w33333333", 32768, 31.21, 11.82), ("w33333333", 65536, 61.80, 23.51),
    ("f1", 1024, 3.00, 2.92), ("f1", 8192, 2.91, 3.04), ("f1", 16384, 2.90, 3.06), ("f1", 32768, 3.90, 4.84), ("f1", 65536, 7.44, 4.65),
    ("f1111", 8192, 3.06, 4.99), ("f1111", 16384, 4.03, 4.92), ("f1111", 32768, 7.91, 9.92), ("f1111", 65536, 15.36, 19.57),
    ("f11111111", 4096, 3.63, 5.32), ("f11111111", 8192, 4.63, 5.17), ("f11111111", 16384, 9.08, 10.34), ("f11111111", 32768, 17.73, 20.46), ("f11111111", 65536, 34.31, 40.71),
    ("f222222", 4096, 3.57, 4.95), ("f222222", 8192, 4.70, 4.87), ("f222222", 16384, 9.28, 9.57), ("f222222", 32768, 17.87, 19.22), ("f222222", 65536, 34.93, 38.23),
    ("f33333333", 2048, 4.34, 3.45), ("f33333333", 4096, 5.70, 5.03), ("f33333333", 8192, 11.09, 4.94), ("f33333333", 16384, 21.68, 9.88), ("f33333333", 32768, 42.08, 19.71), ("f33333333", 65536, 83.41, 39.14),
    ("f6666", 4096, 8.60, 4.73), ("f6666", 8192, 16.73, 8.75), ("f6666", 16384, 32.41, 8.56), ("f6666", 32768, 63.69, 17.39), ("f6666", 65536, 125.89, 34.18),
    ("f61111111", 4096, 6.97, 9.51), ("f61111111", 8192, 9.31, 9.23), ("f61111111", 16384, 18.06, 18.61), ("f61111111", 32768, 34.69, 37.18), ("f61111111", 65536, 68.18, 73.83),
    ("fork_8x1", 8192, 3.32, 4.89), ("fork_8x1", 16384, 4.03, 4.71), ("fork_8x1", 32768, 8.02, 9.61), ("fork_8x1", 65536, 15.54, 18.93),
    ("quadruped", 4096, 3.60, 3.16), ("quadruped", 8192, 5.78, 5.13), ("quadruped", 16384, 10.98, 4.94), ("quadruped", 32768, 21.44, 9.84), ("quadruped", 65536, 42.15, 19.73),
    ("hexapod", 2048, 4.28, 3.54), ("hexapod", 4096, 5.90, 5.20), ("hexapod", 8192, 11.43, 5.00), ("hexapod", 16384, 22.28, 10.17), ("hexapod", 32768, 43.07, 20.18), ("hexapod", 65536, 85.34, 40.51),
    ("humanoid", 4096, 10.75, 6.57), ("humanoid", 8192, 21.09, 11.43), ("humanoid", 16384, 40.52, 11.22), ("humanoid", 32768, 79.16, 22.63), ("humanoid", 65536, 155.93, 45.06),
]


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    open(src, "w").write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(os.path.dirname(build.__file__), "csrc"), src, "-o", lib], check=True)
    fn = C.CDLL(lib).forms

    def run(descs, simds=SIMDS):
        f = np.array([[float(x[k]) for k in FIELDS] for x in descs]).ravel()
        out = (C.c_int * len(descs))()
        fn(len(descs), f.ctypes.data_as(C.POINTER(C.c_double)), simds, out)
        return list(out)

    return run


def _desc(tree, samples, steps=100, **over):
    fb, serial, shared, depth, path_len, path_lanes, key, kids, cmax, cpath = TREES[tree]
    return dict(dict(path=1, folds=1, floating=fb, serial=serial, shared=shared, depth=depth, path_len=path_len,
                     path_lanes=path_lanes, body_key=key, base_children=kids, contacts_max=cmax, contacts_path=cpath,
                     samples=samples, steps=steps, quad_lds=16000, lane_lds=30000, body_lds=16000), **over)


def test_one_instance_takes_the_faster_kernel(choose):
    """Within 5 % of the better of the two measured times (trees of one level at any
    size are that close), whatever the size of the launch."""
    for tree, n, body, path in MEASURED:
        took = body if choose([_desc(tree, n)])[0] == BODY else path
        assert took <= 1.05 * min(body, path), (tree, n, body, path)


def test_a_batch_of_wide_shallow_trees_takes_the_body_kernel(choose):
    for tree in ("w11111111", "f1111", "f222222"):
        assert set(choose([_desc(tree, 512 + 7 * i, 40 + 11 * (i % 4)) for i in range(32)])) == {BODY}, tree
    # beside robots that the path kernel serves better
    mix = [_desc(t, 1024 + 7 * i, 50) for i, t in enumerate(("w11111111", "quadruped", "humanoid", "f1111") * 16)]
    got = choose(mix)
    assert set(got[0::4]) == {BODY} and set(got[3::4]) == {BODY}
    assert BODY not in got[1::4] + got[2::4]


def test_batches_that_fit_at_once_take_the_quad_form(choose):
    got = choose([_desc(t, 64, 50) for t in TREES])
    assert set(got) == {QUAD}


def test_what_the_path_kernel_does_not_take(choose):
    assert choose([_desc("quadruped", 4096, path=0)]) == [BODY]
    assert choose([_desc("quadruped", 4096, path=0), _desc("quadruped", 4096)]) == [BODY, QUAD]
    # no room for the one-lane form's knots; numberings that only the slow body kernels take
    assert choose([_desc("quadruped", 8192, lane_lds=70000)]) != [LANE]
    assert choose([_desc("w11111111", 32768, folds=0)]) == [LANE]
    # three blocks of 50 000 bytes to a compute unit: two turns past 768 wavefronts
    assert choose([_desc("hexapod", 1500, quad_lds=50000, body_lds=50000)]) == [QUAD]
    assert choose([_desc("hexapod", 2000, quad_lds=50000, lane_lds=30000, body_lds=60000)]) == [LANE]


def _plain_split(descs):
    """The split of choose_forms by trying every prefix of the longest rollouts."""
    waves = lambda d, lane: -(-d["samples"] // ((256 if lane else 64) // d["path_lanes"]))  # noqa: E731
    weight = lambda d: (0.65 * d["path_len"] + 1.3 * d["floating"] + 0.4 * d["contacts_path"]) * d["steps"]  # noqa: E731
    if sum(waves(d, False) for d in descs) <= SIMDS:
        return [QUAD] * len(descs)
    order = sorted(range(len(descs)), key=lambda i: -weight(descs[i]))
    best, took = None, None
    for k in range(len(descs), -1, -1):
        form = [QUAD] * len(descs)
        for i in order[k:]:
            if descs[i]["lane_lds"] <= 40 * 1024:
                form[i] = LANE
        t = [weight(d) * (1.65 if f == LANE else 1) for d, f in zip(descs, form)]
        longest = max(t)
        spread = sum(x * waves(d, f == LANE) for x, d, f in zip(t, descs, form)) / SIMDS
        est = max(longest, spread) + 0.2 * min(longest, spread)
        if best is None or est < best * (1 - 1e-12):
            best, took = est, form
    return took


def test_linear_split_equals_the_plain_search(choose):
    rng = random.Random(5)
    seen = set()
    for _ in range(300):
        descs = [_desc(rng.choice(list(TREES)), rng.randint(16, 2048), rng.randint(20, 400), folds=0,
                       lane_lds=rng.choice((30000, 50000))) for _ in range(rng.randint(2, 48))]
        got = choose(descs)
        assert got == _plain_split(descs)
        seen.add(frozenset(got))
    assert {frozenset((QUAD,)), frozenset((LANE, QUAD))} <= seen
