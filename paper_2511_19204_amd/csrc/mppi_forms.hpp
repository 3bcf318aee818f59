// mppi_forms.hpp -- which kernel form each instance of a launch runs in (host
// code without HIP, so that the rule can be tested by itself).
//
// An instance of the body schedule at its default lane count has up to three
// forms with the same results: its own body kernel (one lane per body), and the
// path kernel with a quad of lanes or one lane per root-to-leaf path.  A SIMD
// holds two wavefronts of the body kernel, one of the path kernel.  The quad
// form's step is the shortest of most trees; the one-lane form's takes 1.6 to
// 1.85 times as long and needs a quarter of the wavefronts; the body kernel
// sweeps a tree of one or two levels faster than the path kernel, which walks
// every path as if it had three bodies, and holds more rollouts per wavefront
// where a tree has many short paths.
#pragma once
#include <algorithm>
#include <cmath>
#include <map>
#include <utility>
#include <vector>

namespace mppi {

constexpr int kPathLds = 64 * 1024;  // LDS a block of the path kernel may take
constexpr int kCuLds = 160 * 1024;   // of a compute unit

enum Form { kFormBody = 0, kFormQuad = 1, kFormLane = 2 };

// What the choice looks at: the tree, the size of the launch, LDS bytes of a block.
struct FormDesc {
  bool path = false;    // the path kernel takes it
  bool folds = true;    // the depth-specialised body kernels take it
  bool floating = false, serial = false;  // serial: a fixed-base chain
  bool shared = false;  // several paths share a body
  int depth = 1;        // levels of the tree below the base
  int path_len = 3;     // bodies per path of the path kernel's variant (3, 4 or 6)
  int path_lanes = 4;   // lanes per rollout of the quad form (4 per path)
  int body_key = 4;     // lanes per rollout of the body kernel
  int base_children = 0;
  int contacts_max = 0, contacts_path = 0;  // of a body; summed over a path's indices (the most of each)
  int samples = 1;
  double steps = 1;     // physics steps of a rollout
  int quad_lds = 0, lane_lds = 0, body_lds = 0;
};

// Microseconds of a physics step, fitted to 45 trees on the MI355X (within 10 % of
// each): the wavefront alone on its SIMD, and for the body kernel two of them.
struct StepTime {
  double quad, lane, body, body2;
};
inline StepTime step_time(const FormDesc& d) {
  const double wide = d.floating && d.path_lanes > 16 ? 1 : 0, fb = d.floating, sh = d.shared;
  StepTime t;
  t.quad = 0.6 * d.path_len + 0.8 * fb + 0.3 * d.contacts_path + 0.45 * wide + 0.35 * sh;
  t.lane = 1.29 * d.path_len - 0.85 + 1.25 * fb + 0.45 * d.contacts_path + 0.35 * wide + 0.55 * sh;
  const double more = 0.14 * std::max(0, d.base_children - 4) + 0.55 * d.contacts_max + 0.5 * sh;
  if (d.depth <= 3) {  // (the body kernels' two specialisations)
    const double chain = d.serial ? 0.5 : 0;
    t.body = 1.6 + 0.5 * d.depth - chain + 0.2 * fb + more;
    t.body2 = 2.0 + 0.7 * d.depth - chain + 0.5 * fb + more;
  } else {
    t.body = 1.7 + 0.65 * d.depth + 0.2 * fb + more;
    t.body2 = 2.65 + 0.78 * d.depth + 0.5 * fb + more;
  }
  return t;
}

// blocks of `lds` bytes a SIMD holds (at most `most`), in quarters of a compute unit
inline double resident(int lds, int most) {
  return std::min<double>(most, lds > 0 ? 0.25 * (kCuLds / lds) : most);
}

// A form has to be estimated this much shorter to take an instance off the path
// kernel (the estimates' own error).
constexpr double kBodyGain = 0.97;

// One instance alone: whole turns of the SIMDs.  Measured (quadruped, 60 steps):
// 4 096 samples 0.25 ms in the quad form, 0.35 one-lane, 0.28 body; 6 144: 0.44 /
// 0.37 / 0.41; 16 384: 0.84 / 0.39 / 0.76.  Four one-joint legs, 40 to 120 steps, us a
// step at 8 192 samples: 5.0 one-lane, 3.1 body; a planar two-link arm at 16 384:
// 1.85 quad, 2.1 body; eight one-joint arms at 32 768: 11.9 one-lane, 5.3 body.
inline Form choose_form(const FormDesc& d, int simds) {
  if (!d.path) return kFormBody;
  const StepTime t = step_time(d);
  const int per_quad = 64 / d.path_lanes, per_lane = 256 / d.path_lanes, per_body = 64 / d.body_key;
  auto turns = [](int n, int per, double slots) { return std::ceil(std::ceil((double)n / per) / slots); };
  const double quad_slots = simds * resident(d.quad_lds, 1), filled = std::min(1.0, d.samples / (per_quad * quad_slots));
  // (a quad-form step takes 5 to 8 % longer on a full device than on few SIMDs)
  const double quad = t.quad * (1 + 0.05 * filled) * turns(d.samples, per_quad, quad_slots);
  const double lane = d.lane_lds <= kPathLds ? t.lane * turns(d.samples, per_lane, simds * resident(d.lane_lds, 1)) : 1e300;
  double body = 1e300;
  if (d.folds) {
    const double waves = std::ceil((double)d.samples / per_body), slots = simds * resident(d.body_lds, 2);
    const double full = std::floor(waves / slots), rest = waves - full * slots;
    const double pair = slots > simds ? t.body2 : t.body;
    body = full * pair + (rest <= 0 ? 0 : rest <= simds ? t.body : t.body2);
  }
  if (body < kBodyGain * std::min(quad, lane)) return kFormBody;
  return lane < quad ? kFormLane : kFormQuad;
}

// Weight of an instance's rollouts in a launch of both forms of the path kernel (the
// split below, the order of the work): 0.65 a body, 1.3 the floating base and 0.4 a
// contact a step, the one-lane form's 1.65 of that.
constexpr double kLaneWeight = 1.65;
inline double quad_weight(const FormDesc& d) {
  return (0.65 * d.path_len + 1.3 * d.floating + 0.4 * d.contacts_path) * d.steps;
}

// The instances of one launch.  While all quad-form wavefronts are resident at once
// they are taken.  Past that a mixed launch of the path kernel keeps its longest
// rollouts in the quad form as far as that shortens it: it lasts about as long as
// its longest rollout or its work spread over the SIMDs, whichever is more, and a
// fifth of the other, by the weights above (64 served robots of three kinds 6.58 ms a
// round, a 32-robot mix of equal shares 1.46; by the fitted step times 6.36 and
// 1.60).  Instances whose work is less in the body kernel go there if
// a launch of their own beside the others' pays for itself (16 robots of eight one-joint
// arms, 512 samples, two iterations: 0.61 ms in the path kernel, 0.41 in the body
// kernel; 64 of them at 1 024: 3.3 and 1.6).
inline std::vector<Form> choose_forms(const std::vector<FormDesc>& list, int simds) {
  std::vector<Form> form(list.size(), kFormBody);
  if (list.size() == 1) {
    form[0] = choose_form(list[0], simds);
    return form;
  }
  struct Cand {
    int i;
    StepTime t;     // a rollout's
    double weight;  // quad_weight
    double quad_waves, lane_waves, body_waves;
    bool lane_ok, folds;
    int key;
    double path_work(bool lane) const { return lane && lane_ok ? t.lane * lane_waves : t.quad * quad_waves; }
    double path_time(bool lane) const { return lane && lane_ok ? t.lane : t.quad; }
  };
  std::vector<Cand> all;
  double waves = 0, slots = simds;
  for (int i = 0; i < (int)list.size(); ++i) {
    const FormDesc& d = list[i];
    if (!d.path) continue;
    Cand c;
    c.i = i;
    c.t = step_time(d);
    for (double* x : {&c.t.quad, &c.t.lane, &c.t.body, &c.t.body2}) *x *= d.steps;
    c.weight = quad_weight(d);
    auto count = [&](int per) { return (double)((d.samples + per - 1) / per); };
    c.quad_waves = count(64 / d.path_lanes);
    c.lane_waves = count(256 / d.path_lanes);
    c.body_waves = count(64 / d.body_key);
    c.lane_ok = d.lane_lds <= kCuLds / 4;  // four blocks of a mixed launch to a compute unit
    c.folds = d.folds;
    c.key = d.body_key;
    all.push_back(c);
    form[i] = kFormQuad;
    waves += c.quad_waves;
    slots = std::min(slots, simds * resident(d.quad_lds, 1));
  }
  if (all.empty() || waves <= slots) return form;
  std::stable_sort(all.begin(), all.end(), [](const Cand& a, const Cand& b) { return a.weight > b.weight; });
  auto span = [&](double longest, double work, double on) {
    return std::max(longest, work / on) + 0.2 * std::min(longest, work / on);
  };
  // how many of c, from its start, take the quad form
  auto split = [&](const std::vector<Cand>& c) {
    const int n = (int)c.size();
    double work = 0, tail = 0, best = 1e300;  // tail: the longest of the others
    int best_k = n;
    for (const Cand& x : c) work += x.weight * x.quad_waves;
    for (int k = n; k >= 0; --k) {
      if (k < n) {
        const double w = c[k].lane_ok ? kLaneWeight * c[k].weight : c[k].weight;
        work += w * (c[k].lane_ok ? c[k].lane_waves : c[k].quad_waves) - c[k].weight * c[k].quad_waves;
        tail = std::max(tail, w);
      }
      const double est = span(std::max(tail, k > 0 ? c[0].weight : 0.0), work, simds);
      if (est < best) {
        best = est;
        best_k = k;
      }
    }
    return best_k;
  };
  auto estimate = [&](const std::vector<Cand>& c, int k) {
    double longest = 0, work = 0;
    for (int j = 0; j < (int)c.size(); ++j) {
      longest = std::max(longest, c[j].path_time(j >= k));
      work += c[j].path_work(j >= k);
    }
    return span(longest, work, slots);
  };
  std::vector<Cand> stay;                        // in the path kernel where the others leave it
  std::map<int, std::pair<double, double>> own;  // the others by body kernel: longest rollout, work
  for (const Cand& x : all) {
    const double body = 0.5 * x.t.body2 * x.body_waves;
    if (x.folds && body < kBodyGain * std::min(x.path_work(false), x.path_work(true))) {
      auto& o = own[x.key];
      o.first = std::max(o.first, x.t.body);
      o.second += body;
    } else {
      stay.push_back(x);
    }
  }
  int k = split(all);
  if (!own.empty()) {
    const int ks = split(stay);
    double est = estimate(stay, ks);
    for (const auto& o : own) est += span(o.second.first, o.second.second, simds);
    if (est < kBodyGain * estimate(all, k)) {
      for (const Cand& x : all) form[x.i] = kFormBody;
      for (const Cand& x : stay) form[x.i] = kFormQuad;
      all = stay;
      k = ks;
    }
  }
  for (int j = k; j < (int)all.size(); ++j)
    if (all[j].lane_ok) form[all[j].i] = kFormLane;
  return form;
}

}  // namespace mppi
