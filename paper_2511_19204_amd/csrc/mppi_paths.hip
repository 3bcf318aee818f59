// mppi_paths.hip -- gfx950 rollout kernel that takes the tree by its root-to-leaf
// paths, in two forms: a quad of lanes per path (mppi_path.hpp) or one lane per
// path (mppi_lane.hpp).
#include "mppi_path.hpp"
#include "mppi_lane.hpp"

namespace mppi {

// Block = one wavefront, one work item:
//  * work[blockIdx] = (instance, first sample, with kLaneItem where the one-lane
//    form runs it), or, when work is null, instance 0 in the form `lane_form` and
//    its blockIdx-th block of samples; x0_in / nominal_in as in rollout_kernel;
//  * with preds (one item per block) or pred_out (instance 0): a state prediction
//    over the item's steps, as predict_kernel.
// One launch takes trees of every kind in either form, so the rollouts of a mixed
// batch run side by side; the LDS layout is each item's own.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1))) void path_kernel(
    const DevInst* __restrict__ insts, const int2* __restrict__ work, int lane_form, const float* __restrict__ x0_in,
    const float* __restrict__ nominal_in, const PredItem* __restrict__ preds, float* __restrict__ pred_out,
    int pred_steps) {
  extern __shared__ float smem[];
  const DevInst* I = insts;
  int first = 0, steps = pred_steps;
  bool lane = false;
  float* out = pred_out;
  if (preds) {
    const PredItem it = preds[blockIdx.x];
    I = it.inst;
    steps = it.steps;
    out = it.state_out;
  } else if (!pred_out) {
    if (work) {
      const int2 w = work[blockIdx.x];
      I = insts + w.x;
      lane = (w.y & kLaneItem) != 0;
      first = w.y & ~kLaneItem;
    } else {
      lane = lane_form != 0;
      first = (int)blockIdx.x * ((lane ? 256 : 64) / I->model->path_lanes);
    }
    steps = I->H;
  }
  const bool fb = I->model->fb;
  if (lane) {
    if (fb) lane_item_of<true>(*I, first, smem, x0_in, nominal_in);
    else lane_item_of<false>(*I, first, smem, x0_in, nominal_in);
  } else {
    if (fb) path_item_of<true>(*I, first, smem, steps, out, x0_in, nominal_in);
    else path_item_of<false>(*I, first, smem, steps, out, x0_in, nominal_in);
  }
}

}  // namespace mppi
