// How a first product of up to sixteen sequences counts its tasks (index arithmetic only, for host and device alike).
#pragma once

namespace parse {

constexpr int DEC_MAX_LAYERS = 4;

// The workgroups of a call whose workgroups take several tasks, shared out among its layers by the tasks that these have at most: wgs[l] of the layer's own,
// which take its tasks 0, 1, ..., then each its wgs[l]-th next one.  A workgroup stays with its layer, so its first place past the layer's tasks in use is its last,
// however much the layers differ.  (With layers taking turns, id % layers, and a number of workgroups that is no multiple of the layers' a workgroup goes from layer to
// layer, and ends where the shortest one does.)
// Shares by size: q/k/v of 2048 / 512 / 512 ranks, 4096 columns, four and twelve sequences 15.5 and 16.2 us a call, equal shares 16.8 and 17.7.  Tasks numbered
// over all layers by the groups in use are shared out better but known only once every layer's plan is there: 16.3 and 17.2, and three layers of 1536 ranks 19.3, 18.4
// this way.
__host__ __device__ inline int dec_share(const int *tasks, int n_layers, int units, int (&wgs)[DEC_MAX_LAYERS]) {
  long long all = 0;
  int most = 0, sum = 0;
  for (int l = 0; l < n_layers; ++l) {
    all += tasks[l];
    if (tasks[l] > tasks[most]) most = l;
  }
  for (int l = 0; l < n_layers; ++l) {
    wgs[l] = all <= units ? tasks[l] : (int)((long long)tasks[l] * units / all);
    if (wgs[l] < 1) wgs[l] = 1;
    sum += wgs[l];
  }
  if (all > units && wgs[most] + units - sum >= 1) {           // what rounding left over or took too much
    wgs[most] += units - sum;
    sum = units;
  }
  return sum;
}

// which group in use holds a layer's task `at`, `per` tasks to a group.  Exact: at / per < 64, and (at + 1/2) / per is at least 1/4096 off every integer
__host__ __device__ inline int dec_group_of(int at, int per) { return (int)(((float)at + 0.5f) * (1.0f / (float)per)); }

}  // namespace parse
