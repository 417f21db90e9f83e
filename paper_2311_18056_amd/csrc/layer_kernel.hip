// Launch plans of the persistent layer kernel (device code in layer_impl.h).
#include "layer_kernel.h"

#include <algorithm>

#include "device_common.h"

namespace rqp {

const void* layer_fn_f32(int nc, bool more);
const void* layer_fn_f32x(int nc, bool more);
const void* layer_fn_f64(int nc, bool more);
const void* layer_fn_f64x(int nc, bool more);

template <typename T>
LaunchPlan plan_layer(int n, int m, int grid, bool xt) {
  LaunchPlan p{};
  const int L = n + m;
  if (L < 1 || L > kMaxLayerRows || grid < 1) return p;
  const int cs = layer_col_lanes<T>(L), nc = (L + cs - 1) / cs;
  const int rows = (L + grid - 1) / grid;
  const bool more = layer_takes_more<T>(nc, rows, xt);
  const int reg = more ? layer_more_rows<T>(nc, xt) : layer_reg_rows<T>(nc);
  const void* fn = sizeof(T) == sizeof(double) ? (xt ? layer_fn_f64x(nc, more) : layer_fn_f64(nc, more))
                                               : (xt ? layer_fn_f32x(nc, more) : layer_fn_f32(nc, more));
  int dev = 0, smem_max = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return p;
  if (hipDeviceGetAttribute(&smem_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return p;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return p;
  hipFuncAttributes fa{};
  if (hipFuncGetAttributes(&fa, fn) != hipSuccess) return p;
  // dynamic LDS: the check vector (whole units of the check), then as many of the rows that do not
  // fit in registers as there is room for, then rows of the check matrix
  const long es = sizeof(T), ldw = (L + 3) / 4 * 4, row_bytes = ldw * es;
  const long stage = (L + 255) / 256 * 256;
  const long room = ((long)smem_max - (long)fa.sharedSizeBytes) / 16 * 16 - stage * es;
  if (room < 0) return p;
  p.lds_rows = (int)std::min<long>(std::max(rows - reg, 0), room / row_bytes);
  p.on_chip = reg + (int)(room / row_bytes);
  // the check rows a workgroup has at most, in whole kilobytes (the copy's unit)
  long most = 0;
  int prev = 0;
  double best = 0.0;
  for (int g = 0; g < grid; ++g) {
    best = std::max(best, split_term(g + 1, grid, n, m, L));
    const int next = split_row(best, n, L), rb = L / grid, re = L % grid;
    const int r0 = g * rb + std::min(g, re), r1 = r0 + rb + (g < re ? 1 : 0);
    const long np = r1 > n ? r1 - std::max(r0, n) : 0;
    most = std::max(most, (next - prev) * row_bytes + np * ((n + 3) / 4 * 4) * es);
    prev = next;
  }
  const long rest = room - p.lds_rows * row_bytes;
  p.cache_bytes = (int)(std::min(rest, (most + 1023) / 1024 * 1024) / 1024 * 1024);
  p.check_cols = (int)stage;
  p.col_lanes = cs;
  p.dyn_bytes = (size_t)(stage * es + p.lds_rows * row_bytes + p.cache_bytes);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)((long)smem_max - (long)fa.sharedSizeBytes)) != hipSuccess)
    return p;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kLayerBlock, p.dyn_bytes) != hipSuccess) return p;
  p.max_grid = per_cu * cus;
  p.fn = fn;
  return p;
}

template <typename T>
hipError_t launch_layer(const LayerArgs& a, const LaunchPlan& p, int grid, hipStream_t st) {
  if (!p.fn) return hipErrorInvalidValue;
  LayerArgs copy = a;
  copy.lds_rows = p.lds_rows;
  copy.check_cols = p.check_cols;
  copy.cache_bytes = p.cache_bytes;
  copy.col_lanes = p.col_lanes;
  void* args[] = {&copy};
  return hipLaunchCooperativeKernel(p.fn, dim3(grid), dim3(kLayerBlock), args, p.dyn_bytes, st);
}

template LaunchPlan plan_layer<float>(int, int, int, bool);
template LaunchPlan plan_layer<double>(int, int, int, bool);
template hipError_t launch_layer<float>(const LayerArgs&, const LaunchPlan&, int, hipStream_t);
template hipError_t launch_layer<double>(const LayerArgs&, const LaunchPlan&, int, hipStream_t);

}  // namespace rqp
