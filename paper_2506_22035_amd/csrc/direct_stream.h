// Internal launch interface of the direct engine's register-streaming kernel.
#pragma once
#include <hip/hip_runtime.h>

namespace spider_impl {

// T steps (1, 2, 4 or 8, up to direct2d_stream_max_steps) of a 2-D grid in one launch
// (radius 1 to 3; dtype and zero_taps as for launch_direct), `seg_h` rows per wave.
hipError_t launch_direct2d_stream(int r, int dtype, int zero_taps, int T, const void* in, void* out, int ny, int nx,
                                  const void* coeffs_dev, int seg_h, hipStream_t s);
// Deepest launch on a grid of this many points: 0 where there is no such kernel
// (radius above 3, or zero taps that are skipped at run time).
int direct2d_stream_max_steps(int r, int dtype, int zero_taps, long long points);
// Rows per wave of a launch of T steps.
int direct2d_stream_rows(int r, int T, int ny, int nx, int ncu);

}  // namespace spider_impl
