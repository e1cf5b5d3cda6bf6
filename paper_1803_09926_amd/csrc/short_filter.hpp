// The filter gradient of short launches in one kernel (short_filter.hip).
#pragma once
#include "gconv.hpp"

namespace dwc {

// The way that a shape takes otherwise: two launches, the NCHW small-plane kernels and a second launch, one launch of the generic kernels, or the 16x16 matrix
// instructions and a second launch.
enum FilterWay { FILTER_TWO, FILTER_SMALL_PLANES, FILTER_GENERIC_ONE, FILTER_MATRIX };

// Whether the kernel takes the shape and is the shorter way; depthwise: G = C, Cg = 1, Og = the multiplier.
bool short_bwd_filter_shorter(const GGeom &g, int layout, int dtype, FilterWay way);
hipError_t short_bwd_filter(const GGeom &g, int layout, int dtype, const void *x, const void *dy, float *dw, hipStream_t st);

}  // namespace dwc
