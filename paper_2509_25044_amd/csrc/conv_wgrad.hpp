// Weight and bias gradient of the convolutions (host side of conv3d_wgrad.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace ffdp {

struct ConvWgradPlan {
    int nx, ny, nz, zlen;   // columns of 32 output voxels x a few rows, cut along z every zlen slices
    long long units, upc;   // columns in all, and per chunk
    int nchunks;
    long long part_floats;  // workspace floats: weight partials, then bias partials, per chunk
};
ConvWgradPlan conv_wgrad_plan(const ConvGeom& g);

// P = dL/dy act'(y) in bf16 (pbf), or pbf NULL: formed from dy and y (y NULL:
// no activation), bitwise the same gradients; part: part_floats floats
hipError_t conv_wgrad_launch(const ConvGeom& g, const unsigned short* xa, const unsigned short* xb, const float* dy,
                             const unsigned short* y, float slope, const unsigned short* pbf, float* dw, float* db,
                             float* part, hipStream_t st);

}  // namespace ffdp
