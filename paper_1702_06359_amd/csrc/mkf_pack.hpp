// Host packing of inputs (mkf_pack.cpp).
#pragma once

#include <stddef.h>

namespace mkf {

// What the kernels read of a hit, four floats: (cos, sin, z, r) on a cylinder,
// (cos, sin, r, z) on a disk, (x, y, z, 0) on layers of finite thickness and
// for the 3x3 measurement.
enum class HitForm { kCylinder, kDisk, kXyz };

// Each returns whether every value was fit for use; the output is written
// either way.
bool pack_hits(const double *h, size_t n, HitForm form, float *out);   // finite in FP32, off the axis
bool narrow_all(const double *src, float *dst, size_t n);              // finite in FP32
bool states_in_range(const double *par, size_t n);                     // theta in (0, pi), off the axis

}  // namespace mkf
