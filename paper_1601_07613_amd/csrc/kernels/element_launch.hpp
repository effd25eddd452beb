// Launches of the one-pass element stage (element.hpp), compiled in a file of
// their own.
#pragma once

#include <hip/hip_runtime.h>

#include "../batch_desc.hpp"
#include "../host/internal.hpp"

namespace dgc {

// whether the element pass can run this mesh: it needs the element -> face
// slots, at most as many per element as the kernels hold, and in f32 a mesh
// whose colored step it reproduces in rounding
bool element_stage_ok(const dgc_dmesh *dm, int32_t precision);

// whether a mesh is too scattered for the element pass to be the faster one
bool element_stage_scattered(const dgc_dmesh *dm);

// one SSP-RK3 stage out = a x + b (y + dt rhs(y)) (x null: x = y, with a = 0)
dgc_status launch_element_stage(const dgc_dmesh *dm, const dgc_table_info &ti, int32_t precision, const double *y,
                                const double *x, double *out, double a, double b, double dt, hipStream_t st);

// elements per work-group (the unit of a batch's block map)
int element_stage_elems(int dim);

// stage `stage` of every mesh of a batch whose header has elem_slots > 0
dgc_status launch_element_stage_batched(const dgc_batch::Header &h, const char *dev, int stage, hipStream_t st);

}  // namespace dgc
