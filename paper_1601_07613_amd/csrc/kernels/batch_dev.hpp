// Access to a batch descriptor on the device.
#pragma once

#include <hip/hip_runtime.h>

#include "../batch_desc.hpp"

namespace dgc_dev {

using dgc_batch::Entry;
using dgc_batch::Header;

__device__ __forceinline__ const Header *bh(const char *desc) { return reinterpret_cast<const Header *>(desc); }

__device__ __forceinline__ const Entry *bentry(const char *desc, int32_t m) {
    return reinterpret_cast<const Entry *>(desc + bh(desc)->off_entries) + m;
}

// Pointers read from the descriptor are generic pointers to the compiler.
// They all point to device global memory; casting them through the global
// address space lets it emit global (not flat) loads and stores, whose
// completion counter does not hold back LDS and scalar loads.
// (Through an integer: a direct cast pair is folded away before the
// address-space inference runs.)
template <class T>
__device__ __forceinline__ T *gptr(T *p) {
    return (T *)((__attribute__((address_space(1))) T *)(uintptr_t)p);
}

// the device arrays of one member, as global pointers
struct Member {
    const int32_t *face_lr;
    const uint8_t *face_code;
    const double *face_geo, *elem_geo;
    double *U;
    dgc_batch::RkWs w;
};

__device__ __forceinline__ Member member(const Entry *e, bool f32) {
    return Member{gptr(e->face_lr), gptr(e->face_code), gptr(e->face_geo), gptr(e->elem_geo), gptr(e->U),
                  dgc_batch::rk_ws(gptr(e->ws), (size_t)e->n_dof, f32)};
}

}  // namespace dgc_dev
