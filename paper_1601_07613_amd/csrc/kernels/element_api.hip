// Launches of the one-pass element stage.
#include <hip/hip_runtime.h>

#include <string>

#include "element.hpp"
#include "element_launch.hpp"

namespace dgc {

namespace {

// run f with the kernels' shape for an element type, order and number of face
// slots (f's argument names the template parameters)
template <int DIM, int NP, int Q, int QV, int FS, bool MIXED>
struct Shape {
    static constexpr int kDim = DIM, kNp = NP, kQ = Q, kQv = QV, kFs = FS;
    static constexpr bool kMixed = MIXED;
};
template <class F>
dgc_status dispatch(int elem_type, int p, int max_slots, F &&f) {
#define DGC_ELEM(P, DIM, NP, Q, QV, FS, MIXED) \
    case P: return f(Shape<DIM, NP, Q, QV, FS, MIXED>{});
    if (elem_type == DGC_TRI && max_slots <= 3) {
        switch (p) {
            DGC_ELEM(0, 2, 1, 1, 1, 3, false)
            DGC_ELEM(1, 2, 3, 2, 4, 3, false)
            DGC_ELEM(2, 2, 6, 3, 9, 3, false)
            DGC_ELEM(3, 2, 10, 4, 16, 3, false)
            DGC_ELEM(4, 2, 15, 5, 25, 3, false)
            DGC_ELEM(5, 2, 21, 6, 36, 3, false)
        }
    } else if (elem_type == DGC_TRI) {
        switch (p) {
            DGC_ELEM(0, 2, 1, 1, 1, 6, false)
            DGC_ELEM(1, 2, 3, 2, 4, 6, false)
            DGC_ELEM(2, 2, 6, 3, 9, 6, false)
            DGC_ELEM(3, 2, 10, 4, 16, 6, false)
            DGC_ELEM(4, 2, 15, 5, 25, 6, false)
            DGC_ELEM(5, 2, 21, 6, 36, 6, false)
        }
    } else if (elem_type == DGC_QUAD) {
        switch (p) {
            DGC_ELEM(0, 2, 1, 1, 1, 4, false)
            DGC_ELEM(1, 2, 4, 2, 4, 4, false)
            DGC_ELEM(2, 2, 9, 3, 9, 4, false)
            DGC_ELEM(3, 2, 16, 4, 16, 4, false)
        }
    } else if (elem_type == DGC_MIXED) {
        switch (p) {
            DGC_ELEM(0, 2, 1, 1, 1, 4, true)
            DGC_ELEM(1, 2, 4, 2, 4, 4, true)
            DGC_ELEM(2, 2, 9, 3, 9, 4, true)
            DGC_ELEM(3, 2, 16, 4, 16, 4, true)
        }
    } else if (elem_type == DGC_TET) {
        switch (p) {
            DGC_ELEM(0, 3, 1, 3, 1, 4, false)
            DGC_ELEM(1, 3, 4, 3, 8, 4, false)
            DGC_ELEM(2, 3, 10, 9, 27, 4, false)
        }
    }
#undef DGC_ELEM
    return fail(DGC_E_UNSUPPORTED, "no element stage built for this element type and order");
}

dgc_status launched(const char *what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DGC_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
    return DGC_OK;
}

template <class S, class T>
using Cfg = dgc_dev::ElemCfg<S::kDim, S::kNp, S::kQ, S::kQv, S::kFs, S::kMixed, T>;

template <class S, class T>
constexpr bool built() {
    return sizeof(T) == 8 || dgc_dev::f32_element_shape(S::kDim, S::kNp, S::kFs, S::kMixed);
}

template <class T>
dgc_status launch(const dgc_dmesh *dm, const dgc_dev::ElemStageArgs &A, const dgc_dev::ElemTables &tab,
                  hipStream_t st) {
    return dispatch(dm->elem_type, dm->p, dm->max_slots, [&](auto shape) {
        using S = decltype(shape);
        if constexpr (!built<S, T>()) {
            return fail(DGC_E_UNSUPPORTED, "no f32 element stage built for this element type and order");
        } else {
            using C = Cfg<S, T>;
            hipLaunchKernelGGL((dgc_dev::element_stage_kernel<S::kDim, S::kNp, S::kQ, S::kQv, S::kFs, S::kMixed, T>),
                               dim3((unsigned)((A.n_elem + C::EPB - 1) / C::EPB)), dim3(C::BLOCK),
                               C::lds_bytes(tab.n_codes), st, A, tab, dm->max_slots);
            return launched("element stage launch");
        }
    });
}

template <class T>
dgc_status launch_batch(const dgc_batch::Header &h, const char *dev, int stage, hipStream_t st) {
    return dispatch(h.elem_type, h.p, h.elem_slots, [&](auto shape) {
        using S = decltype(shape);
        if constexpr (S::kMixed) {
            return fail(DGC_E_UNSUPPORTED, "mixed meshes are not batched");
        } else if constexpr (!built<S, T>()) {
            return fail(DGC_E_UNSUPPORTED, "no f32 element stage built for this element type and order");
        } else {
            using C = Cfg<S, T>;
            hipLaunchKernelGGL((dgc_dev::batch_element_stage_kernel<S::kDim, S::kNp, S::kQ, S::kQv, S::kFs, false, T>),
                               dim3(h.nblk_stage), dim3(C::BLOCK), C::lds_bytes(h.n_codes), st, dev, stage);
            return launched("batched element stage launch");
        }
    });
}

}  // namespace

bool element_stage_ok(const dgc_dmesh *dm, int32_t precision) {
    const int most = dm->elem_type == DGC_TRI ? 6 : 4;
    if (!dm->elem_slots || dm->max_slots <= 0 || dm->max_slots > most) return false;
    // f64, ordered numberings: faster at every type and order built, from a few
    // hundred to a million elements.  us a step, colored / element pass, smallest
    // and largest mesh measured:
    //   triangles, 512 and 980,000: p = 0 30 / 13, 222 / 170; p = 1 36 / 16, 545 /
    //     372; p = 2 48 / 27, 1,067 / 610; p = 3 84 / 38, 2,068 / 1,062; p = 4 131 /
    //     66, 4,130 / 1,996; p = 5 215 / 96, 6,869 / 3,829
    //   refined, 2,738 and 944,220: p = 0 81 / 16, 402 / 235 to p = 5 365 / 135,
    //     6,967 / 3,942
    //   parallelograms, 256 and 589,824: p = 0 42 / 13, 190 / 124; p = 1 47 / 19,
    //     489 / 262; p = 2 77 / 38, 1,473 / 606; p = 3 159 / 55, 3,262 / 1,244
    //   mixed, 308 and 191,420: p = 0 62 / 13, 132 / 52 to p = 3 191 / 88, 1,137 / 728
    //   tetrahedra, 384 and 511,104: p = 0 54 / 20, 506 / 309; p = 1 63 / 32, 670 /
    //     505; p = 2 228 / 93, 3,611 / 2,170
    // Numberings without order: element_stage_scattered.
    if (precision == DGC_F64) return true;
    // the f32 form keeps the rounding of the colored kernels (slot order =
    // color order); uniform meshes also need a face of each color per element,
    // as the colored step that carries the volume term does.  us a step as
    // above: triangles p = 0 48 / 14, 238 / 133; p = 3 82 / 40, 1,745 / 1,017;
    // parallelograms p = 3 120 / 69, 1,967 / 1,497; mixed p = 3 117 / 75, 673 / 579
    const bool mixed = dm->elem_type == DGC_MIXED;
    const int faces = dm->elem_type == DGC_TRI ? 3 : 4;
    return (mixed || (dm->max_slots == faces && dm->n_colors == faces)) &&
           dgc_dev::f32_element_shape(dm->elem_type == DGC_TET ? 3 : 2, dm->n_p, faces, mixed);
}

bool element_stage_scattered(const dgc_dmesh *dm) {
    // Where the numbering has no order, every face value, code and neighbour id
    // that an element gathers is a line of its own, about eight a side; a
    // colored launch reads them in face order.  That outweighs the right-hand
    // side's traffic for the shortest records, once the arrays leave the
    // caches.  us a step, colored / element pass, f64, random numbering:
    //   p = 0, the paper's layout (far_percent 64-74): 389k faces of triangles
    //     108 / 110, 480k 124 / 139, 1.47M 318 / 503; 442k of parallelograms
    //     134 / 134, 520k 149 / 164; 594k of a mixed mesh 205 / 195 (f32 184 /
    //     193), 791k 248 / 267; no renumbering (96-99): 389k 129 / 147
    //   p = 1, no renumbering: 480k faces of triangles 242 / 248 (f32 254 /
    //     241), 608k 305 / 319 (309 / 314), 1.47M 752 / 835; 720k of
    //     parallelograms 327 / 351
    //   p = 1, the paper's layout: 1.47M of triangles 656 / 648; 720k of
    //     parallelograms 299 / 311 (f32 300 / 297), 1.18M 504 / 531, 2M 856 / 935
    // Mixed meshes at p = 1, p >= 2 and tetrahedra are faster in one pass.
    const int64_t E = dm->n_face;
    const int far = dm->far_percent;
    if (dm->elem_type == DGC_TET) return false;
    if (dm->p == 0) return far >= 60 && E >= (dm->elem_type == DGC_MIXED ? 700000 : 450000);
    if (dm->p != 1 || dm->elem_type == DGC_MIXED) return false;
    return (far >= 85 && E >= 600000) || (dm->elem_type == DGC_QUAD && far >= 60 && E >= 1100000);
}

dgc_status launch_element_stage(const dgc_dmesh *dm, const dgc_table_info &ti, int32_t precision, const double *y,
                                const double *x, double *out, double a, double b, double dt, hipStream_t st) {
    const dgc_dev::ElemStageArgs A{dm->elem_slots, dm->face_lr, dm->face_code, dm->face_geo, dm->elem_geo,
                                   dm->elem_kind,  dm->n_elem,  dm->n_face,    y,            x,
                                   out,            nullptr,     a,             b,            dt};
    const dgc_dev::ElemTables tab{dm->tables + ti.off_trace, dm->tables + ti.off_proj, dm->tables + ti.off_vb,
                                  dm->tables + ti.off_vd, ti.n_codes};
    return precision == DGC_F32 ? launch<float>(dm, A, tab, st) : launch<double>(dm, A, tab, st);
}

int element_stage_elems(int dim) {
    return dim == 2 ? dgc_dev::ElemCfg<2, 6, 3, 9, 3, false, double>::EPB : dgc_dev::ElemCfg<3, 4, 3, 8, 4, false, double>::EPB;
}

dgc_status launch_element_stage_batched(const dgc_batch::Header &h, const char *dev, int stage, hipStream_t st) {
    return h.precision == DGC_F32 ? launch_batch<float>(h, dev, stage, st) : launch_batch<double>(h, dev, stage, st);
}

}  // namespace dgc
