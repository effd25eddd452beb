// One SSP-RK3 stage in one pass over the elements.
//
// Every element evaluates its volume term, the fluxes of all its faces (a
// face between two elements is evaluated by both, each keeping its own side:
// the same values in f32, in f64 equal to rounding, the own trace being formed
// with 1/sqrt(det J) and tables of the element's own)
// and the stage combination  out = a x + b (y + dt rhs)  with y the stage
// input; the right-hand side never leaves the registers.  Each element writes
// only its own record, so no two work-items touch the same memory and one
// launch covers the whole mesh: a stage reads y (once as the element's own
// record and again, mostly from cache, as its neighbours'), x, the geometry,
// and writes out, where the colored launches read and write the right-hand
// side once per color besides.
//
// A wave owns EW elements, M lanes each (lane = conserved variable m of
// element e; EW = 16 for M = 4, 12 for M = 5).  For a group of FG face slots:
//   1. lane (e, m) forms variable m's traces of both sides at the Q points of
//      every face and stores them in the wave's LDS region;
//   2. the wave's lanes share out the EW * FG * Q points: one lane evaluates
//      the Rusanov flux of all variables at its point, once, and overwrites
//      the neighbour's trace with w_q |f| F*;
//   3. lane (e, m) projects its variable's fluxes onto its N_p modes.
// The exchange stays inside a wave, whose LDS operations execute in order, so
// no work-group barrier is needed and the waves of a work-group run on
// independently.  The volume term is evaluated by the team of four lanes with
// register exchanges (M = 4) or through the same LDS region (M = 5).
// Contributions are added in slot order, the color order of the layout (in
// f64 on conforming meshes in the order of the element's local faces).
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "batch_dev.hpp"
#include "euler_dev.hpp"
#include "volume_team.hpp"

namespace dgc_dev {

// one mesh's arrays and one stage's combination
struct ElemStageArgs {
    const int32_t *slots;      // [ms][n_elem] 2 * face + side, -1 padded
    const int32_t *face_lr;    // [2][n_face]
    const uint8_t *face_code;  // [2][n_face]
    const double *face_geo;    // [DIM + 3][n_face]
    const double *elem_geo;    // [DIM * DIM + 1][n_elem]
    const int8_t *kind;        // [n_elem], mixed meshes
    int64_t n_elem, n_face;
    const double *y, *x;       // stage input; stage-0 state (null: y itself)
    double *out;
    float *shadow;             // f32 form: the new state rounded to f32 (may be null)
    double a, b, dt;
};

// the basis tables of the element type
struct ElemTables {
    const double *trace, *proj, *vb, *vd;
    int n_codes;
};

// 1/x with a second Newton step: within a rounding of the quotient (the
// factor multiplies every trace and projection of the element)
__device__ __forceinline__ double exact_recip(double x) {
    const double r = dev_recip<double>(x);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// x as it is rounded here: not fused into the operation that uses it
template <class T>
__device__ __forceinline__ T rounded(T x) {
    asm("" : "+v"(x));
    return x;
}

// order the wave's LDS writes before its later LDS reads (compiler only: the
// hardware executes one wave's LDS operations in order)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The shapes whose f32 pass rounds as the colored step does, where the colored
// volume term is summed by teams: mixed meshes, parallelograms, and conforming
// triangles at p <= 3.  The others have no f32 kernel.
constexpr bool f32_element_shape(int dim, int n_p, int face_slots, bool mixed) {
    return dim == 2 && (mixed || face_slots == 4 || (face_slots == 3 && n_p <= 10));
}

// Launch shape and LDS sizes, shared by host and device.
template <int DIM, int NP, int Q, int QV, int FS, bool MIXED, class T>
struct ElemCfg {
    static constexpr int M = DIM + 2;
    static constexpr int EW = 64 / M;            // elements per wave
    static constexpr int WAVES = 4;
    static constexpr int BLOCK = 64 * WAVES;
    static constexpr int EPB = EW * WAVES;       // elements per work-group
    static constexpr int NG = DIM + 2;           // side geometry: normal, |f|, 1/sqrt(det J) of the neighbour
    static constexpr int NF = DIM == 3 || FS == 4 ? 4 : 3;  // faces of a conforming element
    static constexpr int NO = DIM == 2 ? 4 : 6;  // orientation codes per local face
    // f32: own and neighbour's tables by face code, in slot order, rounded as
    // the colored kernels round; f64 on conforming meshes whose face rule
    // looks the same from both sides: the sides in the order of the element's
    // local faces, so that its own tables are the same for every lane and
    // come through the scalar cache (FACES).  Not at p = 0, whose tables are
    // constants: in slot order, the color order, a wave's sides lie next to each
    // other in the face arrays, which is most of what that pass reads.
    static constexpr bool PROJ = sizeof(T) == 4;
    static_assert(!PROJ || f32_element_shape(DIM, NP, FS, MIXED), "no f32 pass for this shape");
    static constexpr bool FACES = !PROJ && !MIXED && NP > 1 && FS == NF && (DIM == 2 || Q == 3);
    // The wave's region: planes of one variable's traces at the group's
    // points, own then neighbour's, then planes of the side geometry.  Odd
    // plane lengths spread a store of the M variables over the banks.
    static constexpr int plane(int fg) { return (EW * fg * Q) | 1; }
    static constexpr int gplane(int fg) { return (EW * fg) | 1; }
    static constexpr int group_len(int fg) { return 2 * M * plane(fg) + NG * gplane(fg); }
    // Face slots per group: one; where a side has two points (2 * 16 fill half
    // a wave) two, and all three of a triangle; two for triangles at p = 2;
    // f32 below N_p = 9 all.  Fewer sides at a time leave the flux's share of
    // a wave's lanes the same at three and four points (three sides: 144
    // points in three rounds of 64; one: 48 in one) and take fewer registers
    // and less LDS: 131 registers and three waves per SIMD with three sides,
    // 128 and four with two (991,232 triangles at p = 2: 226 against 219 us a
    // stage; 589,824 parallelograms at p = 2 234 with four sides, 217 with
    // one; both before the late x read below, with which two sides take 116).
    // 2D at p = 0: all sides, three of a refined triangle, whose reads are then
    // in flight together.  One at a time, in face order / all, us a step:
    // 980,000 triangles 286 / 173 (colored launches 219), 589,824
    // parallelograms 225 / 128 (189), 944,292 triangles of a refined mesh 295 /
    // 235, 512 triangles 17.3 / 12.4; tetrahedra at p = 0 (511,104) 316 / 368.
    static constexpr int FG = PROJ ? (NP >= 9 ? 1 : FS)
                              : NP == 1 && DIM == 2 ? (FS > 4 ? 3 : FS)
                              : NP == 3 && FS == 3 ? 3
                              : Q == 2 || (NP == 6 && FS == 3) ? 2 : 1;
    // Refined meshes: only elements beside smaller ones fill more than three
    // slots, so a wave whose elements do not leaves the remaining groups out
    // (the adapted mesh of 200 x 200 x 2 base triangles at p = 2: 144 against
    // 119 us a step).  On mixed meshes, whose triangles leave one of four slots
    // empty, the test made no difference (167 us).
    static constexpr bool PADDED = FS > 4;
    // Each group's reads are issued before the work on the group ahead of it
    // from N_p = 10 on and in 3D.  us a step with / without (registers): triangles
    // p = 3 (145 / 127, three waves per SIMD against four) 512 elements 37.7 /
    // 39.9, 64,800 95 / 88, 980,000 1,067 / 1,045; p = 4 (187 / 155, two against
    // three) 66.0 / 70.4, 188 / 188, 1,998 / 1,830; p = 5 (233 / 196, two) 96 /
    // 107, 294 / 317, 4,101 / 4,342; six slots, 37,992 and 944,292 elements: p = 3
    // (154 / 137, three) 94 / 96, 1,337 / 1,345; p = 4 (193 / 167, two against
    // three) 176 / 146, 2,304 / 2,140; p = 5 (244 / 208, two) 311 / 300, 4,156 /
    // 4,013; parallelograms p = 3 (195 / 169, two) 256 elements 54 / 68, 589,824
    // 1,243 / 1,336; mixed p = 3 (254 / 166, two against three) 308 elements 88 /
    // 101, 191,420 728 / 730; 511,104 tetrahedra p = 0, 1, 2 (115 / 104, 138 /
    // 130, 183 / 177: the same waves) 330 / 344, 510 / 536, 2,179 / 2,275.
    // So small meshes gain at every order and large ones except where it costs
    // a wave; triangles at p = 3 and 4 keep it for the small ones.  Below N_p =
    // 10 it would cost the fourth wave.
    static constexpr bool AHEAD = NP >= 10 || M == 5;
    // the volume term by register exchanges of the team of four lanes, or
    // (M = 5) through the region, QC points at a time; through the region for
    // M = 4 too took 2 % longer on 991,232 triangles at p = 2
    static constexpr bool VTEAM = M == 4;
    // f64 triangles at p = 1: two volume points per trip of the team's loop,
    // and the tables staged before the element's own reads (the other orders
    // stage them behind these).  512 triangles, bound by latency: 17.4, with
    // two points 16.6, with both 16.3 us a step; 991,232: 410 us either way.
    static constexpr bool SMALL = NP == 3 && !PROJ;
    static constexpr int UNR = SMALL ? 2 : team_volume_unroll(NP);
    static constexpr int QC = QV < 4 ? QV : (QV % 4 == 0 ? 4 : 5);   // 48 or 60 of the 64 lanes
    static constexpr int VLEN = VTEAM ? 0 : M * DIM * ((EW * QC) | 1);
    static constexpr int REGION = group_len(FG) > VLEN ? group_len(FG) : VLEN;
    // volume points evaluated while the sides are read
    static constexpr int QH = VTEAM ? QV / 3 : QV / 3 / QC * QC > 0 ? QV / 3 / QC * QC : (QV > QC ? QC : 0);
    __host__ __device__ static constexpr int tab_len(int n_codes) {
        return PROJ ? 2 * n_codes * Q * NP : n_codes * Q * NP + Q;
    }
    static constexpr bool VFUSED = PROJ && !MIXED;
    static constexpr int VTAB = MIXED ? 2 * (1 + DIM) * QV * NP : 0;  // mixed meshes: both kinds' volume tables

    __host__ __device__ static constexpr size_t lds_bytes(int n_codes) {
        return (size_t)(tab_len(n_codes) + VTAB + WAVES * REGION) * sizeof(T);
    }
};

// Volume term of M = 5 variables at the points [Q0, Q1) through the wave's
// LDS region: the point values are exchanged, each point's flux is evaluated
// once.
template <int DIM, int NP, int QV, int QC, int EW, int Q0, int Q1, class T>
__device__ __forceinline__ void volume_wave(int lane, int e, int m, bool lane_ok, const T (&Ji)[DIM * DIM], T isq,
                                            const double *__restrict__ vb, const double *__restrict__ vd,
                                            const T (&c)[NP], T *region, T (&acc)[NP]) {
    constexpr int M = DIM + 2;
    constexpr int P = (EW * QC) | 1;
#pragma unroll 1
    for (int q0 = Q0; q0 < Q1; q0 += QC) {
        const int nq = Q1 - q0 < QC ? Q1 - q0 : QC;
        if (lane_ok) {
#pragma unroll 2
            for (int q = 0; q < nq; ++q) {
                T t = 0;
#pragma unroll
                for (int j = 0; j < NP; ++j) t += T(vb[(q0 + q) * NP + j]) * c[j];
                region[m * P + e * QC + q] = t * isq;
            }
        }
        wave_lds_fence();
        for (int t = lane; t < EW * QC; t += 64) {
            T u[M], F[M * DIM];
#pragma unroll
            for (int i = 0; i < M; ++i) u[i] = region[i * P + t];
            phys_flux<DIM, T>(u, F);
#pragma unroll
            for (int i = 0; i < M * DIM; ++i) region[i * P + t] = F[i];
        }
        wave_lds_fence();
        if (lane_ok) {
#pragma unroll 1
            for (int q = 0; q < nq; ++q) {
                const T *v = region + m * DIM * P + e * QC + q;
                T F[DIM];
#pragma unroll
                for (int d = 0; d < DIM; ++d) F[d] = v[d * P];
#pragma unroll
                for (int d = 0; d < DIM; ++d) {
                    T g = 0;
#pragma unroll
                    for (int i = 0; i < DIM; ++i) g += Ji[d * DIM + i] * F[i];
#pragma unroll
                    for (int j = 0; j < NP; ++j) acc[j] = dev_fma(T(vd[(d * QV + q0 + q) * NP + j]), g, acc[j]);
                }
            }
        }
        wave_lds_fence();
    }
}

// Where point q of a face, in the order of the element's own local face,
// stands among the face's points seen through orientation o: 2D reversed for
// odd o; 3D (three points, one per vertex) the inverse of the o-th
// permutation in lexicographic order, two bits an entry.
template <int DIM, int Q>
__device__ __forceinline__ int point_place(int o, int q) {
    if constexpr (DIM == 2) {
        return (o & 1) ? Q - 1 - q : q;
    } else {
        // inverses of 012 021 102 120 201 210
        constexpr uint64_t inv = 0x24ull | 0x18ull << 6 | 0x21ull << 12 | 0x12ull << 18 | 0x09ull << 24 | 0x06ull << 30;
        return (int)(inv >> (6 * o + 2 * q)) & 3;
    }
}

// The stage of the EPB elements from k0 on (every thread of the work-group
// calls; s_tab holds the trace tables, the face weights or projection tables,
// then on mixed meshes the volume tables).  `mid` stages the tables and meets
// the work-group barrier.
template <int DIM, int NP, int Q, int QV, int FS, bool MIXED, class T, class Mid>
__device__ __forceinline__ void element_stage(const ElemStageArgs &A, const ElemTables &tab, int64_t k0, int ms,
                                              const T *s_tab, T *s_regions, const Mid &mid) {
    using C = ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>;
    constexpr int M = C::M, EW = C::EW, FG = C::FG;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int e = lane / M, m = lane - e * M;
    const int64_t k = k0 + wave * EW + e;
    const bool lane_ok = e < EW && k < A.n_elem;
    const int64_t K = A.n_elem, E = A.n_face;
    const int64_t kc = lane_ok ? k : 0;  // every read is of a valid element
    const int nc = tab.n_codes;
    const T *s_tr = s_tab, *s_w = s_tab + nc * Q * NP;  // weights (f64) or projection tables (f32)
    T *region = s_regions + wave * C::REGION;

    if constexpr (C::SMALL) mid();
    int32_t slot[FS];
#pragma unroll
    for (int s = 0; s < FS; ++s) slot[s] = s < ms ? A.slots[(int64_t)s * K + kc] : -1;
    double yv[NP];
    const size_t base = ((size_t)kc * M + m) * NP;
#pragma unroll
    for (int j = 0; j < NP; ++j) yv[j] = A.y[base + j];
    T Ji[DIM * DIM];
    double sq;
    load_elem_geo<DIM, T>(kc, K, A.elem_geo, Ji, sq);
    const int kind = MIXED ? (A.kind[kc] ? 1 : 0) : 0;

    if constexpr (!C::SMALL) mid();
    // the sides: neighbour (-1 where there is none), codes; read and checked
    // without branches, so that the reads of all sides are in flight together
    int32_t nb[FS];
    int co[FS], cn[FS];
    bool ok[FS];
    const uint32_t E2 = (uint32_t)(2 * E);
#pragma unroll
    for (int i = 0; i < FS; ++i) {
        const uint32_t sl = (uint32_t)slot[i];
        const uint32_t f = sl < E2 ? sl >> 1 : 0u;
        const bool right = sl & 1;
        nb[i] = A.face_lr[(right ? 0 : E) + f];
        co[i] = A.face_code[(right ? E : 0) + f];
        cn[i] = A.face_code[(right ? 0 : E) + f];
    }
    // the volume term at the points [Q0, Q1), without its factor sqrt(det J)
    T c[NP], acc[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        c[j] = T(yv[j]);
        acc[j] = T(0);
    }
    const double isq_d = sizeof(T) == 8 ? exact_recip(sq) : 1.0 / sq;
    const T isq = T(isq_d);
    auto volume = [&](auto first, auto end) {
        constexpr int Q0 = decltype(first)::value, Q1 = decltype(end)::value;
        if constexpr (!C::VTEAM) {
            volume_wave<DIM, NP, QV, C::QC, EW, Q0, Q1, T>(lane, e, m, lane_ok, Ji, isq, tab.vb, tab.vd, c, region,
                                                           acc);
        } else if constexpr (MIXED) {
            const T *s_vb = s_tab + C::tab_len(nc);
            const T *s_vd = s_vb + 2 * QV * NP;
            volume_team_points<DIM, NP, QV, Q0, Q1, T>(m, Ji, isq, s_vb + kind * QV * NP, s_vd + kind * DIM * QV * NP, c,
                                                       acc);
        } else {
            volume_team_points<DIM, NP, QV, Q0, Q1, T, double, C::UNR>(m, Ji, isq, tab.vb, tab.vd, c, acc);
        }
    };
    constexpr int QH = C::QH;
    // the first half of the points covers the reads of the sides, the second
    // half those of the neighbours' records
    volume(std::integral_constant<int, 0>{}, std::integral_constant<int, QH>{});

#pragma unroll
    for (int i = 0; i < FS; ++i) {
        // a side whose slot, neighbour or codes are out of range is skipped,
        // never dereferenced
        ok[i] = lane_ok & ((uint32_t)slot[i] < E2) & (nb[i] < K) & (co[i] < nc) & (cn[i] < nc) &
                ((nb[i] >= 0) | !(slot[i] & 1));
        nb[i] = ok[i] ? nb[i] : -1;
        co[i] = ok[i] ? co[i] : 0;
        cn[i] = ok[i] ? cn[i] : 0;
    }
    // in the order of the local faces
    if constexpr (C::FACES) {
        int32_t sl2[FS], nb2[FS];
        int co2[FS], cn2[FS];
        bool ok2[FS];
#pragma unroll
        for (int f = 0; f < FS; ++f) {
            sl2[f] = -1;
            nb2[f] = -1;
            co2[f] = cn2[f] = 0;
            ok2[f] = false;
#pragma unroll
            for (int i = 0; i < FS; ++i) {
                const bool hit = ok[i] & ((uint32_t)(co[i] - f * C::NO) < (uint32_t)C::NO);
                sl2[f] = hit ? slot[i] : sl2[f];
                nb2[f] = hit ? nb[i] : nb2[f];
                co2[f] = hit ? co[i] - f * C::NO : co2[f];  // the orientation
                cn2[f] = hit ? cn[i] : cn2[f];
                ok2[f] = ok2[f] | hit;
            }
        }
#pragma unroll
        for (int f = 0; f < FS; ++f) {
            slot[f] = sl2[f];
            nb[f] = nb2[f];
            co[f] = co2[f];
            cn[f] = cn2[f];
            ok[f] = ok2[f];
        }
    }

    // The stage-0 state of the combination (the element's own record again
    // where the combination has none).  f32, bound by memory: not read where
    // there is none (500,000 triangles at p = 2: 303 against 316 us a step);
    // f64: without that branch, up front for small records, at the end from
    // N_p = 6 on, where its registers cost a wave (589,824 parallelograms at
    // p = 2: 622 against 648 us a step, 991,232 triangles at p = 1 414 late
    // against 403 early).
    constexpr bool LATE_X = C::PROJ ? NP >= 15 : M == 4 && NP > 4;
    double xv[NP];
    auto read_x = [&]() {
        if constexpr (C::PROJ) {
            if (A.x) {
#pragma unroll
                for (int j = 0; j < NP; ++j) xv[j] = A.x[base + j];
            } else {
#pragma unroll
                for (int j = 0; j < NP; ++j) xv[j] = yv[j];
            }
        } else {
            const double *xp = (A.x ? A.x : A.y) + base;
#pragma unroll
            for (int j = 0; j < NP; ++j) xv[j] = xp[j];
        }
    };
    if constexpr (!LATE_X) read_x();

    // a group's reads: the neighbours' records (the element's own where there
    // is none), and the geometry of side i by lane m = i of the element
    struct Sides {
        T nb[FG][NP];
        double geo[C::NG];
    };
    static_assert(FG <= M, "a lane of the element for every side of a group");
    auto read_group = [&](auto first, Sides &v) {
        constexpr int s0 = decltype(first)::value;
        uint32_t sl = 0;
#pragma unroll
        for (int i = 0; i < FG && s0 + i < FS; ++i) sl = (i == m) & ok[s0 + i] ? (uint32_t)slot[s0 + i] : sl;
        const double *fg = A.face_geo + (sl >> 1);
#pragma unroll
        for (int d = 0; d <= DIM; ++d) v.geo[d] = fg[d * E];
        v.geo[DIM + 1] = fg[(DIM + ((sl & 1) ? 1 : 2)) * E];
#pragma unroll
        for (int i = 0; i < FG && s0 + i < FS; ++i) {
            const int64_t b = nb[s0 + i] >= 0 ? nb[s0 + i] : kc;
            const double *u = A.y + ((size_t)b * M + m) * NP;
#pragma unroll
            for (int j = 0; j < NP; ++j) v.nb[i][j] = T(u[j]);
        }
    };
    Sides sides0;
    read_group(std::integral_constant<int, 0>{}, sides0);
    volume(std::integral_constant<int, QH>{}, std::integral_constant<int, QV>{});
    if constexpr (!C::VFUSED) {
#pragma unroll
        for (int j = 0; j < NP; ++j) acc[j] *= T(sq);
    }

    // one group of face slots
    auto group = [&](auto first, const Sides &v) {
        constexpr int s0 = decltype(first)::value;
        constexpr int G = FS - s0 < FG ? FS - s0 : FG;
        constexpr int P = C::plane(G), GP = C::gplane(G);
        T *s_own = region, *s_nb = region + M * P, *s_geo = region + 2 * M * P;
        if (lane_ok && m < G) {
            bool right = slot[s0] & 1, wall = nb[s0] < 0;
#pragma unroll
            for (int i = 1; i < G; ++i) {
                right = i == m ? slot[s0 + i] & 1 : right;
                wall = i == m ? nb[s0 + i] < 0 : wall;
            }
            T *q = s_geo + e * G + m;
#pragma unroll
            for (int d = 0; d < DIM; ++d) q[d * GP] = T(v.geo[d]);
            q[DIM * GP] = T(C::PROJ ? v.geo[DIM] * isq_d : v.geo[DIM]);
            // negative: this element is the face's right one; 0: wall
            const T is = wall ? T(0) : T(v.geo[DIM + 1]);
            q[(DIM + 1) * GP] = right ? -is : is;
        }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int s = s0 + i;
            if (!ok[s]) continue;
            T *po = s_own + m * P + (e * G + i) * Q, *pn = s_nb + m * P + (e * G + i) * Q;
            const T sn = s_geo[(DIM + 1) * GP + e * G + i], isn = sn < T(0) ? -sn : sn;
            const T *tn = s_tr + cn[s] * Q * NP, *to = s_tr + co[s] * Q * NP;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                T t = 0, u = 0;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    t += (C::FACES ? T(tab.trace[(s * C::NO * Q + q) * NP + j]) : to[q * NP + j]) * c[j];
                    u += tn[q * NP + j] * v.nb[i][j];
                }
                po[C::FACES ? point_place<DIM, Q>(co[s], q) : q] = t * isq;
                pn[q] = u * isn;
            }
        }
        wave_lds_fence();
        for (int t = lane; t < EW * G * Q; t += 64) {
            const int side = t / Q;
            const T *g = s_geo + side;
            T n[DIM], uL[M], uR[M];
#pragma unroll
            for (int d = 0; d < DIM; ++d) n[d] = g[d * GP];
            const T isn = g[(DIM + 1) * GP];
            // the flux in the face's own left-to-right sense, from both of its
            // elements
            const T *pl = (isn < T(0) ? s_nb : s_own) + t, *pr = (isn < T(0) ? s_own : s_nb) + t;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                uL[i] = pl[i * P];
                uR[i] = pr[i * P];
            }
            if (isn == T(0)) wall_ghost<DIM, T>(uL, n, uR);
            T F[M], w = T(1);
            if constexpr (C::PROJ) {
                rusanov_components<DIM, T>(uL, uR, n, F);
            } else {
                rusanov<DIM, T>(uL, uR, n, F);
                w = g[DIM * GP] * s_w[t - side * Q];
                w = isn < T(0) ? w : -w;
            }
#pragma unroll
            for (int i = 0; i < M; ++i) s_nb[i * P + t] = C::PROJ ? F[i] : F[i] * w;
        }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int s = s0 + i;
            if (!ok[s]) {
                if (C::VFUSED && s == 0) {
#pragma unroll
                    for (int j = 0; j < NP; ++j) acc[j] *= T(sq);
                }
                continue;
            }
            const T *pr = (C::PROJ ? s_w : s_tr) + co[s] * Q * NP;
            const T *pf = s_nb + m * P + (e * G + i) * Q;
            T f[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                f[q] = pf[C::FACES ? point_place<DIM, Q>(co[s], q) : q];
                if (!C::PROJ) f[q] *= isq;  // the sign is in the flux
            }
            if constexpr (C::PROJ) {
                const T scale = s_geo[DIM * GP + e * G + i];
                const bool right = slot[s] & 1;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    T a = 0;
#pragma unroll
                    for (int q = 0; q < Q; ++q) a += pr[q * NP + j] * f[q];
                    // the first slot also scales the volume sum, rounded as
                    // the colored kernel that carries the volume term rounds
                    if (C::VFUSED && s == 0)
                        acc[j] = right ? dev_fma(a, scale, rounded(acc[j] * T(sq)))
                                       : dev_fma(acc[j], T(sq), -rounded(scale * a));
                    else acc[j] = dev_fma(a, right ? scale : -scale, acc[j]);
                }
            } else {
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int j = 0; j < NP; ++j)
                        acc[j] = dev_fma(C::FACES ? T(tab.trace[(s * C::NO * Q + q) * NP + j]) : pr[q * NP + j], f[q],
                                         acc[j]);
            }
        }
        if constexpr (s0 + FG < FS) wave_lds_fence();
    };
    auto groups = [&](auto &self, auto first, const Sides &cur) -> void {
        constexpr int s0 = decltype(first)::value;
        if constexpr (s0 + FG < FS) {
            // past the slots that every element fills: whether the wave has
            // any side left
            bool more = true;
            if constexpr (C::PADDED && s0 + FG >= 3) {
                bool left = false;
#pragma unroll
                for (int i = s0 + FG; i < FS; ++i) left = left | ok[i];
                more = __any(left);
            }
            Sides next;
            if constexpr (C::AHEAD) read_group(std::integral_constant<int, s0 + FG>{}, next);
            group(first, cur);
            if (more) {
                if constexpr (!C::AHEAD) read_group(std::integral_constant<int, s0 + FG>{}, next);
                self(self, std::integral_constant<int, s0 + FG>{}, next);
            }
        } else {
            group(first, cur);
        }
    };
    groups(groups, std::integral_constant<int, 0>{}, sides0);
    if (!lane_ok) return;
    if constexpr (LATE_X) read_x();
    // f32: rounded as the combination kernels of the colored step round it,
    // spelled out because the compiler otherwise fuses either product, by
    // shape.  In f64 this order is the further one from the exact sum (65,522
    // triangles at p = 3, four steps: 2.7e-16 against 2.4e-16).
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const double v = C::PROJ ? __builtin_fma(A.a, xv[j], A.b * __builtin_fma(A.dt, (double)acc[j], yv[j]))
                                 : A.a * xv[j] + A.b * (yv[j] + A.dt * (double)acc[j]);
        A.out[base + j] = v;
        if (sizeof(T) == 4 && A.shadow) A.shadow[base + j] = (float)v;
    }
}

// the basis tables into LDS (every thread; ends with a work-group barrier)
template <int DIM, int NP, int Q, int QV, int FS, bool MIXED, class T>
__device__ __forceinline__ void stage_elem_tables(T *s, const ElemTables &tab) {
    const int n = tab.n_codes * Q * NP;
    using C = ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        s[i] = T(tab.trace[i]);
        if constexpr (C::PROJ) s[n + i] = T(tab.proj[i]);
    }
    // the projection table is the weights times the trace table: the weights
    // from its constant mode, whose trace is the same positive value everywhere
    if constexpr (!C::PROJ)
        for (int q = threadIdx.x; q < Q; q += blockDim.x) s[n + q] = T(tab.proj[q * NP] / tab.trace[q * NP]);
    if constexpr (MIXED) {
        T *v = s + C::tab_len(tab.n_codes);
        for (int i = threadIdx.x; i < 2 * QV * NP; i += blockDim.x) v[i] = T(tab.vb[i]);
        for (int i = threadIdx.x; i < 2 * DIM * QV * NP; i += blockDim.x) v[2 * QV * NP + i] = T(tab.vd[i]);
    }
    __syncthreads();
}

// Work-groups are dealt round-robin to the 8 XCDs: give each XCD runs of
// CHUNK consecutive work-groups, whose neighbours' records then sit in its
// own L2 (the last, incomplete round stays as it is): a stage on 991,232
// triangles at p = 2 fetches 577 instead of 750 MB, on 511,104 tetrahedra at
// p = 1 it takes 183 instead of 193 us.
__device__ __forceinline__ unsigned chunked_block(unsigned b, unsigned nb) {
    constexpr unsigned CHUNK = 32;
    const unsigned first = b / (8 * CHUNK) * (8 * CHUNK), r = b - first;
    return first + 8 * CHUNK > nb ? b : first + r % 8 * CHUNK + r / 8;
}

template <int DIM, int NP, int Q, int QV, int FS, bool MIXED, class T>
__global__ __launch_bounds__((ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>::BLOCK)) void element_stage_kernel(ElemStageArgs A, ElemTables tab, int ms) {
    using C = ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>;
    extern __shared__ unsigned char smem_raw[];
    T *s_tab = reinterpret_cast<T *>(smem_raw);
    element_stage<DIM, NP, Q, QV, FS, MIXED, T>(A, tab, (int64_t)chunked_block(blockIdx.x, gridDim.x) * C::EPB, ms, s_tab,
                                                s_tab + C::tab_len(tab.n_codes) + C::VTAB,
                                                [&] { stage_elem_tables<DIM, NP, Q, QV, FS, MIXED, T>(s_tab, tab); });
}

// The stage of every mesh of a batch: a work-group finds its mesh in the
// descriptor's block map.
template <int DIM, int NP, int Q, int QV, int FS, bool MIXED, class T>
__global__ __launch_bounds__((ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>::BLOCK)) void batch_element_stage_kernel(const char *__restrict__ desc, int stage) {
    using C = ElemCfg<DIM, NP, Q, QV, FS, MIXED, T>;
    extern __shared__ unsigned char smem_raw[];
    T *s_tab = reinterpret_cast<T *>(smem_raw);
    const Header *h = bh(desc);
    const double *tables = gptr(h->tables);
    const ElemTables tab{tables + h->off_trace, tables + h->off_proj, tables + h->off_vb, tables + h->off_vd,
                         h->n_codes};
    const unsigned b = chunked_block(blockIdx.x, gridDim.x);
    const int32_t i = reinterpret_cast<const int32_t *>(desc + h->off_map_stage)[b];
    const Entry *en = bentry(desc, i);
    const Member mb = member(en, sizeof(T) == 4);
    ElemStageArgs A;
    A.slots = gptr(en->slots);
    A.face_lr = mb.face_lr;
    A.face_code = mb.face_code;
    A.face_geo = mb.face_geo;
    A.elem_geo = mb.elem_geo;
    A.kind = nullptr;
    A.n_elem = en->n_elem;
    A.n_face = en->n_face;
    A.y = stage == 0 ? mb.U : (stage == 1 ? mb.w.U1 : mb.w.U2);
    A.x = stage == 0 ? nullptr : mb.U;
    A.out = stage == 0 ? mb.w.U1 : (stage == 1 ? mb.w.U2 : mb.U);
    // the f32 shadow that the batched volume and surface calls read is left
    // as a step with separate combinations leaves it: the last stage's input
    A.shadow = stage == 1 ? mb.w.shadow : nullptr;
    A.a = stage == 0 ? 0.0 : (stage == 1 ? 0.75 : 1.0 / 3.0);
    A.b = stage == 0 ? 1.0 : (stage == 1 ? 0.25 : 2.0 / 3.0);
    A.dt = en->dt;
    element_stage<DIM, NP, Q, QV, FS, MIXED, T>(A, tab, ((int64_t)b - en->blk_stage) * C::EPB, en->max_slots,
                                                s_tab, s_tab + C::tab_len(tab.n_codes) + C::VTAB,
                                                [&] { stage_elem_tables<DIM, NP, Q, QV, FS, MIXED, T>(s_tab, tab); });
}

}  // namespace dgc_dev
