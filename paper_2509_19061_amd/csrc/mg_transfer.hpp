// Interpolation weights of the multigrid transfers (bilinear per velocity
// component: linear between coarse faces along the face normal, 3/4 and 1/4
// between coarse rows along the tangent, mirrored at the walls), and the
// prolongation P e_c gathered at one fine unknown.
#pragma once

#include "mg_internal.hpp"

namespace stk {

// Weights of a fine index f on coarse indices along one axis:
// normal axis: f even -> f/2 (1); f odd -> (f-1)/2, (f+1)/2 (1/2 each).
// tangential axis: J = f/2 with 3/4, neighbour J-1 (f even) or J+1 (f odd)
// with 1/4, the neighbour mirrored onto J outside [0, nc).
__device__ __forceinline__ int w_normal(int f, int* c, double* w) {
    if ((f & 1) == 0) { c[0] = f >> 1; w[0] = 1.0; return 1; }
    c[0] = (f - 1) >> 1; w[0] = 0.5;
    c[1] = (f + 1) >> 1; w[1] = 0.5;
    return 2;
}
__device__ __forceinline__ int w_tangent(int f, int nc, int* c, double* w) {
    const int J = f >> 1, nb = (f & 1) ? J + 1 : J - 1;
    if (nb < 0 || nb >= nc) { c[0] = J; w[0] = 1.0; return 1; }
    c[0] = J; w[0] = 0.75;
    c[1] = nb; w[1] = 0.25;
    return 2;
}

// Interpolation terms of one fine unknown: up to 2 x 2 coarse indices with
// weights; absent terms repeat the first index and are masked out.
struct Terms {
    int ci[2], cj[2];
    double wi[2], wj[2];
    int na, nb;
};
__device__ __forceinline__ void pad_terms(Terms& t) {
    if (t.na == 1) { t.ci[1] = t.ci[0]; t.wi[1] = 0.0; }
    if (t.nb == 1) { t.cj[1] = t.cj[0]; t.wj[1] = 0.0; }
}

// (P e_c) at a fine vx / vy unknown (i, j), as double.  The coarse values are
// loaded first, all at once (their indices are inside the coarse arrays
// whether or not the term is used), and the terms added in the order the
// weights list them.
template <typename T>
__device__ __forceinline__ double prolong_sx(const LevelJob<T>& J, int i, int j) {
    Terms t;
    t.na = w_normal(i, t.ci, t.wi);
    t.nb = w_tangent(j, J.cny, t.cj, t.wj);
    pad_terms(t);
    double c[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) c[p][q] = (double)J.cvx[(int64_t)t.cj[q] * J.cld + t.ci[p]];
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double cv = (t.ci[p] >= 1 && t.ci[p] <= J.cnx - 1) ? c[p][q] : 0.0;
            if (p < t.na && q < t.nb) s += t.wi[p] * t.wj[q] * cv;
        }
    return s;
}
template <typename T>
__device__ __forceinline__ double prolong_sy(const LevelJob<T>& J, int i, int j) {
    Terms t;
    t.na = w_tangent(i, J.cnx, t.ci, t.wi);
    t.nb = w_normal(j, t.cj, t.wj);
    pad_terms(t);
    double c[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) c[p][q] = (double)J.cvy[(int64_t)t.cj[q] * J.cld + t.ci[p]];
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double cv = (t.cj[q] >= 1 && t.cj[q] <= J.cny - 1) ? c[p][q] : 0.0;
            if (p < t.na && q < t.nb) s += t.wi[p] * t.wj[q] * cv;
        }
    return s;
}

// The coarse right-hand side P^T r / 4 at one coarse unknown from its 3 x 4 window of fine
// values rv[normal][tangential]: fine faces 2 N - 1 .. 2 N + 1 of the coarse face N with 1/2,
// 1, 1/2, fine rows 2 M - 1 .. 2 M + 2 of the coarse row M with 1/4, 3/4, 3/4, 1/4, mirrored at
// the walls (lo, hi: there is a row below, above).  Terms in window order.
template <typename T>
__device__ __forceinline__ T restrict_sum(const T (&rv)[3][4], bool lo, bool hi) {
    const double wt[4] = {0.25, lo ? 0.75 : 1.0, hi ? 0.75 : 1.0, 0.25};
    double s = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double t = s + (a == 1 ? 0.25 : 0.125) * wt[q] * (double)rv[a][q];
            s = (q == 0 && !lo) || (q == 3 && !hi) ? s : t;
        }
    return T(s);
}
// It and the coarse iterate at the coarse unknown (comp, k): 0, or (J.first) the first sweep
// from 0, w = jac_step(0, omega / d, b, -0) with d the diagonal there.
template <typename T>
__device__ __forceinline__ void store_coarse(const LevelJob<T>& J, int comp, int64_t k, bool unk, T bc, T d, T omega) {
    bc = unk ? bc : T(0);
    (comp == 0 ? J.cbx : J.cby)[k] = bc;
    if (J.first) (comp == 0 ? J.cwx : J.cwy)[k] = unk ? jac_step<T>(T(0), omega / d, bc, -T(0)) : T(0);
    else (comp == 0 ? J.cvx : J.cvy)[k] = T(0);
}

}  // namespace stk
