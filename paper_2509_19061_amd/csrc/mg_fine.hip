// The finest (matrix-free) level of the V-cycle in one pass each way, on the
// register pipeline of jacobi_pipe.hpp:
//   down: nu sweeps v -> w, the residual of w, its restriction to the coarse
//         right-hand side and, from the coarse zero iterate, the first coarse sweep;
//   up:   w + P e_c -> v after nu sweeps.
// The residual is one more level of the pipeline, whose rows stay in registers: a
// coarse row is summed from the last four of them and the neighbouring lanes, and
// written by the lanes of even columns.  The prolongation is added to a row of w
// when it arrives, from three coarse rows held per lane.
//
// Both are bound by memory.  Separate passes for the sweeps, the residual, the
// restriction, the prolongation and the sweeps moved about 32 planes per cycle;
// these move 18 (down: 6 read, 2 written, about 1.5 coarse; up: 6 read, 2 written,
// half a coarse one).
//
// Sums and updates are those of the separate kernels, term by term, so the values
// are the same bits; terms that those kernels leave out are added here as exact 0.
#include <algorithm>
#include <cmath>

#include "coarse_stencil.hpp"
#include "jacobi_pipe.hpp"
#include "mg_internal.hpp"

namespace stk {
namespace {

using namespace pipe;

// Lanes given up on each side: down, the residual is exact K + 1 lanes in and a
// coarse value reaches one lane to the left and two to the right; up, the outermost
// lanes lack a coarse neighbour.  Strips start at even columns.
constexpr int down_left(int K) { return (K + 3) / 2 * 2; }
constexpr int down_strip(int K) { return 62 - K - down_left(K) - K % 2; }
constexpr int up_margin(int K) { return K + 1; }
constexpr int up_strip(int K) { return 64 - 2 * up_margin(K); }
static_assert(down_strip(1) % 2 == 0 && down_strip(2) % 2 == 0 && down_strip(3) % 2 == 0, "even strips");
// the last coarse lane, down_left + down_strip - 2, must find exact residuals two lanes further on
static_assert(down_left(1) + down_strip(1) <= 62 - 1 && down_left(2) + down_strip(2) <= 62 - 2 &&
                  down_left(3) + down_strip(3) <= 62 - 3, "right margin");
// the down pass keeps four residual rows, named by the row modulo 4
constexpr int DOWN_RING = 8;

__device__ __forceinline__ int find_fine_inst(const int* __restrict__ pre, int n, int b) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <typename T, int K, bool SQ>
__global__ __launch_bounds__(64 * WPB, sizeof(T) == 8 ? 2 : 3) void k_fine_down(const LevelJob<T>* __restrict__ jobs,
                                                                               const int* __restrict__ pre,
                                                                               const FineShape* __restrict__ shapes,
                                                                               int n, T omega, FineIo io) {
    const int b = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int inst = find_fine_inst(pre, n, b);
    const LevelJob<T>& J = jobs[inst];
    const FineShape sh = shapes[inst];
    const int wv = (b - pre[inst]) * WPB + rows::wave_in_group();
    const int strip_ = wv % sh.nstrip, segm = wv / sh.nstrip;
    if (segm >= sh.nseg) return;  // the whole wave
    const int nx = J.nx, ny = J.ny, NX = J.cnx, NY = J.cny, lane = threadIdx.x & 63;
    constexpr int M = down_left(K), SWD = down_strip(K);
    const int i = strip_ * SWD - M + lane, y0 = segm * sh.seg, y1 = min(y0 + sh.seg, ny + 1);
    const bool own = lane >= M && lane < M + SWD && i <= nx;
    const int r0 = y0 - K - 2, r1 = y1 + K + 3;
    const PipeRows<T> L(io.vx ? (const T*)io.vx : (const T*)J.vx, io.vy ? (const T*)io.vy : (const T*)J.vy,
                        (const T*)J.ec, (const T*)J.en, io.bx ? (const T*)io.bx : (const T*)J.bx,
                        io.by ? (const T*)io.by : (const T*)J.by, J.ld, nx, ny, i, r0, r1 - r0 + DOWN_RING + 4,
                        io.zero != 0);
    const PipeStore<T> put((T*)J.wx, (T*)J.wy, J.ld, nx, ny, y0, y1, i, own);
    // coarse column of an even lane; weights along x of the vy terms (mirrored at the walls)
    const int I = i >> 1;
    const bool cown = own && (i & 1) == 0;
    const bool cux = I >= 1 && I <= NX - 1;
    const unsigned ccol = (unsigned)I * (unsigned)sizeof(T);
    const unsigned c_x = cown ? ccol : OOB, c_y = cown && I < NX ? ccol : OOB;
    const double h1 = I == 0 ? 1.0 : 0.75, h2 = I == NX - 1 ? 1.0 : 0.75;
    const double g0 = I > 0 ? 0.25 : 0.0, g3 = I < NX - 1 ? 0.25 : 0.0;
    const T *dgx = J.cst, *dgy = J.cst + PL_VY * J.cplane;
    T *cbx = J.cbx, *cby = J.cby, *ox = J.first ? J.cwx : J.cvx, *oy = J.first ? J.cwy : J.cvy;
    const int64_t cld = J.cld;
    const bool first = J.first != 0;
    const RowSpan cs(y0 >> 1, (y1 - y0) / 2 + 2, cld, (int)sizeof(T));  // the segment's coarse rows

    T rx[4], ry[4];  // residual rows by row modulo 4 (relative to the walk)
#pragma unroll
    for (int q = 0; q < 4; ++q) rx[q] = ry[q] = T(0);
    auto diag = [&](int jc, T& dx, T& dy) {  // the coarse level's diagonals of coarse row jc
        const bool in = first && 2 * jc >= y0 && 2 * jc < y1;
        dx = buf_load_at<T>(cs.of(dgx, cld, in), c_x, cs.at(jc));
        dy = buf_load_at<T>(cs.of(dgy, cld, in), c_y, cs.at(jc));
    };
    T dx = T(0), dy = T(0);
    walk<T, K, SQ, true, DOWN_RING>(
        L, r0, r1, AllCells(nx, ny, i), omega, J.idx, J.idy, [](int, int, rows::Row<T>&) {}, put,
        [&](int u, int j, T px, T py) {
            rx[u & 3] = px;
            ry[u & 3] = py;
            if (!(u & 1)) return;  // odd fine rows (the walk starts so that u and j differ in parity)
            // rows j - 3 .. j = 2 jc - 1 .. 2 jc + 2 of coarse row jc
            const int jc = (j - 2) >> 1;
            const T ex = dx, ey = dy;
            diag(jc + 1, dx, dy);
            double sx = 0.0, sy = 0.0;
            {
                const double v0 = jc > 0 ? 0.25 : 0.0, v1 = jc == 0 ? 1.0 : 0.75, v2 = jc == NY - 1 ? 1.0 : 0.75,
                             v3 = jc < NY - 1 ? 0.25 : 0.0;
                const double wv[4] = {v0, v1, v2, v3};
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const T own_ = rx[(u + 1 + q) & 3];
                        const T val = a == 0 ? wave_shift<DPP_FROM_PREV>(own_)
                                             : a == 1 ? own_ : wave_shift<DPP_FROM_NEXT>(own_);
                        sx = __builtin_fma(0.25 * (a == 1 ? 1.0 : 0.5) * wv[q], (double)val, sx);
                    }
            }
            {
                const double hv[4] = {g0, h1, h2, g3};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const T own_ = ry[(u + 1 + q) & 3];
                    const T n1 = wave_shift<DPP_FROM_NEXT>(own_);
                    const T val[4] = {wave_shift<DPP_FROM_PREV>(own_), own_, n1, wave_shift<DPP_FROM_NEXT>(n1)};
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        sy = __builtin_fma(0.25 * (q == 1 ? 1.0 : 0.5) * hv[a], (double)val[a], sy);
                }
            }
            const bool in = 2 * jc >= y0 && 2 * jc < y1;
            const bool ux = cux && jc < NY, uy = jc >= 1 && jc <= NY - 1;
            const T bx = ux ? T(sx) : T(0), by = uy ? T(sy) : T(0);
            const T fx = first && ux ? jac_step<T>(T(0), omega / ex, bx, -T(0)) : T(0);
            const T fy = first && uy ? jac_step<T>(T(0), omega / ey, by, -T(0)) : T(0);
            const unsigned o = cs.at(jc);
            buf_store_at(bx, cs.of(cbx, cld, in && jc < NY), c_x, o);
            buf_store_at(fx, cs.of(ox, cld, in && jc < NY), c_x, o);
            buf_store_at(by, cs.of(cby, cld, in), c_y, o);
            buf_store_at(fy, cs.of(oy, cld, in), c_y, o);
        });
}

// Coarse values of rows m - 1, m, m + 1 at the lane's coarse column, m = r >> 1 of
// the row r that arrives next, and row m + 2 on its way.
template <typename T>
struct CoarseRows {
    T x0, x1, x2, x3, y1, y2, y3;
};

template <typename T, int K, bool SQ>
__global__ __launch_bounds__(64 * WPB, sizeof(T) == 8 ? 2 : 4) void k_fine_up(const LevelJob<T>* __restrict__ jobs,
                                                                             const int* __restrict__ pre,
                                                                             const FineShape* __restrict__ shapes,
                                                                             int n, T omega, FineIo io) {
    const int b = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int inst = find_fine_inst(pre, n, b);
    const LevelJob<T>& J = jobs[inst];
    const FineShape sh = shapes[inst];
    const int wv = (b - pre[inst]) * WPB + rows::wave_in_group();
    const int strip_ = wv % sh.nstrip, segm = wv / sh.nstrip;
    if (segm >= sh.nseg) return;  // the whole wave
    const int nx = J.nx, ny = J.ny, NX = J.cnx, NY = J.cny, lane = threadIdx.x & 63;
    constexpr int M = up_margin(K), SWU = up_strip(K), R = ring_rows<T>(K);
    static_assert(R % 2 == 0, "row parity is that of the step");
    const int i = strip_ * SWU - M + lane, y0 = segm * sh.seg, y1 = min(y0 + sh.seg, ny + 1);
    const bool xcol = i >= 1 && i <= nx - 1, ycol = i >= 0 && i <= nx - 1;
    const int r0 = y0 - K, r1 = y1 + K;
    const PipeRows<T> L((const T*)J.wx, (const T*)J.wy, (const T*)J.ec, (const T*)J.en,
                        io.bx ? (const T*)io.bx : (const T*)J.bx, io.by ? (const T*)io.by : (const T*)J.by, J.ld, nx,
                        ny, i, r0, r1 - r0 + R + 4, false);
    const PipeStore<T> put(io.vx ? (T*)io.vx : (T*)J.vx, io.vy ? (T*)io.vy : (T*)J.vy, J.ld, nx, ny, y0, y1, i,
                           lane >= M && lane < M + SWU);
    const T *ex = J.cvx, *ey = J.cvy;
    const int64_t cld = J.cld;
    const int I = i >> 1;
    const bool odd = i & 1;
    const unsigned ccol = (unsigned)I * (unsigned)sizeof(T);
    const unsigned c_x = I >= 1 && I <= NX - 1 ? ccol : OOB, c_y = I >= 0 && I <= NX - 1 ? ccol : OOB;
    // x weights: vx linear between faces; vy 3/4 and 1/4, mirrored at the walls
    const int nb = odd ? I + 1 : I - 1;
    const bool mirror = nb < 0 || nb >= NX;
    const double a0 = odd ? 0.5 : 1.0, a1 = odd ? 0.5 : 0.0, b0 = mirror ? 1.0 : 0.75, b1 = mirror ? 0.0 : 0.25;
    const int m0 = r0 >> 1;
    const RowSpan cs(m0 - 1, (r1 - r0 + R) / 2 + 6, cld, (int)sizeof(T));
    auto cload = [&](int jc, T& x, T& y) {
        x = buf_load_at<T>(cs.of(ex, cld, jc >= 0 && jc < NY), c_x, cs.at(jc));
        y = buf_load_at<T>(cs.of(ey, cld, jc >= 1 && jc <= NY - 1), c_y, cs.at(jc));
    };
    CoarseRows<T> c;
    T drop;
    cload(m0 - 1, c.x0, drop);
    cload(m0, c.x1, c.y1);
    cload(m0 + 1, c.x2, c.y2);
    cload(m0 + 2, c.x3, c.y3);
    walk<T, K, SQ, false, R>(
        L, r0, r1, AllCells(nx, ny, i), omega, J.idx, J.idy,
        [&](int u, int r, rows::Row<T>& w) {  // row r of w arrives: + P e_c on its unknowns
            const bool rodd = (u + K) & 1;    // y0 is even
            const int m = r >> 1;
            double s = 0.0, t = 0.0;
            {
                const int mb = rodd ? m + 1 : m - 1;
                const bool mir = mb < 0 || mb >= NY;
                const double q0 = mir ? 1.0 : 0.75, q1 = mir ? 0.0 : 0.25;
                const T e0 = c.x1, e1 = rodd ? c.x2 : c.x0;
                const T n0 = wave_shift<DPP_FROM_NEXT>(e0), n1 = wave_shift<DPP_FROM_NEXT>(e1);
                s = __builtin_fma(a0 * q0, (double)e0, s);
                s = __builtin_fma(a0 * q1, (double)e1, s);
                s = __builtin_fma(a1 * q0, (double)(odd ? n0 : T(0)), s);
                s = __builtin_fma(a1 * q1, (double)(odd ? n1 : T(0)), s);
            }
            {
                auto side = [&](T v) {
                    const T p = wave_shift<DPP_FROM_PREV>(v), q = wave_shift<DPP_FROM_NEXT>(v);
                    return odd ? q : p;
                };
                const double q0 = rodd ? 0.5 : 1.0;
                t = __builtin_fma(b0 * q0, (double)c.y1, t);
                if (rodd) t = __builtin_fma(b0 * 0.5, (double)c.y2, t);
                t = __builtin_fma(b1 * q0, (double)side(c.y1), t);
                if (rodd) t = __builtin_fma(b1 * 0.5, (double)side(c.y2), t);
            }
            w.vx = xcol && r >= 0 && r <= ny - 1 ? w.vx + T(s) : T(0);
            w.vy = ycol && r >= 1 && r <= ny - 1 ? w.vy + T(t) : T(0);
            if (rodd) {
                c.x0 = c.x1;
                c.x1 = c.x2;
                c.x2 = c.x3;
                c.y1 = c.y2;
                c.y2 = c.y3;
                cload(m + 3, c.x3, c.y3);
            }
        },
        put, [](int, int, T, T) {});
}

// Rows per wave (even), shared by the instances of a batch: the launch is modelled as
// (waves per SIMD, at least 1.2, whole ones beyond those that fit at once) x (rows
// walked, `fill` of them to fill the pipeline, in whole trips).
int fine_rows(const stk_ctx* ctx, const int* nx, const int* ny, int n, int strip_, int fill, int trip, int per_simd,
              int most) {
    const int64_t cu4 = (int64_t)std::max(ctx->num_cu, 1) * 4;
    int best = 2;
    double cost = 1e300;
    int maxny = 0;
    for (int q = 0; q < n; ++q) maxny = std::max(maxny, ny[q]);
    for (int steps = trip; steps < maxny + 2 + fill + trip; steps += trip) {
        const int H = (steps - fill) / 2 * 2;
        if (H < 2 || H > most) continue;
        int64_t waves = 0;
        for (int q = 0; q < n; ++q)
            waves += (int64_t)((nx[q] + strip_) / strip_) * ((ny[q] + H) / H);
        const double per = std::max((double)(waves + cu4 - 1) / cu4, 1.0);
        const double c = (steps + 4) * (per <= per_simd ? std::max(per, 1.2) : std::ceil(per));
        if (c < cost) {
            cost = c;
            best = H;
        }
    }
    return best;
}

template <typename T, int K, bool SQ>
int launch_fine(stk_ctx* ctx, const Batch& b, const FineShape* shapes, double omega, bool up, const FineIo& io) {
    const dim3 grid((unsigned)b.blocks), block(64 * WPB);
    if (up)
        hipLaunchKernelGGL((k_fine_up<T, K, SQ>), grid, block, 0, ctx->stream,
                           static_cast<const LevelJob<T>*>(b.jobs), b.pre, shapes, b.n, T(omega), io);
    else
        hipLaunchKernelGGL((k_fine_down<T, K, SQ>), grid, block, 0, ctx->stream,
                           static_cast<const LevelJob<T>*>(b.jobs), b.pre, shapes, b.n, T(omega), io);
    STK_HIP(hipGetLastError());
    return STK_OK;
}

}  // namespace

bool mg_fine_takes(int es, int64_t ld) { return max_rows(ld, es) >= 128; }

void mg_fine_shape(const stk_ctx* ctx, int es, const int* nx, const int* ny, const int64_t* ld, int n, int K, bool up,
                   std::vector<FineShape>* shapes, std::vector<int>* pre) {
    const int sw = up ? up_strip(K) : down_strip(K), fill = up ? 2 * K : 2 * K + 5;
    const int trip = up ? (es == 8 ? ring_rows<double>(K) : ring_rows<float>(K)) : DOWN_RING;
    int most = INT32_MAX;
    for (int q = 0; q < n; ++q) most = std::min(most, max_rows(ld[q], es) - 64);
    const int H = fine_rows(ctx, nx, ny, n, sw, fill, trip, es == 8 ? 2 : 3, most);
    shapes->clear();
    pre->assign(1, 0);
    for (int q = 0; q < n; ++q) {
        const FineShape s{(nx[q] + sw) / sw, (ny[q] + H) / H, H};
        shapes->push_back(s);
        pre->push_back(pre->back() + (int)(((int64_t)s.nstrip * s.nseg + WPB - 1) / WPB));
    }
}

template <typename T>
int mg_fine(stk_ctx* ctx, const Batch& b, const FineShape* shapes, int K, bool square, double omega, bool up,
            const FineIo& io) {
    if (!b.n) return STK_OK;
#define STK_FINE(KK)                                                                       \
    case KK:                                                                               \
        return square ? launch_fine<T, KK, true>(ctx, b, shapes, omega, up, io)            \
                      : launch_fine<T, KK, false>(ctx, b, shapes, omega, up, io);
    switch (K) {
        STK_FINE(1)
        STK_FINE(2)
        STK_FINE(3)
        default: return set_error(STK_EINVAL, "internal: %d sweeps in a fused finest-level pass", K);
    }
#undef STK_FINE
}
template int mg_fine<double>(stk_ctx*, const Batch&, const FineShape*, int, bool, double, bool, const FineIo&);
template int mg_fine<float>(stk_ctx*, const Batch&, const FineShape*, int, bool, double, bool, const FineIo&);

}  // namespace stk
