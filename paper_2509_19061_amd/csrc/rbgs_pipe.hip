// Red-black Gauss-Seidel, K sweeps per pass over memory: the four half-sweeps of
// each sweep (vx red, vx black, vy red, vy black) pipelined in registers, as the
// Jacobi sweeps of jacobi_pipe.hpp are.
//
// A wave walks up the rows of its strip.  When row b of a sweep's input is there,
// vx red is relaxed at row b - 1, vx black and vy red at row b - 2 and vy black at
// row b - 3, each in place in a ring of rows; row b - 3 is then row b of the next
// sweep.  A half-sweep relaxes every other lane and selects: the lanes of the other
// colour keep their value.  The differences that both colours need are formed once:
// d(j) = vy(j) - vy(j) of the column before, of the sweep's input, for vx, and
// e(j) = vx(j) - vx(j - 1) of the relaxed vx for vy.  Values are bit for bit those of
// k_rbgs.
//
// Exact rows and columns shrink by 3 a sweep and one more for the last vy row below
// and column to the right: of its 64 columns a wave owns 63 - 6 K, and its walk
// takes 6 K + 1 rows more than it owns.
//
// What bounds it: k_rbgs takes four launches a sweep, each reading nearly all eight
// planes (1001 x 1203 FP64, which the last-level cache holds: 10.4 us each); a pass
// here reads them once for K sweeps and is bound by vector issue (about 200
// instructions a row for K = 2) and, on small grids, by the walk's 6 K + 1 extra rows.
// Ten sweeps: 64^2 FP64 117 -> 57 us; 1001 x 1203 418 -> 140 us, FP32 268 -> 116 us;
// 4096^2 FP64 6.3 -> 1.25 ms, FP32 3.65 -> 0.66 ms.  Three sweeps a pass would need more
// than the 256 registers that two waves per SIMD have in FP64 (222 for two).
#include <algorithm>

#include "jacobi_pipe.hpp"
#include "stk_internal.hpp"

namespace stk {
namespace {

using namespace pipe;

constexpr int KMAX = 2;
__host__ __device__ constexpr int rb_strip(int K) { return 63 - 6 * K; }
// ring of rows and steps per unrolled trip: even (the colours alternate by renaming)
template <typename T>
constexpr int rb_ring(int K) { return (3 * K + 1 + ahead<T>()) / ahead<T>() * ahead<T>(); }
// Waves per SIMD the registers must leave room for.
template <typename T>
constexpr int rb_occupancy(int K) { return sizeof(T) == 8 ? 2 : K == 1 ? 4 : 3; }

// The relaxed value n in the lanes that take it, if row j is one of lo .. hi.  n is
// opaque, or the compiler turns the select into a branch around its whole half-sweep and
// the steps into many blocks; j is, or it keeps the rows' masks in scalar registers from
// one half-sweep to the next and spills them.
template <typename T>
__device__ __forceinline__ T take_rows(bool take, int j, int lo, int hi, T n, T v) {
    asm volatile("" : "+v"(n), "+s"(j));
    return take & (j >= lo) & (j <= hi) ? n : v;
}

template <typename T>
struct RbCoef {
    T A, N, bx, by, gx, gy;
};

template <typename T, int K, bool SQ>
__global__ __launch_bounds__(64 * WPB, rb_occupancy<T>(K)) void k_rbgs_pipe(Grid<T> g, const T* __restrict__ pvx,
                                                                           const T* __restrict__ pvy,
                                                                           T* __restrict__ ox, T* __restrict__ oy,
                                                                           Shape sh) {
    constexpr int PFD = ahead<T>(), R = rb_ring<T>(K);
    static_assert(R >= 3 * K + 2 && R % PFD == 0 && R % 2 == 0, "ring");
    const int wv = xcd_tile((int)blockIdx.x, (int)gridDim.x) * WPB + rows::wave_in_group();
    const int strip_ = wv % sh.nstrip, segm = wv / sh.nstrip;
    if (segm >= sh.nseg) return;  // the whole wave
    const int nx = g.nx, ny = g.ny, lane = threadIdx.x & 63;
    const int i = strip_ * rb_strip(K) - 3 * K + lane, y0 = segm * sh.seg, y1 = min(y0 + sh.seg, ny + 1);
    const int r0 = y0 - 3 * K - 1, r1 = y0 + sh.seg + 3 * K;
    const PipeRows<T> L(pvx, pvy, g.ec, g.en, g.bx, g.by, g.ld, nx, ny, i, r0, r1 - r0 + PFD, false);
    const PipeStore<T> put(ox, oy, g.ld, nx, ny, y0, y1, i, lane >= 3 * K && lane < 63 - 3 * K);

    const bool odd = (i + r0) & 1, xcol = i >= 1 && i <= nx - 1, ycol = i >= 0 && i <= nx - 1;
    const bool xp[2] = {xcol && !odd, xcol && odd}, yp[2] = {ycol && !odd, ycol && odd};
    const Scale<T> sv = stencil_scale(g.idx, g.idy);
    const Scale<T> sc{wave_uniform(sv.a), wave_uniform(sv.n), wave_uniform(sv.kap), wave_uniform(sv.ry),
                      wave_uniform(sv.rx)};
    T vx[R], vy[R], d[K][R], e[K][R], er[K][R];
    RbCoef<T> cf[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        vx[q] = vy[q] = T(0);
        cf[q] = RbCoef<T>{T(0), T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int s = 0; s < K; ++s) d[s][q] = e[s][q] = er[s][q] = T(0);
    }
    rows::Row<T> q[PFD];
#pragma unroll
    for (int p = 0; p < PFD; ++p) q[p] = L.load(r0 + p);
    for (int rb = r0; rb < r1; rb += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int r = rb + u;
            const rows::Row<T> w = q[u % PFD];
            q[u % PFD] = L.load(r + PFD);
            if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);  // as in jacobi_pipe.hpp
            auto at = [&](int t) { return (u + 4 * R - t) % R; };   // slot of row r - t
            RbCoef<T>& c0 = cf[u];
            RbCoef<T>& c1 = cf[at(1)];
            vx[u] = w.vx;
            vy[u] = w.vy;
            c0.A = coef_a(w.ec, sc);
            c0.N = coef_n(w.en, sc);
            c0.bx = w.bx;
            c0.by = w.by;
            {  // the factors of row r - 1, whose upper shear coefficient is now here
                const T aL = wave_shift<DPP_FROM_PREV>(c1.A), nR = wave_shift<DPP_FROM_NEXT>(c1.N);
                const T Ab = cf[at(2)].A;
                c1.gx = jac_factor(g.omega, SQ ? (c1.N + c0.N) + (aL + c1.A) : diagx_scaled<T>(aL, c1.A, c1.N, c0.N, sc.ry));
                c1.gy = jac_factor(g.omega, SQ ? (c1.N + nR) + (Ab + c1.A)
                                               : diagy_scaled<T>(coef_b(Ab, sc), coef_b(c1.A, sc), c1.N, nR, sc.rx));
            }
#pragma unroll
            for (int s = 0; s < K; ++s) {
                const int b = 3 * s;  // this sweep's input row is r - b
                // vx of colour c at row r - t
                auto relax_x = [&](int c, int t) {
                    const int j = r - t;
                    const RbCoef<T>& C = cf[at(t)];
                    T& v = vx[at(t)];
                    const T ex = wave_shift<DPP_FROM_NEXT>(v) - v, exl = wave_shift<DPP_FROM_PREV>(ex);
                    const T up = vx[at(t - 1)] - v, dn = v - vx[at(t + 1)];
                    T m = C.A * ex;
                    m = fmaT(-wave_shift<DPP_FROM_PREV>(C.A), exl, m);
                    m = fmaT(cf[at(t - 1)].N, SQ ? up + d[s][at(t - 1)] : fmaT(sc.ry, up, d[s][at(t - 1)]), m);
                    m = fmaT(-C.N, SQ ? dn + d[s][at(t)] : fmaT(sc.ry, dn, d[s][at(t)]), m);
                    v = take_rows(xp[(c + u + t) & 1], j, 0, ny - 1, jac_step<T>(v, C.gx, C.bx, m), v);
                };
                // vy of colour c at row r - t
                auto relax_y = [&](int c, int t) {
                    const int j = r - t;
                    const RbCoef<T>& C = cf[at(t)];
                    T& v = vy[at(t)];
                    const T rt = wave_shift<DPP_FROM_NEXT>(v) - v, lt = wave_shift<DPP_FROM_PREV>(rt);
                    const T up = vy[at(t - 1)] - v, dn = v - vy[at(t + 1)];
                    T B = C.A, Bb = cf[at(t + 1)].A;
                    if (!SQ) {  // an opaque kap: B is formed where it is used, not held for the ring's rows
                        Scale<T> sk = sc;
                        asm volatile("" : "+s"(sk.kap));
                        B = coef_b(B, sk);
                        Bb = coef_b(Bb, sk);
                    }
                    T m = B * up;
                    m = fmaT(-Bb, dn, m);
                    m = fmaT(wave_shift<DPP_FROM_NEXT>(C.N), SQ ? rt + er[s][at(t)] : fmaT(sc.rx, rt, er[s][at(t)]), m);
                    m = fmaT(-C.N, SQ ? lt + e[s][at(t)] : fmaT(sc.rx, lt, e[s][at(t)]), m);
                    v = take_rows(yp[(c + u + t) & 1], j, 1, ny - 1, jac_step<T>(v, C.gy, C.by, m), v);
                };
                d[s][at(b)] = vy[at(b)] - wave_shift<DPP_FROM_PREV>(vy[at(b)]);
                relax_x(0, b + 1);
                relax_x(1, b + 2);
                e[s][at(b + 2)] = vx[at(b + 2)] - vx[at(b + 3)];
                er[s][at(b + 2)] = wave_shift<DPP_FROM_NEXT>(e[s][at(b + 2)]);
                relax_y(0, b + 2);
                relax_y(1, b + 3);
            }
            put(r - 3 * K, vx[at(3 * K)], vy[at(3 * K)]);
        }
    }
}

// Launch shape, as pipe_shape (jacobi_pipe.hip): w waves per SIMD, w = 1, 2, ..., each a
// segment of equal rows, where a wave alone on its SIMD leaves issue slots unused.
template <typename T>
Shape rb_shape(const stk_ctx* ctx, int nx, int ny, int64_t ld, int K) {
    const int U = rb_ring<T>(K), over = 6 * K + 1;
    const int64_t ns = (nx + 1 + rb_strip(K) - 1) / rb_strip(K), cu4 = (int64_t)std::max(ctx->num_cu, 1) * 4;
    Shape best{K, (int)ns, 0, 0};
    double cost = 1e300;
    for (int w = 1; w <= rb_occupancy<T>(K); ++w) {
        const int64_t most = max_rows(ld, (int)sizeof(T)) - over;  // rows of a segment that a window can address
        const int64_t segs = std::max<int64_t>((ny + most) / most, std::min<int64_t>(w * cu4 / ns, ny + 1));
        const int steps = ((int)((ny + 1 + segs - 1) / segs) + over + U - 1) / U * U, H = steps - over;
        const int64_t nseg = (ny + 1 + H - 1) / H, per_simd = (ns * nseg + cu4 - 1) / cu4;
        const double c = (steps + 4) * std::max(sizeof(T) == 8 ? 1.2 : 1.35, (double)per_simd);
        if (c < cost) {
            cost = c;
            best.nseg = (int)nseg;
            best.seg = H;
        }
    }
    return best;
}

template <typename T, int K>
int launch_k(stk_ctx* ctx, const Grid<T>& g, const T* vx, const T* vy, T* ox, T* oy) {
    const Shape sh = rb_shape<T>(ctx, g.nx, g.ny, g.ld, K);
    const dim3 grid((unsigned)(((int64_t)sh.nstrip * sh.nseg + WPB - 1) / WPB)), block(64 * WPB);
    if (g.idx == g.idy)
        hipLaunchKernelGGL((k_rbgs_pipe<T, K, true>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, sh);
    else
        hipLaunchKernelGGL((k_rbgs_pipe<T, K, false>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, sh);
    STK_HIP(hipGetLastError());
    return STK_OK;
}

template <typename T>
int launch_t(stk_ctx* ctx, const stk_grid* g, const FieldPtrs& f, double omega, int K, const void* vx, const void* vy,
             void* ox, void* oy) {
    const Grid<T> gg{static_cast<const T*>(f.eta_c), static_cast<const T*>(f.eta_n), static_cast<const T*>(f.bx),
                     static_cast<const T*>(f.by), g->ld, g->nx, g->ny, T(1.0 / g->dx), T(1.0 / g->dy), T(omega)};
    const T *a = static_cast<const T*>(vx), *b = static_cast<const T*>(vy);
    T *c = static_cast<T*>(ox), *d = static_cast<T*>(oy);
    return K == 1 ? launch_k<T, 1>(ctx, gg, a, b, c, d) : launch_k<T, KMAX>(ctx, gg, a, b, c, d);
}

}  // namespace

int rbgs_pipe_sweeps(int left) { return std::min(left, KMAX); }

int launch_rbgs_pipe(stk_ctx* ctx, stk_dtype dt, const stk_grid* g, const FieldPtrs& f, double omega, int sweeps,
                     const void* vx, const void* vy, void* ox, void* oy) {
    return dt == STK_F64 ? launch_t<double>(ctx, g, f, omega, sweeps, vx, vy, ox, oy)
                         : launch_t<float>(ctx, g, f, omega, sweeps, vx, vy, ox, oy);
}

}  // namespace stk
