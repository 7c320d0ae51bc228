// K damped Jacobi sweeps per pass over memory (jacobi_pipe.hpp): the kernel of
// every smoother that equals plain Jacobi (Sec. 5 (ii), (iii); RAS, Sec. 4.3,
// with an overlap of at least k - 1, whose values do not depend on the tiles).
#include <algorithm>

#include "jacobi_pipe.hpp"
#include "stk_internal.hpp"

namespace stk {
namespace {

using namespace pipe;

template <typename T, int K, bool SQ>
__global__ __launch_bounds__(64 * WPB, pipe_occupancy<T>(K)) void k_jacobi_pipe(Grid<T> g, const T* __restrict__ vx,
                                                                               const T* __restrict__ vy,
                                                                               T* __restrict__ ox, T* __restrict__ oy,
                                                                               Shape sh) {
    const int wv = xcd_tile((int)blockIdx.x, (int)gridDim.x) * WPB + rows::wave_in_group();
    const int strip_ = wv % sh.nstrip, segm = wv / sh.nstrip;
    if (segm >= sh.nseg) return;  // the whole wave
    const int nx = g.nx, ny = g.ny, lane = threadIdx.x & 63;
    const int i = strip_ * strip(K) - K + lane, y0 = segm * sh.seg, y1 = min(y0 + sh.seg, ny + 1);
    const int r0 = y0 - K, r1 = y0 + sh.seg + K;
    const PipeRows<T> L(vx, vy, g.ec, g.en, g.bx, g.by, g.ld, nx, ny, i, r0, r1 - r0 + ahead<T>(), false);
    const PipeStore<T> put(ox, oy, g.ld, nx, ny, y0, y1, i, lane >= K && lane < 64 - K);
    walk<T, K, SQ, false, ring_rows<T>(K)>(L, r0, r1, AllCells(nx, ny, i), g.omega, g.idx, g.idy,
                                           [](int, int, rows::Row<T>&) {}, put, [](int, int, T, T) {});
}

// Launch shape: about w waves per SIMD, w = 1, 2, ..., each a segment of equal
// rows (rounded so that the walk is a whole number of unrolled trips).  The
// waves of a SIMD share its issue slots, so a launch takes about (waves per
// SIMD) x (rows walked + 2K rows that fill the pipeline); a single wave leaves
// some of them unused (FP64 x 1.1, FP32 x 1.35: 2048^2, K = 7, one or two
// waves per SIMD, 69 / 66 us and 56 / 45 us).  *us: that time.
template <typename T>
Shape pipe_shape(const stk_ctx* ctx, int nx, int ny, int64_t ld, int K, double* us) {
    const int U = ring_rows<T>(K);
    const int64_t ns = (nx + 1 + strip(K) - 1) / strip(K), cu4 = (int64_t)std::max(ctx->num_cu, 1) * 4;
    Shape best{K, (int)ns, 0, 0};
    double cost = 1e300;
    for (int w = 1; w <= pipe_occupancy<T>(K); ++w) {
        const int64_t most = max_rows(ld, (int)sizeof(T)) - 2 * K;  // rows of a segment that a window can address
        const int64_t segs = std::max<int64_t>((ny + most) / most, std::min<int64_t>(w * cu4 / ns, ny + 1));
        const int steps = ((int)((ny + 1 + segs - 1) / segs) + 2 * K + U - 1) / U * U, H = steps - 2 * K;
        const int64_t nseg = (ny + 1 + H - 1) / H, per_simd = (ns * nseg + cu4 - 1) / cu4;
        const double c = (steps + 4) * std::max(sizeof(T) == 8 ? 1.1 : 1.35, (double)per_simd);
        if (c < cost) {
            cost = c;
            best.nseg = (int)nseg;
            best.seg = H;
        }
    }
    if (us) *us = cost * step_us<T>(K);
    return best;
}

// Sweeps per pass for `left` sweeps in all: the count whose passes, equal in
// size, take the least time.  A pass takes the longest of its steps and its
// eight planes at 5 TB/s (measured 4.6 to 5.0), and 3 us between launches.
// FP64 stops at 7, where two waves per SIMD still fit their registers (8: one
// wave, 283 us against 247 us for 7 at 4096^2, no faster per sweep), FP32 at 10.
template <typename T>
int pick_sweeps(const stk_ctx* ctx, const stk_grid* g, int left) {
    const int kmax = sizeof(T) == 8 ? 7 : 10;
    const double mem = 8.0 * sizeof(T) * g->nx * g->ny / 5e6;
    int best = 1, last = 0;
    double cost = 1e300;
    for (int m = (left + kmax - 1) / kmax; m <= left; ++m) {
        const int K = (left + m - 1) / m;
        if (K == last) continue;
        last = K;
        double us = 0.0;
        pipe_shape<T>(ctx, g->nx, g->ny, g->ld, K, &us);
        const double c = m * (std::max(us, mem) + 3.0);
        if (c < cost) {
            cost = c;
            best = K;
        }
        if (K == 1) break;
    }
    return best;
}

template <typename T, int K>
int launch_k(stk_ctx* ctx, const Grid<T>& g, const T* vx, const T* vy, T* ox, T* oy) {
    const Shape sh = pipe_shape<T>(ctx, g.nx, g.ny, g.ld, K, nullptr);
    const dim3 grid((unsigned)(((int64_t)sh.nstrip * sh.nseg + WPB - 1) / WPB)), block(64 * WPB);
    if (g.idx == g.idy)
        hipLaunchKernelGGL((k_jacobi_pipe<T, K, true>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, sh);
    else
        hipLaunchKernelGGL((k_jacobi_pipe<T, K, false>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, sh);
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
    switch (K) {
        case 1: return launch_k<T, 1>(ctx, gg, a, b, c, d);
        case 2: return launch_k<T, 2>(ctx, gg, a, b, c, d);
        case 3: return launch_k<T, 3>(ctx, gg, a, b, c, d);
        case 4: return launch_k<T, 4>(ctx, gg, a, b, c, d);
        case 5: return launch_k<T, 5>(ctx, gg, a, b, c, d);
        case 6: return launch_k<T, 6>(ctx, gg, a, b, c, d);
        case 7: return launch_k<T, 7>(ctx, gg, a, b, c, d);
        case 8: return launch_k<T, 8>(ctx, gg, a, b, c, d);
        case 9: return launch_k<T, 9>(ctx, gg, a, b, c, d);
        case 10: return launch_k<T, 10>(ctx, gg, a, b, c, d);
        default: return set_error(STK_EINVAL, "internal: %d sweeps in one pass", K);
    }
}

}  // namespace

bool jacobi_pipe_takes(stk_dtype dt, const stk_grid* g) {
    return pipe::max_rows(g->ld, (int)elem_size(dt)) >= 128 && g->ny < INT32_MAX - 4096;
}

int jacobi_pipe_sweeps(const stk_ctx* ctx, stk_dtype dt, const stk_grid* g, int left) {
    return dt == STK_F64 ? pick_sweeps<double>(ctx, g, left) : pick_sweeps<float>(ctx, g, left);
}

// As ras_pipe_us (2 x 2 to 300 x 300, k = 6 to 10: within 12 and 9 %).
double jacobi_pipe_us(const stk_ctx* ctx, stk_dtype dt, const stk_grid* g, int sweeps) {
    double us = 0.0;
    if (dt == STK_F64) {
        pipe_shape<double>(ctx, g->nx, g->ny, g->ld, sweeps, &us);
        return 0.3 + 1.1 * us;
    }
    pipe_shape<float>(ctx, g->nx, g->ny, g->ld, sweeps, &us);
    return 3.6 + 0.93 * us;
}

int launch_jacobi_pipe(stk_ctx* ctx, stk_dtype dt, const stk_grid* g, const FieldPtrs& f, double omega, int sweeps,
                       const void* vx, const void* vy, void* ox, void* oy) {
    return dt == STK_F64 ? launch_t<double>(ctx, g, f, omega, sweeps, vx, vy, ox, oy)
                         : launch_t<float>(ctx, g, f, omega, sweeps, vx, vy, ox, oy);
}

}  // namespace stk
