// RAS outer iterations with a thin overlap (h < k - 1) on the register pipeline of
// jacobi_pipe.hpp: what lies outside a tile's grown window keeps its value through the
// sweeps, as the walls do, so a frozen row or column is one that is not relaxed.
//
// The walk runs over stretched columns and rows: the windows of the tiles with their
// frozen rings, T + 2 h + 2 each, one after the other, so that a column or row near a cut
// appears once in every window that holds it, and neighbouring positions of one window
// are neighbours in the grid.  The first and last position of a window are frozen and
// take nothing from the window beside it.  Strips and segments are then cut as for
// Jacobi, wherever they fall: of its 64 positions a wave loses K on either side, and the
// grid is (T + 2 h + 2) / T longer each way.
//
// What bounds it: vector issue, as for Jacobi, with the stretched cells on top; from
// about 4096^2 on, the eight planes.  One pass of k = 4 sweeps on 64 x 64 tiles without
// overlap, before (an LDS pipeline with one wave per level) and now: 1501 x 1100 FP32
// 32.1 -> 19.9 us, FP64 41.5 -> 27.0; 4096^2 FP32 186 -> 127, FP64 268 -> 238 us.  On
// 16 x 16 tiles at 4096^2 FP32 562 -> 137 us; 128 x 128 (one tile per workgroup's LDS)
// 2.57 ms -> 125 us.
#include <algorithm>

#include "jacobi_pipe.hpp"
#include "stk_internal.hpp"

namespace stk {
namespace {

using namespace pipe;

// Waves per SIMD the registers must leave room for; the selects and the windows' bounds
// take more of them than the Jacobi passes do.
template <typename T>
constexpr int ras_occupancy(int K) { return sizeof(T) == 8 ? (K <= 3 ? 3 : K <= 6 ? 2 : 1) : K <= 4 ? 4 : K <= 6 ? 3 : 2; }

// One direction, stretched: position e of tile t = e / P is grid index t T + base + e % P.
struct Stretch {
    int P, T, h, base;
    unsigned magic;  // ceil(2^32 / P): e / P is the high half of e magic while e P < 2^32
    __host__ __device__ __forceinline__ int tile(int e) const {
        return (int)(((uint64_t)(unsigned)e * magic) >> 32);
    }
    // grid index of e, o: its place in the window
    __host__ __device__ __forceinline__ int at(int e, int& o) const {
        const int t = tile(e);
        o = e - t * P;
        return t * T + base + o;
    }
    __host__ __device__ __forceinline__ bool relaxed(int o) const { return o >= 1 && o <= P - 2; }
    __host__ __device__ __forceinline__ bool owned(int o) const { return o > h && o <= h + T; }
    // the first position that owns index 0 or more, and one past the last that owns n or less
    __host__ __device__ __forceinline__ int first() const { return -base; }
    __host__ int end(int n) const { return (n - base - h - 1) / T * P + (n - base - h - 1) % T + h + 2; }
};

struct RasCut {
    Stretch x, y;
    int e0x, e0y, e1y, nstrip, nseg, seg;
};

// Rows of the walk: PipeRows of the grid rows behind the stretched ones.
template <typename T>
struct RasRows {
    PipeRows<T> rows;
    Stretch y;
    __device__ __forceinline__ rows::Row<T> load(int e) const {
        int o;
        return rows.load(y.at(max(e, 0), o));
    }
};
struct RasCells {
    static constexpr bool SELECT = true;  // the windows lie side by side
    bool x, y;
    int ny;
    Stretch s;
    __device__ __forceinline__ bool row_x(int e) const {
        int o;
        const int j = s.at(max(e, 0), o);
        return s.relaxed(o) && j >= 0 && j <= ny - 1;
    }
    __device__ __forceinline__ bool row_y(int e) const {
        int o;
        const int j = s.at(max(e, 0), o);
        return s.relaxed(o) && j >= 1 && j <= ny - 1;
    }
};

template <typename T, int K, bool SQ>
__global__ __launch_bounds__(64 * WPB, ras_occupancy<T>(K)) void k_ras_pipe(Grid<T> g, const T* __restrict__ vx,
                                                                           const T* __restrict__ vy,
                                                                           T* __restrict__ ox, T* __restrict__ oy,
                                                                           RasCut c) {
    const int wv = xcd_tile((int)blockIdx.x, (int)gridDim.x) * WPB + rows::wave_in_group();
    const int strip_ = wv % c.nstrip, segm = wv / c.nstrip;
    if (segm >= c.nseg) return;  // the whole wave
    const int nx = g.nx, ny = g.ny, lane = threadIdx.x & 63;
    const int ex = c.e0x + strip_ * strip(K) - K + lane;
    int o;
    const int i = c.x.at(max(ex, 0), o);
    const int ea = c.e0y + segm * c.seg, eb = min(ea + c.seg, c.e1y), e0 = ea - K, e1 = ea + c.seg + K;
    int oy0;
    const int low = c.y.at(max(e0, 0), oy0) - 2 * c.y.h - 2;  // no row of the walk is lower
    const RasRows<T> L{PipeRows<T>(vx, vy, g.ec, g.en, g.bx, g.by, g.ld, nx, ny, i, low,
                                   e1 - e0 + ahead<T>() + 2 * c.y.h + 3, false),
                       c.y};
    const bool own = lane >= K && lane < 64 - K && c.x.owned(o) && i >= 0;
    const PipeStore<T> st(ox, oy, g.ld, nx, ny, low, low + e1 - e0 + 2 * c.y.h + 3, i, own);
    const bool in = ex >= 0 && c.x.relaxed(o);
    const RasCells relax{in && i >= 1 && i <= nx - 1, in && i >= 0 && i <= nx - 1, ny, c.y};
    walk<T, K, SQ, false, ring_rows<T>(K)>(
        L, e0, e1, relax, g.omega, g.idx, g.idy, [](int, int, rows::Row<T>&) {},
        [&](int e, T ux, T uy) {
            int oj;
            const int j = c.y.at(max(e, 0), oj);
            st.store(j, e >= ea && e < eb && c.y.owned(oj) && j >= 0 && j <= ny, ux, uy);
        },
        [](int, int, T, T) {});
}

Stretch stretch(int T, int h, int s) {
    const int P = T + 2 * h + 2;
    return {P, T, h, s - T - h - 1, (unsigned)((((uint64_t)1 << 32) + P - 1) / P)};
}

// Strips and segments, as pipe_shape (jacobi_pipe.hip); a wave alone on its SIMD also waits
// for the scalar arithmetic of the stretched rows (FP64 k = 4, 64 x 64 tiles, one and two
// waves per SIMD: 1501 x 1100 30.4 and 27.0 us, 2048^2 57 and 52 us).
// *us: the modelled time, as there.
template <typename T>
RasCut ras_cut(const stk_ctx* ctx, const stk_grid* g, int Tx, int Ty, int h, int K, int sx, int sy, double* us) {
    RasCut c{stretch(Tx, h, sx), stretch(Ty, h, sy), 0, 0, 0, 0, 0, 0};
    c.e0x = c.x.first();
    c.e0y = c.y.first();
    c.e1y = c.y.end(g->ny);
    const int U = ring_rows<T>(K), ex = c.x.end(g->nx) - c.e0x, ey = c.e1y - c.e0y;
    const int64_t ns = (ex + strip(K) - 1) / strip(K), cu4 = (int64_t)std::max(ctx->num_cu, 1) * 4;
    const int64_t most = max_rows(g->ld, (int)sizeof(T)) - 2 * K - 2 * h - 3;
    c.nstrip = (int)ns;
    double cost = 1e300;
    for (int w = 1; w <= ras_occupancy<T>(K); ++w) {
        const int64_t segs = std::max<int64_t>((ey + most - 1) / most, std::min<int64_t>(w * cu4 / ns, ey));
        const int steps = ((int)((ey + segs - 1) / segs) + 2 * K + U - 1) / U * U, H = steps - 2 * K;
        const int64_t nseg = (ey + H - 1) / H, per_simd = (ns * nseg + cu4 - 1) / cu4;
        const double t = (steps + 4) * std::max(1.35, (double)per_simd);
        if (t < cost) {
            cost = t;
            c.nseg = (int)nseg;
            c.seg = H;
        }
    }
    if (us) *us = cost * step_us<T>(K);
    return c;
}

template <typename T, int K>
int launch_k(stk_ctx* ctx, const Grid<T>& g, const RasCut& c, const T* vx, const T* vy, T* ox, T* oy) {
    const dim3 grid((unsigned)(((int64_t)c.nstrip * c.nseg + WPB - 1) / WPB)), block(64 * WPB);
    if (g.idx == g.idy)
        hipLaunchKernelGGL((k_ras_pipe<T, K, true>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, c);
    else
        hipLaunchKernelGGL((k_ras_pipe<T, K, false>), grid, block, 0, ctx->stream, g, vx, vy, ox, oy, c);
    STK_HIP(hipGetLastError());
    return STK_OK;
}

template <typename T>
int launch_t(stk_ctx* ctx, const stk_grid* g, const FieldPtrs& f, double omega, int Tx, int Ty, int h, int K, int sx,
             int sy, const void* vx, const void* vy, void* ox, void* oy) {
    const Grid<T> gg{static_cast<const T*>(f.eta_c), static_cast<const T*>(f.eta_n), static_cast<const T*>(f.bx),
                     static_cast<const T*>(f.by), g->ld, g->nx, g->ny, T(1.0 / g->dx), T(1.0 / g->dy), T(omega)};
    const RasCut cut = ras_cut<T>(ctx, g, Tx, Ty, h, K, sx, sy, nullptr);
    const T *a = static_cast<const T*>(vx), *b = static_cast<const T*>(vy);
    T *c = static_cast<T*>(ox), *d = static_cast<T*>(oy);
    switch (K) {
        case 2: return launch_k<T, 2>(ctx, gg, cut, a, b, c, d);
        case 3: return launch_k<T, 3>(ctx, gg, cut, a, b, c, d);
        case 4: return launch_k<T, 4>(ctx, gg, cut, a, b, c, d);
        case 5: return launch_k<T, 5>(ctx, gg, cut, a, b, c, d);
        case 6: return launch_k<T, 6>(ctx, gg, cut, a, b, c, d);
        case 7: return launch_k<T, 7>(ctx, gg, cut, a, b, c, d);
        case 8: return launch_k<T, 8>(ctx, gg, cut, a, b, c, d);
        case 9: return launch_k<T, 9>(ctx, gg, cut, a, b, c, d);
        case 10: return launch_k<T, 10>(ctx, gg, cut, a, b, c, d);
        default: return set_error(STK_EINVAL, "internal: %d sweeps in one pass", K);
    }
}

}  // namespace

bool ras_pipe_takes(const stk_ctx* ctx, stk_dtype dt, const stk_grid* g, int tile_x, int tile_y, int halo, int kt) {
    if (kt < 2 || kt > PIPE_MAX_SWEEPS || halo >= kt - 1 || !jacobi_pipe_takes(dt, g)) return false;
    // positions (Stretch): at most n (T + 2 h + 2) / T + 2 (T + 2 h + 2) of them
    auto fits = [&](int n, int T) {
        const int64_t P = (int64_t)T + 2 * halo + 2;
        return ((n / T + 4) * P + 4096) * P < ((int64_t)1 << 32);
    };
    return fits(g->nx, tile_x) && fits(g->ny, tile_y);
}

// A pass's time on an idle chip, from the modelled steps (2 to 200 tiles of 8 to 64, k = 6 to
// 10: FP64 within 9 % of the measured one in nine of ten cases, FP32 within 8 %).
double ras_pipe_us(const stk_ctx* ctx, stk_dtype dt, const stk_grid* g, int tile_x, int tile_y, int halo, int kt) {
    double us = 0.0;
    if (dt == STK_F64) {
        ras_cut<double>(ctx, g, tile_x, tile_y, halo, kt, 0, 0, &us);
        return 0.3 + 1.16 * us;
    }
    ras_cut<float>(ctx, g, tile_x, tile_y, halo, kt, 0, 0, &us);
    return 3.0 + 1.35 * us;
}

int launch_ras_pipe(stk_ctx* ctx, stk_dtype dt, const stk_grid* g, const FieldPtrs& f, double omega, int tile_x,
                    int tile_y, int halo, int kt, int sx, int sy, const void* vx, const void* vy, void* ox, void* oy) {
    return dt == STK_F64 ? launch_t<double>(ctx, g, f, omega, tile_x, tile_y, halo, kt, sx, sy, vx, vy, ox, oy)
                         : launch_t<float>(ctx, g, f, omega, tile_x, tile_y, halo, kt, sx, sy, vx, vy, ox, oy);
}

}  // namespace stk
