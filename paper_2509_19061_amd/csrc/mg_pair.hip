// Two applications of a stored Galerkin stencil in one pass: on the way down a
// coarse level's second pre-smoothing sweep and its residual, on the way up the
// prolongation and both post-smoothing sweeps.
//
// A level's stored stencil is four fifths of the bytes of a sweep (32 planes
// against 6 of vectors), and on the small levels a launch costs more than its
// bytes; applied separately, each of the four passes of a V(2, 2)-cycle reads
// the planes again.  Here a workgroup takes a region of RX x RY positions.  Each
// of its threads owns one row of the operator (a position and a component),
// loads its 31 coefficients once and keeps them in registers for both
// applications; the velocities are staged in LDS.  The first application is
// computed on the whole region, into a second window, the second on the region
// without its two-cell rim, which is what the workgroup owns.
//
// Why these regions: with the coefficients (62 VGPRs in FP64) at most 128 VGPRs
// a thread allow 16 waves per CU, 512 positions.  A region of 32 x 16 owns 66 %
// of its positions (64 x 8 would own 47 %) and takes about 10 us, however few
// there are; one of 16 x 16 owns 56 % and takes 7.5 us, so it serves levels whose
// regions all run at once (a 128^2 level: 8.3 against 10.9 us; 256^2: 13.4
// against 12.0; 1024^2: 144 against 136).  The rim's coefficients are the
// neighbours' own and come from L2.  The large levels are bound by the sum of
// what a region does in turn: L1 accesses for the coefficients, LDS reads and
// the row sums.
//
// The row sums run in the slot order of stencil_av_l on the same operands, and
// the updates are the shared ones, so the values are the bits of the separate
// kernels.
#include <algorithm>

#include "coarse_stencil.hpp"
#include "mg_internal.hpp"
#include "mg_transfer.hpp"
#include "wave.hpp"

namespace stk {
namespace {

constexpr int RIM = 2;  // reach of the stencil
constexpr int RY = 16, OY = RY - 2 * RIM, WY = RY + 2 * RIM;  // region, owned and first window rows
constexpr int RX_WIDE = 32, RX_SMALL = 16;
constexpr int DIAG[2] = {7, 23};                      // slots of the diagonals
static_assert(offset_slot(0, 0, 0, 0) == DIAG[0] && offset_slot(1, 1, 0, 0) == DIAG[1], "diagonal slots");

__device__ __forceinline__ int find_pair_inst(const int* __restrict__ pre, int n, int b) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The 31 coefficients of row (A, i, j).  Planes are read through buffer
// resources of one plane: a neighbour above or below the box is out of its
// range and reads 0; one left or right of it is in the padding or in column
// nx (the host requires ld >= nx + 2), which hold 0.  in = false: no loads.
template <typename T, int A>
__device__ __forceinline__ void load_row(const LevelJob<T>& J, int i, int j, bool in, T (&cf)[NCOEF]) {
    const unsigned es = sizeof(T), size = (unsigned)((J.ny + 1) * J.ld) * es;
    const int at = (int)(((int64_t)j * J.ld + i) * es);
#pragma unroll
    for (int q = 0; q < NCOEF; ++q) {
        const SlotSrc s = slot_src(A, q);
        const int off = at + (s.ndy * (int)J.ld + s.ndx) * (int)es;
        cf[q] = buf_load<T>(buf_rsrc((const T*)(J.st + s.plane * J.plane), size), in ? (unsigned)off : OOB);
    }
}
// (A v) of the row at window element `e` of component planes of `stride` and
// row length W: the slot order of stencil_av_l.
template <typename T, int A, int W>
__device__ __forceinline__ T row_sum(const T (&cf)[NCOEF], const T* win, int stride, int e) {
    T s = T(0);
#pragma unroll
    for (int q = 0; q < NCOEF; ++q) {
        const T v = win[slot_comp(A, q) * stride + e + slot_dy(A, q) * W + slot_dx(A, q)];
        s += cf[q] * v;
    }
    return s;
}

// UP = false: v holds the first sweep; w <- the second, r <- its residual.
// UP = true: v <- two sweeps of w + P e_c.
// REST (down): the residual is restricted here as well and not stored.  A coarse unknown
// takes fine values from one position below its own pair to one above, so a region owns two
// positions less each way, REST_X x REST_Y at an even start: worth it where the regions
// still run all at once (128^2 FP64: 8.5 us for 7.2 and the restriction's 4.5, and a launch;
// V-cycle 1280 x 960 FP32 165 -> 159.5 us).
constexpr int REST_X = RX_SMALL - 2 * RIM - 2, REST_Y = RY - 2 * RIM - 2;

template <typename T, bool UP, int RX, bool REST>
__global__ __launch_bounds__(2 * RX * RY, REST ? 2 : 4) void k_mg_pair(const LevelJob<T>* __restrict__ jobs,
                                                            const int* __restrict__ pre, int n, T omega) {
    constexpr int NPOS = RX * RY, NTH = 2 * NPOS, WX = RX + 2 * RIM, LOW = REST ? RIM + 1 : RIM;
    constexpr int OX = REST ? REST_X : RX - 2 * RIM, OYR = REST ? REST_Y : OY;  // owned, from LOW on
    static_assert(!REST || (!UP && RX == RX_SMALL), "the restricting form");
    __shared__ T win[2 * WX * WY], mid[2 * NPOS];
    const int b = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int inst = find_pair_inst(pre, n, b);
    const LevelJob<T>& J = jobs[inst];
    const int nx = J.nx, ny = J.ny, lb = b - pre[inst], ntx = (nx + 1 + OX - 1) / OX;
    const int i0 = (lb % ntx) * OX - LOW, j0 = (lb / ntx) * OYR - LOW;  // position of region element (0, 0)
    const int64_t ld = J.ld;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int comp = wave / (NPOS / 64), e = (int)threadIdx.x & (NPOS - 1), x = e % RX, y = e / RX;
    const int i = i0 + x, j = j0 + y;
    const bool unk = comp == 0 ? is_vx_unknown(nx, ny, i, j) : is_vy_unknown(nx, ny, i, j);
    const int64_t k = (int64_t)j * ld + i;
    T cf[NCOEF];
    if (comp == 0) load_row<T, 0>(J, i, j, unk, cf);
    else load_row<T, 1>(J, i, j, unk, cf);
    const T rhs = unk ? (comp == 0 ? J.bx : J.by)[k] : T(0);
    // REST: the coarse unknown of this thread and its diagonal
    constexpr int CX = REST_X / 2, CY = REST_Y / 2;
    const int cc = (int)threadIdx.x / (CX * CY), I = (i0 + LOW) / 2 + (int)threadIdx.x % CX;
    const int Jc = (j0 + LOW) / 2 + (int)threadIdx.x / CX % CY;
    const int64_t ck = (int64_t)Jc * J.cld + I;
    const bool cin = REST && cc < 2 && (cc == 0 ? I <= J.cnx && Jc < J.cny : I < J.cnx && Jc <= J.cny);
    T cd = T(1);
    if (REST && cin && J.first) cd = J.cst[cc * PL_VY * J.cplane + ck];
    for (int q = threadIdx.x; q < 2 * WX * WY; q += NTH) {
        const int c = q / (WX * WY), r = (q / WX) % WY, ii = i0 - RIM + q % WX, jj = j0 - RIM + r;
        T val;
        if constexpr (UP) {
            val = T(0);
            const int64_t kk = (int64_t)jj * ld + ii;
            if (c == 0 && is_vx_unknown(nx, ny, ii, jj)) val = J.wx[kk] + T(prolong_sx(J, ii, jj));
            else if (c == 1 && is_vy_unknown(nx, ny, ii, jj)) val = J.wy[kk] + T(prolong_sy(J, ii, jj));
        } else {
            val = c == 0 ? ldvx<T>(J.vx, ld, nx, ny, ii, jj) : ldvy<T>(J.vy, ld, nx, ny, ii, jj);
        }
        win[q] = val;
    }
    __syncthreads();
    const int we = (y + RIM) * WX + x + RIM;
    T u = T(0), g = T(0);
    if (comp == 0) {
        const T av = row_sum<T, 0, WX>(cf, win, WX * WY, we);
        g = omega / cf[DIAG[0]];
        u = jac_step<T>(win[we], g, rhs, -av);
    } else {
        const T av = row_sum<T, 1, WX>(cf, win, WX * WY, we);
        g = omega / cf[DIAG[1]];
        u = jac_step<T>(win[WX * WY + we], g, rhs, -av);
    }
    u = unk ? u : T(0);
    mid[comp * NPOS + e] = u;
    __syncthreads();
    const bool box = comp == 0 ? i <= nx && j < ny : i < nx && j <= ny;
    const bool own = box && x >= LOW && x < LOW + OX && y >= LOW && y < LOW + OYR;
    if (!REST && !own) return;
    const bool second = x >= RIM && x < RX - RIM && y >= RIM && y < RY - RIM;
    T av = T(0);
    if (!REST || second) av = comp == 0 ? row_sum<T, 0, RX>(cf, mid, NPOS, e) : row_sum<T, 1, RX>(cf, mid, NPOS, e);
    if constexpr (UP) {
        const T o = jac_step<T>(u, g, rhs, -av);
        (comp == 0 ? J.vx : J.vy)[k] = unk ? o : T(0);
    } else {
        if (own) (comp == 0 ? J.wx : J.wy)[k] = u;
        const T r = unk ? rhs + av : T(0);
        if constexpr (!REST) {
            (comp == 0 ? J.rx : J.ry)[k] = r;
        } else {  // the first window is free
            if (second) win[comp * NPOS + e] = r;
            __syncthreads();
            if (!cin) return;
            const int N = cc == 0 ? I : Jc, M = cc == 0 ? Jc : I, E = cc == 0 ? J.cny : J.cnx, F = cc == 0 ? J.cnx : J.cny;
            T rv[3][4];
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = min(max(2 * N - 1 + a, 0), 2 * F), t = min(max(2 * M - 1 + q, 0), 2 * E - 1);
                    rv[a][q] = win[cc * NPOS + ((cc == 0 ? t : n) - j0) * RX + (cc == 0 ? n : t) - i0];
                }
            store_coarse<T>(J, cc, ck, N >= 1 && N <= F - 1, restrict_sum<T>(rv, M > 0, M < E - 1), cd, omega);
        }
    }
}

// The same two applications by a walk up a strip of 64 positions, 60 of them owned, for
// levels that fill the chip several times over.  The workgroup's waves hold RG rows of each
// component at a time.  A step takes the first application of RG rows and the second of the
// RG rows below, whose coefficients have stayed in registers since their own step, and loads
// those of the RG rows above in their place.  Both windows are rings of RING rows in LDS, one
// barrier a step.  A region computes half as much again as it owns, the walk a tenth; and of
// the regions only one fits on a CU, which then either loads or computes, of these workgroups
// two (FP64: two sets of coefficients, 208 to 240 VGPRs; with a third, to load a step ahead,
// they spill).  Level of 2048^2, down and up: FP64 497 and 502 us by regions, 375 and 405 by
// the walk; 1024^2 136, 135 and 103, 113; 512^2 38, 32 and 33, 33; FP32 1024^2 81, 79 and
// 54, 77, 512^2 25, 21 and 22, 32.  Going up, the walk waits for its prolongation, so it
// takes over later.
constexpr int RG = 2, WALK_OWN = 64 - 2 * RIM, WALK_W = 64 + 2 * RIM, RING = 16;

template <typename T, int A>
__device__ __forceinline__ T ring_sum(const T (&cf)[NCOEF], const T* win, const int (&rb)[5], int x) {
    T s = T(0);
#pragma unroll
    for (int q = 0; q < NCOEF; ++q) {
        const T v = win[slot_comp(A, q) * RING * WALK_W + rb[slot_dy(A, q) + 2] + x + slot_dx(A, q)];
        s += cf[q] * v;
    }
    return s;
}

template <typename T, bool UP>
__global__ __launch_bounds__(128 * RG, sizeof(T) == 4 ? 3 : 2) void k_mg_pair_walk(const LevelJob<T>* __restrict__ jobs,
                                                             const int* __restrict__ pre,
                                                             const FineShape* __restrict__ shapes, int n, T omega) {
    static_assert(2 * RG + 8 <= RING, "the rows in use at a time");
    __shared__ T win[2 * RING * WALK_W], mid[2 * RING * WALK_W];
    const int b = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int inst = find_pair_inst(pre, n, b);
    const LevelJob<T>& J = jobs[inst];
    const FineShape sh = shapes[inst];
    const int nx = J.nx, ny = J.ny, lb = b - pre[inst], lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), comp = wave / RG, y = wave % RG;
    const int x0 = lb % sh.nstrip * WALK_OWN - RIM, i = x0 + lane, x = lane + RIM;  // x: window column of i
    const int y0 = lb / sh.nstrip * sh.seg, y1 = min(y0 + sh.seg, ny + 1), G = (y1 - y0 + 2 * RIM + RG - 1) / RG;
    const int64_t ld = J.ld;
    const bool col = comp == 0 ? i >= 1 && i <= nx - 1 : i >= 0 && i <= nx - 1;
    const bool own = lane >= RIM && lane < 64 - RIM && (comp == 0 ? i <= nx : i < nx);
    auto unknown = [&](int j) { return col && (comp == 0 ? j >= 0 && j <= ny - 1 : j >= 1 && j <= ny - 1); };
    auto bases = [&](int j, int (&rb)[5]) {
#pragma unroll
        for (int d = 0; d < 5; ++d) rb[d] = ((j + d - 2) & (RING - 1)) * WALK_W;
    };
    // the staged iterate of this wave's component at grid column ii, row jj
    auto staged = [&](int ii, int jj) {
        T val = T(0);
        const int64_t kk = (int64_t)jj * ld + ii;
        if (comp == 0 ? is_vx_unknown(nx, ny, ii, jj) : is_vy_unknown(nx, ny, ii, jj)) {
            if constexpr (UP) val = comp == 0 ? J.wx[kk] + T(prolong_sx(J, ii, jj)) : J.wy[kk] + T(prolong_sy(J, ii, jj));
            else val = (comp == 0 ? J.vx : J.vy)[kk];
        }
        return val;
    };
    auto put_row = [&](int jj, T a, T c) {
        T* p = win + (comp * RING + (jj & (RING - 1))) * WALK_W;
        p[lane] = a;
        if (lane < 2 * RIM) p[64 + lane] = c;
    };
    T cf[2][NCOEF], rhs[2], g[2];
    auto coefs = [&](T (&c)[NCOEF], T& r, int j) {
        const bool in = unknown(j);
        if (comp == 0) load_row<T, 0>(J, i, j, in, c);
        else load_row<T, 1>(J, i, j, in, c);
        r = buf_load<T>(buf_rsrc((const T*)(comp == 0 ? J.bx : J.by), (size_t)((ny + 1) * ld) * sizeof(T)),
                        in ? (unsigned)(((int64_t)j * ld + i) * (int)sizeof(T)) : OOB);
    };
    const int j0 = y0 - RIM + y;
    for (int q = 0; q < RG + 2 * RIM; q += RG)
        if (y + q < RG + 2 * RIM) {
            const int jj = y0 - 2 * RIM + y + q;
            put_row(jj, staged(x0 - RIM + lane, jj), lane < 2 * RIM ? staged(x0 - RIM + 64 + lane, jj) : T(0));
        }
    coefs(cf[0], rhs[0], j0);
    __syncthreads();
    for (int s0 = 0; s0 <= G; s0 += 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int s = s0 + q, j = j0 + s * RG;
            if (s > G) break;
            if (s < G) {
                const int jn = j + RG + RIM;
                const T na = staged(x0 - RIM + lane, jn);
                const T nc = lane < 2 * RIM ? staged(x0 - RIM + 64 + lane, jn) : T(0);
                int rb[5];
                bases(j, rb);
                T av;
                if (comp == 0) {
                    av = ring_sum<T, 0>(cf[q], win, rb, x);
                    g[q] = omega / cf[q][DIAG[0]];
                } else {
                    av = ring_sum<T, 1>(cf[q], win, rb, x);
                    g[q] = omega / cf[q][DIAG[1]];
                }
                const T v = win[comp * RING * WALK_W + rb[2] + x];
                const T u = unknown(j) ? jac_step<T>(v, g[q], rhs[q], -av) : T(0);
                mid[comp * RING * WALK_W + rb[2] + x] = u;
                if (!UP && own && j >= y0 && j < y1 && (comp == 1 || j < ny))
                    (comp == 0 ? J.wx : J.wy)[(int64_t)j * ld + i] = u;
                put_row(jn, na, nc);
            }
            __syncthreads();
            const int jr = j - RG, p = 1 - q;  // the rows below
            if (own && jr >= y0 && jr < y1 && (comp == 1 || jr < ny)) {
                int rb[5];
                bases(jr, rb);
                const T av = comp == 0 ? ring_sum<T, 0>(cf[p], mid, rb, x) : ring_sum<T, 1>(cf[p], mid, rb, x);
                const int64_t k = (int64_t)jr * ld + i;
                if constexpr (UP) {
                    const T o = jac_step<T>(mid[comp * RING * WALK_W + rb[2] + x], g[p], rhs[p], -av);
                    (comp == 0 ? J.vx : J.vy)[k] = unknown(jr) ? o : T(0);
                } else {
                    (comp == 0 ? J.rx : J.ry)[k] = unknown(jr) ? rhs[p] + av : T(0);
                }
            }
            if (s + 1 < G) coefs(cf[p], rhs[p], j + RG);
        }
    }
}

}  // namespace

int mg_pair_tiles(int nx, int ny, PairKind kind) {
    const int ox = kind == PAIR_WIDE ? RX_WIDE - 2 * RIM : kind == PAIR_SMALL ? RX_SMALL - 2 * RIM : REST_X;
    const int oy = kind == PAIR_REST ? REST_Y : OY;
    return ((nx + 1 + ox - 1) / ox) * ((ny + 1 + oy - 1) / oy);
}

template <typename T>
int mg_pair(stk_ctx* ctx, const Batch& b, double omega, bool up, PairKind kind) {
    if (!b.n) return STK_OK;
    const auto* jobs = static_cast<const LevelJob<T>*>(b.jobs);
    const dim3 grid((unsigned)b.blocks), block(2 * (kind == PAIR_WIDE ? RX_WIDE : RX_SMALL) * RY);
    const auto kernel = kind == PAIR_REST ? k_mg_pair<T, false, RX_SMALL, true>
                        : kind == PAIR_WIDE ? (up ? k_mg_pair<T, true, RX_WIDE, false> : k_mg_pair<T, false, RX_WIDE, false>)
                                            : (up ? k_mg_pair<T, true, RX_SMALL, false> : k_mg_pair<T, false, RX_SMALL, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, jobs, b.pre, b.n, T(omega));
    STK_HIP(hipGetLastError());
    return STK_OK;
}

void mg_pair_walk_shape(const stk_ctx* ctx, int es, const int* nx, const int* ny, int n, std::vector<FineShape>* shapes,
                        std::vector<int>* pre) {
    const int64_t slots = (int64_t)std::max(ctx->num_cu, 1) * (es == 8 ? 4 : 8) / RG;
    int best = RG * 4;
    double cost = 1e300;
    int tall = 0;
    for (int q = 0; q < n; ++q) tall = std::max(tall, ny[q] + 1);
    for (int G = 2 * RIM / RG + 2; RG * (G - 1) - 2 * RIM < tall; ++G) {
        const int H = RG * G - 2 * RIM;
        int64_t wg = 0;
        for (int q = 0; q < n; ++q) wg += (int64_t)((nx[q] + WALK_OWN) / WALK_OWN) * ((ny[q] + H) / H);
        const double c = (double)((wg + slots - 1) / slots) * (G + 2);
        if (c < cost) {
            cost = c;
            best = H;
        }
    }
    shapes->clear();
    pre->assign(1, 0);
    for (int q = 0; q < n; ++q) {
        shapes->push_back(FineShape{(nx[q] + WALK_OWN) / WALK_OWN, (ny[q] + best) / best, best});
        pre->push_back(pre->back() + shapes->back().nstrip * shapes->back().nseg);
    }
}

template <typename T>
int mg_pair_walk(stk_ctx* ctx, const Batch& b, const FineShape* shapes, double omega, bool up) {
    if (!b.n) return STK_OK;
    const auto* jobs = static_cast<const LevelJob<T>*>(b.jobs);
    const dim3 grid((unsigned)b.blocks), block(128 * RG);
    if (up)
        hipLaunchKernelGGL((k_mg_pair_walk<T, true>), grid, block, 0, ctx->stream, jobs, b.pre, shapes, b.n,
                           T(omega));
    else
        hipLaunchKernelGGL((k_mg_pair_walk<T, false>), grid, block, 0, ctx->stream, jobs, b.pre, shapes, b.n,
                           T(omega));
    STK_HIP(hipGetLastError());
    return STK_OK;
}
template int mg_pair_walk<double>(stk_ctx*, const Batch&, const FineShape*, double, bool);
template int mg_pair_walk<float>(stk_ctx*, const Batch&, const FineShape*, double, bool);

template int mg_pair<double>(stk_ctx*, const Batch&, double, bool, PairKind);
template int mg_pair<float>(stk_ctx*, const Batch&, double, bool, PairKind);

}  // namespace stk
