// Temporally blocked damped Jacobi with the sweeps pipelined in registers.
//
// A wave owns a strip of 64 - 2K columns and a segment of rows; its 64 lanes
// hold the strip and K columns on each side, and it walks up the rows once for
// K sweeps.  When row r arrives from memory, sweep level 1 relaxes row r - 1,
// level 2 row r - 2 and so on: each level needs one row ahead of the level
// below, which that level has just produced, so all K levels advance by one
// row per step with nothing but registers between them.  There is no LDS and
// no barrier, and waves never wait for each other.  A level's values are exact
// one column and one row further in than the level below, so the K columns at
// either side and the first K rows of the walk are discarded.
//
// Work per level and cell.  The operator's differences are shared: the shear
// strain of node (i, j) serves the rows j - 1 and j of vx and the columns
// i - 1 and i of vy, the normal differences both neighbours of a cell.  Each is
// formed once, in the shared expression order (stencil.hpp), and carried to
// the next row in a register or to the next column by DPP, which leaves 18 or
// 19 floating-point operations and 8 moves per cell and sweep; the values are
// bit for bit those of the gathering kernels.  The coefficients of a row
// (A, N and their neighbours, b, omega / d) are formed once, when it arrives,
// and live in a register ring of K + 2 rows until the last level has passed.
//
// Cells that are not relaxed (walls, outside the grid) carry omega / d = 0.
//
// What bounds it: the eight planes of memory traffic up to K = 5 (4096^2 FP64:
// 0.22 - 0.23 ms a pass whatever K is, 4.6 - 4.9 TB/s of the 5.8 a flat stream
// of the same planes reaches), then vector issue.  Against the LDS pipeline
// with one wave per level that ran these sweeps before (4096^2): FP64 k = 4
// 0.238 -> 0.232 ms a pass, and 0.246 ms for K = 7 (480 GLUP/s against 284);
// FP32 0.156 ms for k = 4 -> 0.122, and 0.145 for K = 8 (920 against 520).  Where
// few waves share a SIMD, a step's scalar instructions count as much as its vector
// ones: with rows addressed by one scalar offset (RowSpan) 20 sweeps of 2048^2 take
// 175 us instead of 205 in FP64 and 115 instead of 131 in FP32.
#pragma once

#include "rowstream.hpp"

namespace stk {
namespace pipe {

constexpr int WPB = 4;  // waves per workgroup (independent)
// rows loaded ahead of the walk
template <typename T>
constexpr int ahead() { return sizeof(T) == 8 ? 2 : 4; }

// Rows of the coefficient ring, and steps per unrolled trip (the ring slots,
// the load queue and the carried rows rotate by renaming): K + 2, made a
// multiple of the load queue.
template <typename T>
constexpr int ring_rows(int K) { return (K + 1 + ahead<T>()) / ahead<T>() * ahead<T>(); }
__host__ __device__ constexpr int strip(int K) { return 64 - 2 * K; }

// Most rows a window may have (RowSpan), with the rows loaded ahead.
inline int max_rows(int64_t ld, int es) {
    const int64_t n = (int64_t)UINT32_MAX / (ld * es) - 64;
    return (int)(n < 0 ? 0 : n > INT32_MAX / 2 ? INT32_MAX / 2 : n);
}

// Launch geometry of one grid: strips x segments waves of `seg` rows each
// (seg + 2K is a multiple of the unrolled trip).
struct Shape {
    int K, nstrip, nseg, seg;
};

// Waves per SIMD the registers of K sweeps must leave room for.
template <typename T>
constexpr int pipe_occupancy(int K) { return sizeof(T) == 8 ? (K <= 3 ? 3 : K <= 7 ? 2 : 1) : (K <= 4 ? 4 : K <= 8 ? 3 : 2); }

// Time of one step of one wave that has the SIMD to itself, in us: about 217
// (FP64, K = 7) or 180 (FP32, K = 8) vector instructions; measured 0.48 and
// 0.30 (2048^2, two waves per SIMD).
template <typename T>
inline double step_us(int K) { return sizeof(T) == 8 ? 2.2e-3 * (30 + 27 * K) : 1.6e-3 * (44 + 17 * K); }

// A wave's window of consecutive rows of an array: row r of [r0, r0 + n) starts
// (r - r0) row bytes beyond a base that is formed once.  A row is then one scalar
// offset for every array of the window, where a buffer resource per row and array
// took about ten scalar instructions each, issue slots that a wave alone on its
// SIMD does not have.  The host keeps n row bytes below 2^32.
struct RowSpan {
    int r0;
    unsigned rowb, bytes;
    __device__ __forceinline__ RowSpan(int r0_, int n, int64_t ld, int es)
        : r0(r0_), rowb((unsigned)(ld * es)), bytes((unsigned)n * rowb) {}
    __device__ __forceinline__ unsigned at(int r) const { return (unsigned)(r - r0) * rowb; }
    template <typename P>
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t of(P p, int64_t ld, bool ok) const {
        return buf_rsrc(p + (int64_t)r0 * ld, ok ? bytes : 0);
    }
};

// Rows of velocity, viscosities and right-hand side at this lane's column, walls and
// everything outside the arrays 0 (the rows of rows::Loader).  zero: the velocity is
// 0 and not read.
template <typename T>
struct PipeRows {
    const T *vx, *vy, *ec, *en, *bx, *by;
    int64_t ld;
    int ny;
    unsigned o_inner, o_cell;
    RowSpan span;
    bool zero;
    __device__ __forceinline__ PipeRows(const T* vx_, const T* vy_, const T* ec_, const T* en_, const T* bx_,
                                        const T* by_, int64_t ld_, int nx, int ny_, int i, int r0, int n, bool zero_)
        : vx(vx_), vy(vy_), ec(ec_), en(en_), bx(bx_), by(by_), ld(ld_), ny(ny_),
          o_inner(i >= 1 && i <= nx - 1 ? (unsigned)i * (unsigned)sizeof(T) : OOB),
          o_cell(i >= 0 && i <= nx - 1 ? (unsigned)i * (unsigned)sizeof(T) : OOB), span(r0, n, ld_, (int)sizeof(T)),
          zero(zero_) {}
    __device__ __forceinline__ rows::Row<T> load(int r) const {
        const bool x = r >= 0 && r <= ny - 1, y = r >= 1 && r <= ny - 1;
        const unsigned o = span.at(r);
        rows::Row<T> q;
        q.vx = buf_load_at<T>(span.of(vx, ld, x && !zero), o_inner, o);
        q.vy = buf_load_at<T>(span.of(vy, ld, y && !zero), o_cell, o);
        q.ec = buf_load_at<T>(span.of(ec, ld, x), o_cell, o);
        q.en = buf_load_at<T>(span.of(en, ld, y), o_inner, o);
        q.bx = buf_load_at<T>(span.of(bx, ld, x), o_inner, o);
        q.by = buf_load_at<T>(span.of(by, ld, y), o_cell, o);
        q.p = T(0);
        return q;
    }
};

// Stores of finished velocity rows y0 <= j < y1 at this lane's column, walls 0 (own:
// the lane owns its column).
template <typename T>
struct PipeStore {
    T *ox, *oy;
    int64_t ld;
    int ny, y0, y1;
    unsigned s_x, s_y;
    bool xcol;
    RowSpan span;
    __device__ __forceinline__ PipeStore(T* ox_, T* oy_, int64_t ld_, int nx, int ny_, int y0_, int y1_, int i, bool own)
        : ox(ox_), oy(oy_), ld(ld_), ny(ny_), y0(y0_), y1(y1_),
          s_x(own && i <= nx ? (unsigned)i * (unsigned)sizeof(T) : OOB),
          s_y(own && i < nx ? (unsigned)i * (unsigned)sizeof(T) : OOB), xcol(i >= 1 && i <= nx - 1),
          span(y0_, y1_ - y0_, ld_, (int)sizeof(T)) {}
    __device__ __forceinline__ void operator()(int j, T ux, T uy) const { store(j, j >= y0 && j < y1, ux, uy); }
    __device__ __forceinline__ void store(int j, bool in, T ux, T uy) const {
        const unsigned o = span.at(j);
        buf_store_at(xcol ? ux : T(0), span.of(ox, ld, in && j <= ny - 1), s_x, o);
        buf_store_at(j >= 1 && j <= ny - 1 ? uy : T(0), span.of(oy, ld, in), s_y, o);
    }
};

// One row's coefficients at the lane's column: A = 2 eta_c idx^2 at (i, j) and
// (i - 1, j), N = eta_n idx idy at (i, j) and (i + 1, j), the right-hand side
// and the Jacobi factors of vx(i, j) and vy(i, j).
template <typename T>
struct Coef {
    T A, aL, N, nR, bx, by, gx, gy;
};
// A level's carried state, of the level below it at row j: v, the node strains
// of row j (S scaled for vx, Q for vy), and vy(j) - vy(j - 1).
template <typename T>
struct State {
    T vx, vy, S, Q, ey;
};

// The operator at row j from the state (row j) and the new row j + 1 of the
// level below (nx, ny); c: the coefficients of row j, nR: N(i + 1, j), Ab:
// A(i, j - 1), Nt: N(i, j + 1).  m: (M v) at row j, v: the level below there.
template <typename T, bool SQ>
__device__ __forceinline__ void level(State<T>& s, T nx, T ny, const Coef<T>& c, T nR, T Ab, T Nt, const Scale<T>& sc,
                                      T& mx, T& my, T& vx, T& vy) {
    const T a = nx - s.vx;
    const T d = ny - wave_shift<DPP_FROM_PREV>(ny);
    const T S1 = SQ ? a + d : fmaT(sc.ry, a, d);
    const T Q1 = SQ ? S1 : fmaT(sc.rx, d, a);
    const T ey = ny - s.vy;
    const T ex = wave_shift<DPP_FROM_NEXT>(s.vx) - s.vx;
    const T exl = wave_shift<DPP_FROM_PREV>(ex);
    const T Qr = wave_shift<DPP_FROM_NEXT>(s.Q);
    mx = c.A * ex;
    mx = fmaT(-c.aL, exl, mx);
    mx = fmaT(Nt, S1, mx);
    mx = fmaT(-c.N, s.S, mx);
    T B = c.A, Bb = Ab;
    if (!SQ) {
        // B = A kap is formed by every level: an opaque copy of the (scalar) kap
        // keeps the compiler from holding B of all the ring's rows in registers
        Scale<T> sk = sc;
        asm volatile("" : "+s"(sk.kap));
        B = coef_b(c.A, sk);
        Bb = coef_b(Ab, sk);
    }
    my = B * ey;
    my = fmaT(-Bb, s.ey, my);
    my = fmaT(nR, Qr, my);
    my = fmaT(-c.N, s.Q, my);
    vx = s.vx;
    vy = s.vy;
    s.vx = nx;
    s.vy = ny;
    s.S = S1;
    s.Q = Q1;
    s.ey = ey;
}

// The cells a wave relaxes: does this lane's column have vx, vy unknowns, and does row r.
// All others keep their value through every sweep.  SELECT: by a select, where a factor
// omega / d of 0 would let a non-finite neighbour through to them; the walls and what lies
// beyond have no neighbour but the unknowns beside them, which that neighbour reaches first.
struct AllCells {
    static constexpr bool SELECT = false;
    bool x, y;
    int ny;
    __device__ __forceinline__ AllCells(int nx, int ny_, int i)
        : x(i >= 1 && i <= nx - 1), y(i >= 0 && i <= nx - 1), ny(ny_) {}
    __device__ __forceinline__ bool row_x(int r) const { return r >= 0 && r <= ny - 1; }
    __device__ __forceinline__ bool row_y(int r) const { return r >= 1 && r <= ny - 1; }
};

// K sweeps of the rows that load(r) delivers for r0 <= r < r1 (at column i of each
// lane; arrive(u, r, row) may change the row's velocity when it arrives), and,
// with RES, the residual b - M v of their result.  put(j, ux, uy) receives row
// j = r - K of the last sweep, putr(u, j, rx, ry) row j = r - K - 1 of the residual
// (0 off the unknowns); both get every row, in order, and keep what is theirs.
// u: the step within the unrolled trip of R steps (a compile-time value).
// SQ: square cells (ry = rx = kap = 1 exactly, so B = A and the two strains are
// the same sum).
template <typename T, int K, bool SQ, bool RES, int R, typename LD, typename CELLS, typename ARR, typename PUT,
          typename PUTR>
__device__ __forceinline__ void walk(const LD& L, int r0, int r1, const CELLS& relax, T omega, T idx, T idy,
                                     const ARR& arrive, const PUT& put, const PUTR& putr) {
    constexpr int PFD = ahead<T>(), NL = K + (RES ? 1 : 0);
    static_assert(R >= NL + 2 && R % PFD == 0, "the ring holds NL + 2 rows and the load queue rotates by renaming");
    // many FP64 sweeps on cells that are not square: N(i + 1, j) is taken again
    // by each level rather than kept in the ring, so that 256 registers do
    constexpr bool KEEP_NR = SQ || sizeof(T) == 4 || NL <= 5;
    const Scale<T> sv = stencil_scale(idx, idy);
    const Scale<T> sc{wave_uniform(sv.a), wave_uniform(sv.n), wave_uniform(sv.kap), wave_uniform(sv.ry),
                      wave_uniform(sv.rx)};
    State<T> st[NL];
    Coef<T> cf[R];
    bool takes_x[R], takes_y[R];  // SELECT: this lane relaxes the row
#pragma unroll
    for (int s = 0; s < NL; ++s) st[s] = State<T>{T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int q = 0; q < R; ++q) {
        cf[q] = Coef<T>{T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
        takes_x[q] = takes_y[q] = false;
    }
    rows::Row<T> q[PFD];
#pragma unroll
    for (int p = 0; p < PFD; ++p) q[p] = L.load(r0 + p);
    for (int rb = r0; rb < r1; rb += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int r = rb + u;
            if (!KEEP_NR) {  // never taken: a block of its own per step, or the compiler keeps the N(i + 1, j)
                             // of all the ring's rows after all
                int never = 0;
                asm volatile("" : "+s"(never));
                if (never) __builtin_amdgcn_s_sleep(0);
            }
            rows::Row<T> w = q[u % PFD];
            q[u % PFD] = L.load(r + PFD);
            // FP64 steps stay apart, or the compiler mixes them and delays the loads (20 sweeps at
            // 2048^2: 219 us, 175 us with the barrier; FP32 1501 x 1100 is 73 us without, 81 us with)
            if (sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
            arrive(u, r, w);
            Coef<T>& c0 = cf[u];                 // row r
            Coef<T>& c1 = cf[(u + R - 1) % R];   // row r - 1
            const Coef<T>& c2 = cf[(u + R - 2) % R];
            c0.A = coef_a(w.ec, sc);
            c0.N = coef_n(w.en, sc);
            c0.aL = wave_shift<DPP_FROM_PREV>(c0.A);
            if (KEEP_NR) c0.nR = wave_shift<DPP_FROM_NEXT>(c0.N);
            c0.bx = w.bx;
            c0.by = w.by;
            {  // the factors of row r - 1, whose upper shear coefficient is now here
                const int j = r - 1;
                const T nR = KEEP_NR ? c1.nR : wave_shift<DPP_FROM_NEXT>(c1.N);
                const T dx = SQ ? (c1.N + c0.N) + (c1.aL + c1.A) : diagx_scaled<T>(c1.aL, c1.A, c1.N, c0.N, sc.ry);
                const T dy = SQ ? (c1.N + nR) + (c2.A + c1.A)
                                : diagy_scaled<T>(coef_b(c2.A, sc), coef_b(c1.A, sc), c1.N, nR, sc.rx);
                const T gx = jac_factor(omega, dx), gy = jac_factor(omega, dy);
                if constexpr (CELLS::SELECT) {
                    takes_x[(u + R - 1) % R] = relax.x & relax.row_x(j);
                    takes_y[(u + R - 1) % R] = relax.y & relax.row_y(j);
                    c1.gx = gx;
                    c1.gy = gy;
                } else {
                    c1.gx = (relax.x && relax.row_x(j)) ? gx : T(0);
                    c1.gy = (relax.y && relax.row_y(j)) ? gy : T(0);
                }
            }
            T ux = w.vx, uy = w.vy;
#pragma unroll
            for (int s = 1; s <= NL; ++s) {  // level s: row r - s
                const Coef<T>& c = cf[(u + 2 * R - s) % R];
                const T Ab = cf[(u + 2 * R - s - 1) % R].A, Nt = cf[(u + 2 * R - s + 1) % R].N;
                const T nR = KEEP_NR ? c.nR : wave_shift<DPP_FROM_NEXT>(c.N);
                T mx, my, vx, vy;
                level<T, SQ>(st[s - 1], ux, uy, c, nR, Ab, Nt, sc, mx, my, vx, vy);
                if (RES && s == NL) {
                    const int j = r - NL;
                    putr(u, j, (relax.x && relax.row_x(j)) ? c.bx - mx : T(0),
                         (relax.y && relax.row_y(j)) ? c.by - my : T(0));
                } else {
                    ux = jac_step<T>(vx, c.gx, c.bx, mx);
                    uy = jac_step<T>(vy, c.gy, c.by, my);
                    if constexpr (CELLS::SELECT) {
                        asm volatile("" : "+v"(ux), "+v"(uy));  // or the compiler makes branches of the selects
                        ux = takes_x[(u + 2 * R - s) % R] ? ux : vx;
                        uy = takes_y[(u + 2 * R - s) % R] ? uy : vy;
                    }
                    if (s == K) put(r - K, ux, uy);
                }
            }
        }
    }
}

}  // namespace pipe
}  // namespace stk
