// ffmg_krylov.hip -- GMRES(m) smoothing steps for the multigrid V-cycle
// (Sec. 3.3: GMRES(m), m = 2 or 3, replaces weighted Jacobi and keeps the
// V-cycle stable at rotation angles near 10 degrees).
//
// One smoothing step is one restart cycle of GMRES from the current iterate:
// with r0 = b - A u, u is replaced by the u + z, z in span{r0, A r0, ...,
// A^{m-1} r0}, of least residual norm.  The basis is kept unnormalised,
// Z_0 = r0 and Z_{j+1} = A Z_j - sum_{i<=j} (d_ij / n_i) Z_i with
// d_ij = <Z_i, A Z_j> (Hermitian product, classical Gram-Schmidt: all d_ij
// of one step from one pass) and n_i = |Z_i|^2, so that v_i = Z_i / sqrt(n_i)
// is Arnoldi's orthonormal basis and H_ij = d_ij / sqrt(n_i n_j),
// H_{j+1,j} = sqrt(n_{j+1} / n_j).  The (m+1) x m least-squares problem
// min |sqrt(n_0) e_1 - H y| is solved on the device by one thread with
// complex Givens rotations (FP64), and u += sum_j (y_j / sqrt(n_j)) Z_j.
//
// Kernels (a point a thread, tiles of 64 x 8 points in 2D): the residual and
// A Z_0 with the partial |Z_0|^2 and <Z_0, A Z_0>, as one pass or two; for
// j = 1 .. m - 1 one pass that forms Z_j from W = A Z_{j-1} and Z_0 .. Z_{j-1}
// (on the tile and around it, through LDS in 2D, so that the orthogonalisation
// needs no pass of its own) and applies A to it, with the partial |Z_j|^2 and
// <Z_i, A Z_j>; the norm of Z_m (not stored); the small problem and the update.
// Each pass adds the previous passes' partial sums itself, in block order (every
// block the same sums, so no pass waits on a one-block kernel): m + 2 or m + 3
// launches per step.
// The reference kernel path (a pass per product and one for the
// orthogonalisation, each finished by a one-block kernel: 4 m + 3 launches)
// computes the same values in the same order, so both give the same bits.
// Partial sums are FP64 in both precisions.  A level of at most
// GM_BLOCK_MAX_POINTS points runs the whole step in one workgroup, of 256
// threads up to 1024 points and 1024 threads above (for small m with the
// vectors in registers and the stencil's input staged in LDS; the reference
// path reads and writes them in global memory).
#include "ffmg_internal.hpp"
#include "ffmg_point.hpp"
#include "ffmg_wave.hpp"

namespace ffmg {

namespace {

// Threads of the grid-wide passes' blocks (GM_BLOCKS at most).  Every
// block of a pass adds up all blocks' partial sums of the pass before, so few
// large blocks: with 1024 of 256 threads a pass read 57 MB of partial sums
// (511 x 511, FP32, m = 3: the four passes that do, 33 us then, 25 us now).
constexpr int GM_BT = 512;
// partial-sum slots: n_i at slot i (i <= m), d_ij (re, im) at NSLOT_D + 2 (j GMRES_MAX_M + i)
constexpr int NSLOT_D = GMRES_MAX_M + 1;

__device__ __forceinline__ void grid_coords(size_t j, int mx, int my, int &ix, int &iy, int &iz)
{
    split3(j, mx, my, ix, iy, iz);   // 32-bit divisions where j fits
}

// (A z)_j from the five (seven) stencil values, zero outside the grid: the
// point functions of every other kernel, so the bits agree with them.  zat(k)
// gives z at point k (a load, or a value formed on the fly); zc = zat(j).
template <typename T, int DIM, typename ZAt>
__device__ __forceinline__ cx<T> apply_at_f(const Stencil<T> &P, ZAt zat, cx<T> zc, cx<T> qj, size_t j)
{
    int ix, iy, iz;
    grid_coords(j, P.mx, P.my, ix, iy, iz);
    const cx<T> zero = {T(0), T(0)};
    const size_t sx = 1, sy = (size_t)P.mx, sz = (size_t)P.mx * P.my;
    cx<T> w = ix > 0 ? zat(j - sx) : zero, e = ix < P.mx - 1 ? zat(j + sx) : zero;
    cx<T> s = iy > 0 ? zat(j - sy) : zero, n = iy < P.my - 1 ? zat(j + sy) : zero;
    cx<T> L = lap_xy(P, zc, w, e, s, n);
    if (DIM == 3) {
        cx<T> d = iz > 0 ? zat(j - sz) : zero, up = iz < P.mz - 1 ? zat(j + sz) : zero;
        L = lap_add_z(P, L, zc, d, up);
    }
    return apply_point(P, L, zc, qj);
}

// The 2D product where the coordinates of point j are known.
template <typename T, typename ZAt>
__device__ __forceinline__ cx<T> apply_xy_f(const Stencil<T> &P, ZAt zat, cx<T> zc, cx<T> qj, size_t j, int ix, int iy)
{
    const cx<T> zero = {T(0), T(0)};
    const size_t sy = (size_t)P.mx;
    cx<T> w = ix > 0 ? zat(j - 1) : zero, e = ix < P.mx - 1 ? zat(j + 1) : zero;
    cx<T> s = iy > 0 ? zat(j - sy) : zero, n = iy < P.my - 1 ? zat(j + sy) : zero;
    return apply_point(P, lap_xy(P, zc, w, e, s, n), zc, qj);
}

template <typename T, int DIM>
__device__ __forceinline__ cx<T> apply_pt(const Stencil<T> &P, const cx<T> *__restrict__ z, cx<T> qj, size_t j, int ix,
                                          int iy)
{
    if constexpr (DIM == 2) return apply_xy_f<T>(P, [&](size_t k) { return z[k]; }, z[j], qj, j, ix, iy);
    else return apply_at_f<T, DIM>(P, [&](size_t k) { return z[k]; }, z[j], qj, j);
}

template <typename T, int DIM>
__device__ __forceinline__ cx<T> apply_at(const Stencil<T> &P, const cx<T> *__restrict__ z, cx<T> qj, size_t j)
{
    return apply_at_f<T, DIM>(P, [&](size_t k) { return z[k]; }, z[j], qj, j);
}

// The points of this thread in a pass over a level: in 2D the block's tiles of
// GM_TX x GM_TY points, a point a thread, else every gridDim.x-th run of GM_BT
// points.  Every pass of a step takes them alike, so their sums agree between
// the default and the reference passes.  visit(j, ix, iy, own): own is false for
// a thread without a point in the tile (2D only; j is then 0).
constexpr int GM_TX = 64, GM_TY = GM_BT / GM_TX;
__host__ __device__ constexpr int gm_tiles_x(int mx) { return (mx + GM_TX - 1) / GM_TX; }
__host__ __device__ constexpr int gm_tiles(int mx, int my) { return gm_tiles_x(mx) * ((my + GM_TY - 1) / GM_TY); }
template <int DIM, typename T, typename F>
__device__ __forceinline__ void for_points(const Stencil<T> &P, size_t N, F visit)
{
    if constexpr (DIM == 2) {
        const int tx = gm_tiles_x(P.mx), nt = gm_tiles(P.mx, P.my);
        for (int tile = blockIdx.x; tile < nt; tile += gridDim.x) {
            const int ix = (tile % tx) * GM_TX + (int)(threadIdx.x % GM_TX);
            const int iy = (tile / tx) * GM_TY + (int)(threadIdx.x / GM_TX);
            const bool own = ix < P.mx && iy < P.my;
            visit(own ? (size_t)iy * P.mx + ix : 0, ix, iy, own);
        }
    } else {
        for (size_t j = (size_t)blockIdx.x * GM_BT + threadIdx.x; j < N; j += (size_t)gridDim.x * GM_BT)
            visit(j, 0, 0, true);
    }
}

// Sums of NV doubles per thread of a block into parts[slot[v] * GM_BLOCKS +
// blockIdx.x] (by halving, within each wave and over the waves).
template <int NV>
__device__ __forceinline__ void block_partials(const double (&acc)[NV], const int (&slot)[NV],
                                               double *__restrict__ parts)
{
    constexpr int NW = GM_BT / 64;
    __shared__ double red[NV * NW];
    double s[(NV + 3) / 4];
    wave_sums<NV>(acc, s);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, v0 = wave_sum_value(lane >> 4);
#pragma unroll
    for (int h = 0; h < (NV + 3) / 4; ++h)
        if ((lane & 15) == 0 && 4 * h + v0 < NV) red[(4 * h + v0) * NW + wv] = s[h];
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if ((int)threadIdx.x != v) continue;
        double a[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) a[w] = red[v * NW + w];
#pragma unroll
        for (int st = NW / 2; st > 0; st >>= 1)
#pragma unroll
            for (int w = 0; w < st; ++w) a[w] += a[w + st];
        parts[(size_t)slot[v] * GM_BLOCKS + blockIdx.x] = a[0];
    }
}

// The sums over the nb blocks of the partials of slots slot0 + v into out[v],
// v < NV (lane-strided, then by halving; a wave takes every GM_BT / 64-th
// value).  A lane's loads are issued together, before they are added in order:
// a chain of load and add takes longer than the pass on a small level.
template <int NV>
__device__ __forceinline__ void reduce_slots(const double *parts, int nb, int slot0, double *out)
{
    constexpr int NL = GM_BLOCKS / 64, NW = GM_BT / 64, NR = (NV + NW - 1) / NW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double x[NR][NL];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const double *p = parts + (size_t)(slot0 + min(wv + r * NW, NV - 1)) * GM_BLOCKS;
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (64 * k < nb) x[r][k] = p[min(lane + 64 * k, nb - 1)];
    }
    double a[NR], s[(NR + 3) / 4];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        a[r] = 0.0;
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (64 * k < nb && lane + 64 * k < nb) a[r] += x[r][k];
    }
    wave_sums<NR>(a, s);
#pragma unroll
    for (int r = 0; r < NR; ++r)
        if (lane == wave_sum_lane(r & 3) && wv + r * NW < NV) out[wv + r * NW] = s[r / 4];
}

// The small least-squares problem (one thread, FP64; H is in registers, as every
// index is a constant once the loops are unrolled, up to 4 columns, and in LDS
// beyond): from the squared norms n[0..M]
// and the products d[2 (j GMRES_MAX_M + i)] = <Z_i, A Z_j> (re, im), the
// coefficients c[2 j] (re, im) of the unnormalised basis vectors, c_j = y_j /
// sqrt(n_j), zero past a breakdown (after k columns).
template <int M>
__device__ __forceinline__ void gm_solve_in(const double *n, const double *d, double *c, cd (&H)[M + 1][M])
{
    cd g[M + 1], cs[M], sn[M], y[M];
#pragma unroll
    for (int j = 0; j < M; ++j) c[2 * j] = c[2 * j + 1] = 0.0;
    double nv[M + 1];
#pragma unroll
    for (int j = 0; j <= M; ++j) nv[j] = n[j];
    if (!(nv[0] > 0.0)) return;
    int k = M;
#pragma unroll
    for (int j = 0; j < M; ++j) {
        if (j >= k) continue;
#pragma unroll
        for (int i = 0; i <= j; ++i) {
            const double sc = 1.0 / sqrt(nv[i] * nv[j]);
            H[i][j] = cd{d[2 * (j * GMRES_MAX_M + i)] * sc, d[2 * (j * GMRES_MAX_M + i) + 1] * sc};
        }
        const double nn = nv[j + 1];
        H[j + 1][j] = cd{nn > 0.0 ? sqrt(nn / nv[j]) : 0.0, 0.0};
        if (!(nn > 0.0)) k = j + 1;   // the Krylov space is invariant: solve with j + 1 columns
    }
#pragma unroll
    for (int i = 0; i <= M; ++i) g[i] = cd{0.0, 0.0};
    g[0] = cd{sqrt(nv[0]), 0.0};
#pragma unroll
    for (int j = 0; j < M; ++j) {
        if (j >= k) continue;
#pragma unroll
        for (int i = 0; i < j; ++i) {
            const cd t = cs[i] * H[i][j] + sn[i] * H[i + 1][j];
            H[i + 1][j] = cd{-sn[i].re, sn[i].im} * H[i][j] + cs[i] * H[i + 1][j];
            H[i][j] = t;
        }
        const cd a = H[j][j], cc = H[j + 1][j];
        const double r = sqrt(a.re * a.re + a.im * a.im + cc.re * cc.re + cc.im * cc.im);
        cs[j] = cd{1.0, 0.0};
        sn[j] = cd{0.0, 0.0};
        if (r == 0.0) continue;
        const double aa = sqrt(a.re * a.re + a.im * a.im);
        if (aa == 0.0) {
            cs[j] = cd{0.0, 0.0};
            sn[j] = cd{cc.re / r, -cc.im / r};
        } else {
            cs[j] = cd{aa / r, 0.0};
            const cd ph = {a.re / aa, a.im / aa};
            sn[j] = ph * cd{cc.re / r, -cc.im / r};
        }
        H[j][j] = cs[j] * a + sn[j] * cc;
        H[j + 1][j] = cd{0.0, 0.0};
        const cd t = cs[j] * g[j] + sn[j] * g[j + 1];
        g[j + 1] = cd{-sn[j].re, sn[j].im} * g[j] + cs[j] * g[j + 1];
        g[j] = t;
    }
#pragma unroll
    for (int i = M - 1; i >= 0; --i) {
        if (i >= k) continue;
        cd t = g[i];
#pragma unroll
        for (int j = i + 1; j < M; ++j)
            if (j < k) t = t - H[i][j] * y[j];
        const cd dd_ = H[i][i];
        const double dd = dd_.re * dd_.re + dd_.im * dd_.im;
        y[i] = dd > 0.0 ? cd{(t.re * dd_.re + t.im * dd_.im) / dd, (t.im * dd_.re - t.re * dd_.im) / dd}
                        : cd{0.0, 0.0};
        const double sc = 1.0 / sqrt(nv[i]);
        c[2 * i] = y[i].re * sc;
        c[2 * i + 1] = y[i].im * sc;
    }
}

// The small problem's matrix in LDS (as doubles: a shared variable has no
// constructor), aligned as the complex values it is read as.
template <int M>
struct alignas(alignof(cd)) GmMatrix {
    double v[2 * (M + 1) * M];
};

template <int M>
__device__ __forceinline__ void gm_solve_small(const double *n, const double *d, double *c)
{
    if constexpr (M <= 4) {
        cd H[M + 1][M];
        gm_solve_in<M>(n, d, c, H);
    } else {
        static_assert(alignof(GmMatrix<M>) >= alignof(cd) && sizeof(GmMatrix<M>) == sizeof(cd[M + 1][M]),
                      "GmMatrix is read as cd[M + 1][M]");
        __shared__ GmMatrix<M> Hs;
        gm_solve_in<M>(n, d, c, reinterpret_cast<cd(&)[M + 1][M]>(Hs.v));
    }
}

// Z0 = b - A u (zero: u is 0 and is set to 0), partial n_0 = |Z0|^2.
template <typename T, int DIM>
__global__ __launch_bounds__(GM_BT) void k_gm_resid(cx<T> *__restrict__ u, int zero, const cx<T> *__restrict__ b,
                                                  const cx<T> *__restrict__ q, cx<T> *__restrict__ z0, Stencil<T> P,
                                                  size_t N, double *__restrict__ parts, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    double acc[1] = {0.0};
    for_points<DIM>(P, N, [&](size_t j, int ix, int iy, bool own) {
        if (!own) return;
        cx<T> r = b[j];
        if (zero) {
            u[j] = cx<T>{T(0), T(0)};
        } else {
            cx<T> Au = apply_pt<T, DIM>(P, u, q[j], j, ix, iy);
            r = cx<T>{r.re - Au.re, r.im - Au.im};
        }
        z0[j] = r;
        acc[0] += (double)r.re * (double)r.re + (double)r.im * (double)r.im;
    });
    const int slot[1] = {0};
    block_partials<1>(acc, slot, parts);
}

// W = A Z_j into w (the reference path: Z_{j+1}'s slot); partial d_ij =
// <Z_i, W> for i <= j (j = NJ - 1).
template <typename T, int DIM, int NJ>
__global__ __launch_bounds__(GM_BT) void k_gm_apply_dots(cx<T> *__restrict__ Z, cx<T> *__restrict__ w, size_t N,
                                                       const cx<T> *__restrict__ q, Stencil<T> P,
                                                       double *__restrict__ parts, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    constexpr int j = NJ - 1;
    const cx<T> *zj = Z + (size_t)j * N;
    double acc[2 * NJ];
#pragma unroll
    for (int v = 0; v < 2 * NJ; ++v) acc[v] = 0.0;
    for_points<DIM>(P, N, [&](size_t p, int ix, int iy, bool own) {
        if (!own) return;
        cx<T> Wp = apply_pt<T, DIM>(P, zj, q[p], p, ix, iy);
        w[p] = Wp;
        const double wr = Wp.re, wi = Wp.im;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const cx<T> zi = Z[(size_t)i * N + p];
            acc[2 * i] += (double)zi.re * wr + (double)zi.im * wi;       // conj(z_i) w
            acc[2 * i + 1] += (double)zi.re * wi - (double)zi.im * wr;
        }
    });
    int slot[2 * NJ];
#pragma unroll
    for (int v = 0; v < 2 * NJ; ++v) slot[v] = NSLOT_D + 2 * (j * GMRES_MAX_M) + v;
    block_partials<2 * NJ>(acc, slot, parts);
}

// The first two passes in one: Z_0 = b - A u (formed at the point and its
// neighbours; from a zero guess b itself, and u is set to 0), W = A Z_0, the
// partial |Z_0|^2 and <Z_0, W>.  The values and partial sums of k_gm_resid
// followed by k_gm_apply_dots<1>.
template <typename T, int DIM, bool ZERO>
__global__ __launch_bounds__(GM_BT) void k_gm_resid_dots(cx<T> *__restrict__ u, const cx<T> *__restrict__ b,
                                                         const cx<T> *__restrict__ q, cx<T> *__restrict__ z0,
                                                         cx<T> *__restrict__ w, Stencil<T> P, size_t N,
                                                         double *__restrict__ parts, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    double acc[3] = {0.0, 0.0, 0.0};
    for_points<DIM>(P, N, [&](size_t j, int ix, int iy, bool own) {
        if (!own) return;
        const cx<T> qj = q[j];
        cx<T> zc, Wp;
        if constexpr (ZERO) {
            zc = b[j];
            Wp = apply_pt<T, DIM>(P, b, qj, j, ix, iy);
            u[j] = cx<T>{T(0), T(0)};
        } else {
            // u is read at up to two points' distance: not written in this pass
            auto resid = [&](size_t k, int kx, int ky, cx<T> qk) {
                const cx<T> r = b[k], Au = apply_pt<T, DIM>(P, u, qk, k, kx, ky);
                return cx<T>{r.re - Au.re, r.im - Au.im};
            };
            const cx<T> zero = {T(0), T(0)};
            const size_t sy = (size_t)P.mx;
            zc = resid(j, ix, iy, qj);
            const cx<T> zw = ix > 0 ? resid(j - 1, ix - 1, iy, q[j - 1]) : zero;
            const cx<T> ze = ix < P.mx - 1 ? resid(j + 1, ix + 1, iy, q[j + 1]) : zero;
            const cx<T> zs = iy > 0 ? resid(j - sy, ix, iy - 1, q[j - sy]) : zero;
            const cx<T> zn = iy < P.my - 1 ? resid(j + sy, ix, iy + 1, q[j + sy]) : zero;
            Wp = apply_point(P, lap_xy(P, zc, zw, ze, zs, zn), zc, qj);
        }
        z0[j] = zc;
        w[j] = Wp;
        const double wr = Wp.re, wi = Wp.im;
        acc[0] += (double)zc.re * (double)zc.re + (double)zc.im * (double)zc.im;
        acc[1] += (double)zc.re * wr + (double)zc.im * wi;
        acc[2] += (double)zc.re * wi - (double)zc.im * wr;
    });
    const int slot[3] = {0, NSLOT_D, NSLOT_D + 1};
    block_partials<3>(acc, slot, parts);
}

// The coefficients of the orthogonalisation of A Z_{J-1} against Z_0 ..
// Z_{J-1}: g_i = d_{i,J-1} / n_i (zero where n_i is).
template <typename T, int J>
__device__ __forceinline__ void orth_coeffs(const double *__restrict__ S, cx<T> (&g)[J])
{
#pragma unroll
    for (int i = 0; i < J; ++i) {
        const double ni = S[i];
        const double dr = S[GM_D + 2 * ((J - 1) * GMRES_MAX_M + i)], di = S[GM_D + 2 * ((J - 1) * GMRES_MAX_M + i) + 1];
        g[i] = cx<T>{T(ni > 0.0 ? dr / ni : 0.0), T(ni > 0.0 ? di / ni : 0.0)};
    }
}

// Z_J = W - sum_{i<J} g_i Z_i at point p (W = A Z_{J-1}).
template <typename T, int J>
__device__ __forceinline__ cx<T> orth_at(const cx<T> *__restrict__ W, const cx<T> *__restrict__ Z, size_t N,
                                         const cx<T> (&g)[J], size_t p)
{
    cx<T> v = W[p];
#pragma unroll
    for (int i = 0; i < J; ++i) {
        const cx<T> zi = Z[(size_t)i * N + p];
        v = cx<T>{v.re - (g[i].re * zi.re - g[i].im * zi.im), v.im - (g[i].re * zi.im + g[i].im * zi.re)};
    }
    return v;
}

// The scalars a fused pass needs to orthogonalise A Z_{J-1} (the previous
// passes' results), into the block's copy Sl of the S layout: n_i (i < J - 1)
// from S, where the first block of an earlier pass left them; n_{J-1} and
// d_{i,J-1} (i < J) summed from the previous passes' partials in the order of
// k_gm_reduce (every block sums them; the first block also stores them in S
// for the later passes).
template <int J>
__device__ __forceinline__ void step_scalars(const double *__restrict__ parts, int nb, double *__restrict__ S,
                                             double *Sl)
{
    constexpr int dcol = GM_D + 2 * ((J - 1) * GMRES_MAX_M);
    if (threadIdx.x < J - 1) Sl[threadIdx.x] = S[threadIdx.x];
    reduce_slots<1>(parts, nb, J - 1, Sl + (J - 1));
    reduce_slots<2 * J>(parts, nb, NSLOT_D + 2 * ((J - 1) * GMRES_MAX_M), Sl + dcol);
    __syncthreads();
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) S[J - 1] = Sl[J - 1];
        if (threadIdx.x < 2 * J) S[dcol + threadIdx.x] = Sl[dcol + threadIdx.x];
    }
}

// One pass for 1 <= J < m: Z_J = A Z_{J-1} - sum_{i<J} g_i Z_i, formed from
// wprev = A Z_{J-1} at the point and its stencil neighbours and stored; wout
// = A Z_J; the partial |Z_J|^2 and <Z_i, A Z_J> (i <= J).  The values and
// partial sums of k_gm_orth<J> followed by k_gm_apply_dots<J + 1>.
template <typename T, int DIM, int J>
__global__ __launch_bounds__(GM_BT) void k_gm_orth_apply(cx<T> *__restrict__ Z, const cx<T> *__restrict__ wprev,
                                                       cx<T> *__restrict__ wout, size_t N,
                                                       const cx<T> *__restrict__ q, Stencil<T> P,
                                                       double *__restrict__ S, double *__restrict__ parts,
                                                       const int *__restrict__ stop)
{
    if (stop && *stop) return;
    __shared__ double Sl[GM_S];
    step_scalars<J>(parts, gridDim.x, S, Sl);
    cx<T> g[J];
    orth_coeffs<T, J>(Sl, g);
    cx<T> *zJ = Z + (size_t)J * N;
    constexpr int NV = 1 + 2 * (J + 1);   // |Z_J|^2, then <Z_i, A Z_J> (re, im) for i <= J
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    // Z_J, A Z_J and the sums at point p from Z_J there and A Z_J
    auto add = [&](size_t p, cx<T> zc, cx<T> Wp) {
        zJ[p] = zc;
        wout[p] = Wp;
        acc[0] += (double)zc.re * (double)zc.re + (double)zc.im * (double)zc.im;
        const double wr = Wp.re, wi = Wp.im;
#pragma unroll
        for (int i = 0; i <= J; ++i) {
            const cx<T> zi = (i < J) ? Z[(size_t)i * N + p] : zc;
            acc[1 + 2 * i] += (double)zi.re * wr + (double)zi.im * wi;
            acc[2 + 2 * i] += (double)zi.re * wi - (double)zi.im * wr;
        }
    };
    if constexpr (DIM == 2) {
        // Z_J of the tile and a point around it through LDS (0 outside the grid),
        // formed once a point: with each point forming its neighbours' 1023^2 took
        // 16.6 us (J = 1) and 21.0 (J = 2), now 14.0 and 15.8, 511^2 8.2 and 9.7, now
        // 7.4 and 8.7 (FP32)
        constexpr int HX = GM_TX + 2, HY = GM_TY + 2;
        __shared__ cx<T> zs[HY * HX];
        const cx<T> zero = {T(0), T(0)};
        const int t = threadIdx.x, lx = t % GM_TX, ly = t / GM_TX;
        // the point around the tile that threads below 2 (GM_TX + GM_TY) add
        const bool ring = t < 2 * (GM_TX + GM_TY);
        const int k = t < 2 * GM_TX ? t : t - 2 * GM_TX;
        const int hx = t < 2 * GM_TX ? k % GM_TX : (k < GM_TY ? -1 : GM_TX);
        const int hy = t < 2 * GM_TX ? (k < GM_TX ? -1 : GM_TY) : k % GM_TY;
        for_points<DIM>(P, N, [&](size_t p, int ix, int iy, bool own) {
            const cx<T> zc = own ? orth_at<T, J>(wprev, Z, N, g, p) : zero;
            cx<T> zh = zero;
            const int gx = ix - lx + hx, gy = iy - ly + hy;
            if (ring && gx >= 0 && gx < P.mx && gy >= 0 && gy < P.my)
                zh = orth_at<T, J>(wprev, Z, N, g, (size_t)gy * P.mx + gx);
            __syncthreads();   // every thread is past its reads of the tile before
            cx<T> *c = zs + (ly + 1) * HX + lx + 1;
            *c = zc;
            if (ring) zs[(hy + 1) * HX + hx + 1] = zh;
            __syncthreads();
            if (own) add(p, zc, apply_point(P, lap_xy(P, zc, c[-1], c[1], c[-HX], c[HX]), zc, q[p]));
        });
    } else {
        for_points<DIM>(P, N, [&](size_t p, int, int, bool) {
            const cx<T> zc = orth_at<T, J>(wprev, Z, N, g, p);
            add(p, zc, apply_at_f<T, DIM>(P, [&](size_t k) { return orth_at<T, J>(wprev, Z, N, g, k); }, zc, q[p], p));
        });
    }
    int slot[NV];
    slot[0] = J;
#pragma unroll
    for (int v = 1; v < NV; ++v) slot[v] = NSLOT_D + 2 * (J * GMRES_MAX_M) + (v - 1);
    block_partials<NV>(acc, slot, parts);
}

// The last Arnoldi vector's partial norm: n_M = |A Z_{M-1} - sum_{i<M} g_i
// Z_i|^2 (the vector itself is not needed).
template <typename T, int DIM, int M>
__global__ __launch_bounds__(GM_BT) void k_gm_orth_norm(const cx<T> *__restrict__ Z, const cx<T> *__restrict__ wprev,
                                                        Stencil<T> P, size_t N, double *__restrict__ S, double *__restrict__ parts,
                                                      const int *__restrict__ stop)
{
    if (stop && *stop) return;
    __shared__ double Sl[GM_S];
    step_scalars<M>(parts, gridDim.x, S, Sl);
    cx<T> g[M];
    orth_coeffs<T, M>(Sl, g);
    double acc[1] = {0.0};
    for_points<DIM>(P, N, [&](size_t p, int, int, bool own) {
        if (!own) return;
        const cx<T> v = orth_at<T, M>(wprev, Z, N, g, p);
        acc[0] += (double)v.re * (double)v.re + (double)v.im * (double)v.im;
    });
    const int slot[1] = {M};
    block_partials<1>(acc, slot, parts);
}

// The small problem and the update u += sum_j c_j Z_j in one pass: every
// block sums n_M from the partials, takes the other scalars from S and solves
// the small problem (the first block also stores n_M and the coefficients).
template <typename T, int M>
__global__ __launch_bounds__(GM_BT) void k_gm_solve_update(cx<T> *__restrict__ u, const cx<T> *__restrict__ Z,
                                                         size_t N, double *__restrict__ S,
                                                         const double *__restrict__ parts,
                                                         const int *__restrict__ stop)
{
    if (stop && *stop) return;
    __shared__ double Sl[GM_S];
    if (threadIdx.x < M) Sl[threadIdx.x] = S[threadIdx.x];
    for (int t = threadIdx.x; t < 2 * M * GMRES_MAX_M; t += GM_BT) Sl[GM_D + t] = S[GM_D + t];
    reduce_slots<1>(parts, gridDim.x, M, Sl + M);
    __syncthreads();
    if (threadIdx.x == 0) gm_solve_small<M>(Sl, Sl + GM_D, Sl + GM_C);
    __syncthreads();
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) S[M] = Sl[M];
        if (threadIdx.x < 2 * M) S[GM_C + threadIdx.x] = Sl[GM_C + threadIdx.x];
    }
    cx<T> c[M];
#pragma unroll
    for (int j = 0; j < M; ++j) c[j] = cx<T>{T(Sl[GM_C + 2 * j]), T(Sl[GM_C + 2 * j + 1])};
    for (size_t p = (size_t)blockIdx.x * GM_BT + threadIdx.x; p < N; p += (size_t)gridDim.x * GM_BT) {
        cx<T> v = u[p];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const cx<T> zj = Z[(size_t)j * N + p];
            v = cx<T>{v.re + (c[j].re * zj.re - c[j].im * zj.im), v.im + (c[j].re * zj.im + c[j].im * zj.re)};
        }
        u[p] = v;
    }
}

// Z_{j+1} = W - sum_{i<=j} (d_ij / n_i) Z_i in place, partial |Z_{j+1}|^2.
template <typename T, int DIM, int NJ>
__global__ __launch_bounds__(GM_BT) void k_gm_orth(cx<T> *__restrict__ Z, Stencil<T> P, size_t N, const double *__restrict__ S,
                                                 double *__restrict__ parts, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    cx<T> g[NJ];
    orth_coeffs<T, NJ>(S, g);
    cx<T> *w = Z + (size_t)NJ * N;
    double acc[1] = {0.0};
    for_points<DIM>(P, N, [&](size_t p, int, int, bool own) {
        if (!own) return;
        const cx<T> v = orth_at<T, NJ>(w, Z, N, g, p);
        w[p] = v;
        acc[0] += (double)v.re * (double)v.re + (double)v.im * (double)v.im;
    });
    const int slot[1] = {NJ};
    block_partials<1>(acc, slot, parts);
}

// out[v] = sum over the nb blocks of the partials of slot0 + v for v < NV (one
// block); SOLVE_M > 0: then the small problem (out lies in S: neither is
// restrict, or the loads of S may come before the store, by the scalar cache).
template <int NV, int SOLVE_M>
__global__ __launch_bounds__(GM_BT) void k_gm_reduce(const double *__restrict__ parts, int nb, int slot0, double *out,
                                                     double *S, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    reduce_slots<NV>(parts, nb, slot0, out);
    if constexpr (SOLVE_M > 0) {
        __syncthreads();
        if (threadIdx.x == 0) gm_solve_small<SOLVE_M>(S, S + GM_D, S + GM_C);
    }
}

// u += sum_j c_j Z_j.
template <typename T, int M>
__global__ __launch_bounds__(GM_BT) void k_gm_update(cx<T> *__restrict__ u, const cx<T> *__restrict__ Z, size_t N,
                                                   const double *__restrict__ S, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    cx<T> c[M];
#pragma unroll
    for (int j = 0; j < M; ++j) c[j] = cx<T>{T(S[GM_C + 2 * j]), T(S[GM_C + 2 * j + 1])};
    for (size_t p = (size_t)blockIdx.x * GM_BT + threadIdx.x; p < N; p += (size_t)gridDim.x * GM_BT) {
        cx<T> v = u[p];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const cx<T> zj = Z[(size_t)j * N + p];
            v = cx<T>{v.re + (c[j].re * zj.re - c[j].im * zj.im), v.im + (c[j].re * zj.im + c[j].im * zj.re)};
        }
        u[p] = v;
    }
}

// A whole GMRES(M) step on a small level in one workgroup of BT threads: the
// same passes, separated by workgroup barriers (global memory written before
// a barrier is seen after it within the workgroup), the sums reduced in LDS
// and the small solve by thread 0.
constexpr int GM_BLOCK_THREADS = 1024;
constexpr int GM_SMALL_THREADS = 256;
constexpr size_t GM_SMALL_POINTS = 1024;   // = GM_REG_PTS * GM_SMALL_THREADS
constexpr size_t GM_BLOCK_MAX_POINTS = 4096;
constexpr size_t GM_RESID_DOTS_POINTS = (size_t)1 << 18;   // k_gm_resid_dots from a guess

template <int NV, int BT>
__device__ __forceinline__ void block_reduce_bt(const double (&acc)[NV], double *out, double *red)
{
    double s[(NV + 3) / 4];
    block_sums<NV, BT / 64>(acc, s, red);
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if ((int)threadIdx.x == wave_sum_lane(v & 3)) out[v] = s[v / 4];
    __syncthreads();
}

template <typename T, int DIM, int NJ, int BT>
__device__ __forceinline__ void gm_block_arnoldi(cx<T> *__restrict__ Z, size_t N, const cx<T> *__restrict__ q,
                                                 const Stencil<T> &P, double *n, double *d,
                                                 double *red)
{
    constexpr int j = NJ - 1;
    const cx<T> *zj = Z + (size_t)j * N;
    cx<T> *w = Z + (size_t)NJ * N;
    double acc[2 * NJ];
#pragma unroll
    for (int v = 0; v < 2 * NJ; ++v) acc[v] = 0.0;
    for (size_t p = threadIdx.x; p < N; p += BT) {
        cx<T> Wp = apply_at<T, DIM>(P, zj, q[p], p);
        w[p] = Wp;
        const double wr = Wp.re, wi = Wp.im;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const cx<T> zi = Z[(size_t)i * N + p];
            acc[2 * i] += (double)zi.re * wr + (double)zi.im * wi;
            acc[2 * i + 1] += (double)zi.re * wi - (double)zi.im * wr;
        }
    }
    block_reduce_bt<2 * NJ, BT>(acc, d + 2 * (j * GMRES_MAX_M), red);
    cx<T> g[NJ];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const double ni = n[i];
        const double dr = d[2 * (j * GMRES_MAX_M + i)], di = d[2 * (j * GMRES_MAX_M + i) + 1];
        g[i] = cx<T>{T(ni > 0.0 ? dr / ni : 0.0), T(ni > 0.0 ? di / ni : 0.0)};
    }
    double nacc[1] = {0.0};
    for (size_t p = threadIdx.x; p < N; p += BT) {
        cx<T> v = w[p];
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const cx<T> zi = Z[(size_t)i * N + p];
            v = cx<T>{v.re - (g[i].re * zi.re - g[i].im * zi.im), v.im - (g[i].re * zi.im + g[i].im * zi.re)};
        }
        w[p] = v;
        nacc[0] += (double)v.re * (double)v.re + (double)v.im * (double)v.im;
    }
    block_reduce_bt<1, BT>(nacc, n + NJ, red);
}

template <typename T, int DIM, int NJ, int M, int BT>
__device__ __forceinline__ void gm_block_arnoldi_all(cx<T> *Z, size_t N, const cx<T> *q, const Stencil<T> &P,
                                                     double *n, double *d, double *red)
{
    gm_block_arnoldi<T, DIM, NJ, BT>(Z, N, q, P, n, d, red);
    if constexpr (NJ < M) gm_block_arnoldi_all<T, DIM, NJ + 1, M, BT>(Z, N, q, P, n, d, red);
}

template <typename T, int DIM, int M, int BT>
__global__ __launch_bounds__(BT) void k_gm_step_block(const cx<T> *__restrict__ b, const cx<T> *__restrict__ q,
                                                        cx<T> *__restrict__ u, int zero, cx<T> *__restrict__ Z,
                                                        Stencil<T> P, size_t N, const int *__restrict__ stop)
{
    if (stop && *stop) return;
    __shared__ double red[2 * GMRES_MAX_M * (BT / 64)];
    __shared__ double n[GMRES_MAX_M + 1], d[2 * GMRES_MAX_M * GMRES_MAX_M], c[2 * GMRES_MAX_M];
    double acc[1] = {0.0};
    for (size_t p = threadIdx.x; p < N; p += BT) {
        cx<T> r = b[p];
        if (zero) {
            u[p] = cx<T>{T(0), T(0)};
        } else {
            cx<T> Au = apply_at<T, DIM>(P, u, q[p], p);
            r = cx<T>{r.re - Au.re, r.im - Au.im};
        }
        Z[p] = r;
        acc[0] += (double)r.re * (double)r.re + (double)r.im * (double)r.im;
    }
    block_reduce_bt<1, BT>(acc, n, red);
    gm_block_arnoldi_all<T, DIM, 1, M, BT>(Z, N, q, P, n, d, red);
    if (threadIdx.x == 0) gm_solve_small<M>(n, d, c);
    __syncthreads();
    cx<T> cc[M];
#pragma unroll
    for (int j = 0; j < M; ++j) cc[j] = cx<T>{T(c[2 * j]), T(c[2 * j + 1])};
    for (size_t p = threadIdx.x; p < N; p += BT) {
        cx<T> v = u[p];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const cx<T> zj = Z[(size_t)j * N + p];
            v = cx<T>{v.re + (cc[j].re * zj.re - cc[j].im * zj.im), v.im + (cc[j].re * zj.im + cc[j].im * zj.re)};
        }
        u[p] = v;
    }
}

// The same step with the level's vectors held in registers (thread t holds
// the points p = t + BT k, k < GM_REG_PTS) and only the vector that A is
// applied to staged in LDS (dynamic shared memory, N + 1 values, the last one
// zero): no global traffic inside the step but the loads of b, q, u and the
// store of u.  The values, the sums and their order are those of
// k_gm_step_block.
//
// Bound by the chain of sums and, with 1024 threads, by one CU's vector rate,
// so what every product needs again is formed once: the LDS offsets of a
// point's neighbours (16 bits each; the zero's where there is none), and one
// division a coefficient instead of one a coefficient and thread.  The sums end
// in every wave (one barrier each); the scalars are wave-uniform registers.
// FP32, m = 3: 31 x 31 9.9 us (15.0 with the neighbours found from each point's
// coordinates, sums by shuffles and the scalars in LDS), 63 x 63 17.5 us (25.6).
constexpr int GM_REG_PTS = (int)(GM_BLOCK_MAX_POINTS / GM_BLOCK_THREADS);   // also for the small blocks
static_assert(2 * GM_BLOCK_MAX_POINTS <= 65535, "neighbour offsets in units of 8 bytes");

template <typename T>
__device__ __forceinline__ cx<T> staged(const cx<T> *stage, unsigned off8)
{
    return *reinterpret_cast<const cx<T> *>(reinterpret_cast<const unsigned char *>(stage) + 8 * off8);
}

// A z at a point from the stage; nb: the point's neighbours, west | east << 16,
// south | north << 16, down | up << 16, in units of 8 bytes.
template <typename T, int DIM>
__device__ __forceinline__ cx<T> apply_staged(const Stencil<T> &P, const cx<T> *stage, unsigned nx, unsigned ny,
                                              unsigned nz, cx<T> zc, cx<T> qj)
{
    cx<T> L = lap_xy(P, zc, staged(stage, nx & 0xffff), staged(stage, nx >> 16), staged(stage, ny & 0xffff),
                     staged(stage, ny >> 16));
    if (DIM == 3) L = lap_add_z(P, L, zc, staged(stage, nz & 0xffff), staged(stage, nz >> 16));
    return apply_point(P, L, zc, qj);
}

// The scalars of the step, the same in every wave.
struct GmScalars {
    double n[GMRES_MAX_M + 1], d[2 * GMRES_MAX_M * GMRES_MAX_M];
};

template <typename T, int DIM, int NJ, int M, int BT>
__device__ __forceinline__ void gm_reg_arnoldi(cx<T> (&Z)[M + 1][GM_REG_PTS], const cx<T> (&qv)[GM_REG_PTS],
                                               cx<T> *stage, const unsigned (&nbr)[3][GM_REG_PTS],
                                               const Stencil<T> &P, int N, GmScalars &sc,
                                               double (&red)[2][2 * M * (BT / 64)])
{
    constexpr int j = NJ - 1, NH = (2 * NJ + 3) / 4;
    // every thread is past its reads of the stage: a block-wide sum came after them
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        if (p < N) stage[p] = Z[j][k];
    }
    __syncthreads();
    double acc[2 * NJ], s[NH];
#pragma unroll
    for (int v = 0; v < 2 * NJ; ++v) acc[v] = 0.0;
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        if (p < N) {
            const cx<T> Wp = apply_staged<T, DIM>(P, stage, nbr[0][k], nbr[1][k], nbr[2][k], Z[j][k], qv[k]);
            Z[NJ][k] = Wp;
            const double wr = Wp.re, wi = Wp.im;
#pragma unroll
            for (int i = 0; i < NJ; ++i) {
                const cx<T> zi = Z[i][k];
                acc[2 * i] += (double)zi.re * wr + (double)zi.im * wi;
                acc[2 * i + 1] += (double)zi.re * wi - (double)zi.im * wr;
            }
        }
    }
    block_sums<2 * NJ, BT / 64>(acc, s, red[1]);
    cx<T> g[NJ];
    const bool odd = (threadIdx.x >> 4) & 1;   // the rows of 16 lanes that hold values 2 and 3 of four
    T gv[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const double ni = 2 * h + 1 < NJ ? (odd ? sc.n[2 * h + 1 < NJ ? 2 * h + 1 : 0] : sc.n[2 * h]) : sc.n[2 * h];
        gv[h] = T(ni > 0.0 ? s[h] / ni : 0.0);
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const int re = wave_sum_lane(2 * (i & 1)), im = wave_sum_lane(2 * (i & 1) + 1);
        sc.d[2 * (j * GMRES_MAX_M + i)] = lane_value(s[i / 2], re);
        sc.d[2 * (j * GMRES_MAX_M + i) + 1] = lane_value(s[i / 2], im);
        g[i] = cx<T>{lane_value(gv[i / 2], re), lane_value(gv[i / 2], im)};
    }
    double nacc[1] = {0.0}, ns[1];
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        if (p < N) {
            cx<T> v = Z[NJ][k];
#pragma unroll
            for (int i = 0; i < NJ; ++i) {
                const cx<T> zi = Z[i][k];
                v = cx<T>{v.re - (g[i].re * zi.re - g[i].im * zi.im), v.im - (g[i].re * zi.im + g[i].im * zi.re)};
            }
            Z[NJ][k] = v;
            nacc[0] += (double)v.re * (double)v.re + (double)v.im * (double)v.im;
        }
    }
    block_sums<1, BT / 64>(nacc, ns, red[0]);
    sc.n[NJ] = lane_value(ns[0], 0);
    if constexpr (NJ < M) gm_reg_arnoldi<T, DIM, NJ + 1, M, BT>(Z, qv, stage, nbr, P, N, sc, red);
}

template <typename T, int DIM, int M, int BT>
__global__ __launch_bounds__(BT) void k_gm_step_reg(const cx<T> *__restrict__ b, const cx<T> *__restrict__ q,
                                                      cx<T> *__restrict__ u, int zero, Stencil<T> P, int N,
                                                      const int *__restrict__ stop)
{
    if (stop && *stop) return;
    extern __shared__ __attribute__((aligned(16))) unsigned char gm_stage_raw[];
    __shared__ double red[2][2 * M * (BT / 64)], c[2 * GMRES_MAX_M];
    cx<T> *stage = reinterpret_cast<cx<T> *>(gm_stage_raw);
    const cx<T> zc = {T(0), T(0)};
    cx<T> qv[GM_REG_PTS], uv[GM_REG_PTS], Z[M + 1][GM_REG_PTS];
    unsigned nbr[3][GM_REG_PTS];
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        qv[k] = uv[k] = zc;
#pragma unroll
        for (int j = 0; j <= M; ++j) Z[j][k] = zc;
        if (p < N) {
            qv[k] = q[p];
            Z[0][k] = b[p];
            if (!zero) {
                uv[k] = u[p];
                stage[p] = uv[k];
            }
        }
    }
    if (threadIdx.x == 0) stage[N] = zc;
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = min((int)threadIdx.x + BT * k, N - 1), sy = P.mx, sz = P.mx * P.my;
        int ix, iy, iz;
        split3((unsigned)p, P.mx, P.my, ix, iy, iz);
        auto off = [&](bool in, int i) { return (unsigned)(sizeof(cx<T>) / 8) * (unsigned)(in ? i : N); };
        nbr[0][k] = off(ix > 0, p - 1) | off(ix < P.mx - 1, p + 1) << 16;
        nbr[1][k] = off(iy > 0, p - sy) | off(iy < P.my - 1, p + sy) << 16;
        nbr[2][k] = DIM == 2 ? 0 : off(iz > 0, p - sz) | off(iz < P.mz - 1, p + sz) << 16;
    }
    __syncthreads();
    GmScalars sc;
    double acc[1] = {0.0}, ns[1];
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        if (p < N) {
            cx<T> r = Z[0][k];
            if (!zero) {
                const cx<T> Au = apply_staged<T, DIM>(P, stage, nbr[0][k], nbr[1][k], nbr[2][k], uv[k], qv[k]);
                r = cx<T>{r.re - Au.re, r.im - Au.im};
            }
            Z[0][k] = r;
            acc[0] += (double)r.re * (double)r.re + (double)r.im * (double)r.im;
        }
    }
    block_sums<1, BT / 64>(acc, ns, red[0]);
    sc.n[0] = lane_value(ns[0], 0);
    gm_reg_arnoldi<T, DIM, 1, M, BT>(Z, qv, stage, nbr, P, N, sc, red);
    if (threadIdx.x == 0) gm_solve_small<M>(sc.n, sc.d, c);
    __syncthreads();
    cx<T> cc[M];
#pragma unroll
    for (int j = 0; j < M; ++j) cc[j] = cx<T>{T(c[2 * j]), T(c[2 * j + 1])};
#pragma unroll
    for (int k = 0; k < GM_REG_PTS; ++k) {
        const int p = (int)threadIdx.x + BT * k;
        if (p < N) {
            cx<T> v = uv[k];
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const cx<T> zj = Z[j][k];
                v = cx<T>{v.re + (cc[j].re * zj.re - cc[j].im * zj.im), v.im + (cc[j].re * zj.im + cc[j].im * zj.re)};
            }
            u[p] = v;
        }
    }
}

// Whether a step on a level of at most GM_BLOCK_MAX_POINTS points keeps its
// vectors in registers: small m (the m + 1 vectors, four points each, within
// the 128 registers a thread of a 1024-thread workgroup has).
template <typename T, int M>
constexpr bool gm_reg_step() { return sizeof(T) == 4 ? M <= 4 : M <= 3; }

template <typename T, int DIM, int M, int BT>
static void launch_step_reg(const cx<T> *b, const cx<T> *q, cx<T> *u, bool zero, const Stencil<T> &P, size_t N,
                            hipStream_t s, const int *stop)
{
    static const bool attr_set = [] {
        (void)hipFuncSetAttribute((const void *)k_gm_step_reg<T, DIM, M, BT>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)((GM_REG_PTS * BT + 1) * sizeof(cx<T>)));
        return true;
    }();
    (void)attr_set;
    hipLaunchKernelGGL((k_gm_step_reg<T, DIM, M, BT>), dim3(1), dim3(BT), (N + 1) * sizeof(cx<T>), s, b, q, u, zero ? 1 : 0,
                       P, (int)N, stop);
}

template <typename T, int DIM, int NJ, int M>
void launch_arnoldi_all(cx<T> *Z, size_t N, const cx<T> *q, const Stencil<T> &P, double *S, double *parts, int nb,
                        hipStream_t s, const int *stop)
{
    constexpr int j = NJ - 1;
    hipLaunchKernelGGL((k_gm_apply_dots<T, DIM, NJ>), dim3(nb), dim3(GM_BT), 0, s, Z, Z + (size_t)NJ * N, N, q, P,
                       parts, stop);
    hipLaunchKernelGGL((k_gm_reduce<2 * NJ, 0>), dim3(1), dim3(GM_BT), 0, s, parts, nb,
                       NSLOT_D + 2 * (j * GMRES_MAX_M), S + GM_D + 2 * (j * GMRES_MAX_M), S, stop);
    hipLaunchKernelGGL((k_gm_orth<T, DIM, NJ>), dim3(nb), dim3(GM_BT), 0, s, Z, P, N, S, parts, stop);
    hipLaunchKernelGGL((k_gm_reduce<1, NJ == M ? M : 0>), dim3(1), dim3(GM_BT), 0, s, parts, nb, NJ, S + NJ, S,
                       stop);
    if constexpr (NJ < M) launch_arnoldi_all<T, DIM, NJ + 1, M>(Z, N, q, P, S, parts, nb, s, stop);
}

// The fused passes for J = 1 .. M - 1 (A Z_{J-1} in slot M + ((J - 1) & 1),
// A Z_J into the other of the two).
template <typename T, int DIM, int J, int M>
void launch_orth_apply_all(cx<T> *Z, size_t N, const cx<T> *q, const Stencil<T> &P, double *S, double *parts, int nb,
                           hipStream_t s, const int *stop)
{
    if constexpr (J < M) {
        hipLaunchKernelGGL((k_gm_orth_apply<T, DIM, J>), dim3(nb), dim3(GM_BT), 0, s, Z,
                           Z + (size_t)(M + ((J - 1) & 1)) * N, Z + (size_t)(M + (J & 1)) * N, N, q, P, S, parts,
                           stop);
        launch_orth_apply_all<T, DIM, J + 1, M>(Z, N, q, P, S, parts, nb, s, stop);
    }
}

template <typename T, int DIM, int M>
void launch_step_m(const LevelGeom &g, const Stencil<T> &P, const cx<T> *b, const cx<T> *q, cx<T> *u, bool zero,
                   cx<T> *Z, double *S, double *parts, hipStream_t s, const int *stop, bool fused)
{
    const size_t N = g.N();
    if (N <= GM_BLOCK_MAX_POINTS) {   // small level: the whole step in one workgroup
        // levels of at most GM_SMALL_POINTS points in a 256-thread workgroup (its
        // block-wide sums take 4 waves instead of 16)
        const bool small = N <= GM_SMALL_POINTS;
        if constexpr (gm_reg_step<T, M>()) {
            if (fused) {
                if (small) launch_step_reg<T, DIM, M, GM_SMALL_THREADS>(b, q, u, zero, P, N, s, stop);
                else launch_step_reg<T, DIM, M, GM_BLOCK_THREADS>(b, q, u, zero, P, N, s, stop);
                return;
            }
        }
        if (small)
            hipLaunchKernelGGL((k_gm_step_block<T, DIM, M, GM_SMALL_THREADS>), dim3(1), dim3(GM_SMALL_THREADS), 0, s,
                               b, q, u, zero ? 1 : 0, Z, P, N, stop);
        else
            hipLaunchKernelGGL((k_gm_step_block<T, DIM, M, GM_BLOCK_THREADS>), dim3(1), dim3(GM_BLOCK_THREADS), 0, s,
                               b, q, u, zero ? 1 : 0, Z, P, N, stop);
        return;
    }
    const size_t runs = DIM == 2 ? (size_t)gm_tiles(P.mx, P.my) : (N + GM_BT - 1) / GM_BT;
    const int nb = (int)std::min<size_t>(runs, GM_BLOCKS);
    // The first two passes as one where that costs less than a launch: from a zero
    // guess the residual is b; else a point forms it five times (2D), up to 2^18
    // points (FP32, two launches against one: 127^2 6.9 us and 4.8, 255^2 6.9
    // and 5.3, 511^2 8.7 and 7.6; 1023^2, where the two take 14, is bound by
    // vector rate instead).
    cx<T> *w0 = Z + (size_t)M * N;
    if (fused && zero)
        hipLaunchKernelGGL((k_gm_resid_dots<T, DIM, true>), dim3(nb), dim3(GM_BT), 0, s, u, b, q, Z, w0, P, N, parts,
                           stop);
    bool paired = fused && zero;
    if constexpr (DIM == 2) {
        if (fused && !zero && N < GM_RESID_DOTS_POINTS) {
            hipLaunchKernelGGL((k_gm_resid_dots<T, DIM, false>), dim3(nb), dim3(GM_BT), 0, s, u, b, q, Z, w0, P, N,
                               parts, stop);
            paired = true;
        }
    }
    if (!paired)
        hipLaunchKernelGGL((k_gm_resid<T, DIM>), dim3(nb), dim3(GM_BT), 0, s, u, zero ? 1 : 0, b, q, Z, P, N, parts,
                           stop);
    if (fused) {
        if (!paired)
            hipLaunchKernelGGL((k_gm_apply_dots<T, DIM, 1>), dim3(nb), dim3(GM_BT), 0, s, Z, w0, N, q, P, parts, stop);
        launch_orth_apply_all<T, DIM, 1, M>(Z, N, q, P, S, parts, nb, s, stop);
        hipLaunchKernelGGL((k_gm_orth_norm<T, DIM, M>), dim3(nb), dim3(GM_BT), 0, s, Z,
                           Z + (size_t)(M + ((M - 1) & 1)) * N, P, N, S, parts, stop);
        hipLaunchKernelGGL((k_gm_solve_update<T, M>), dim3(nb), dim3(GM_BT), 0, s, u, Z, N, S, parts, stop);
        return;
    }
    hipLaunchKernelGGL((k_gm_reduce<1, 0>), dim3(1), dim3(GM_BT), 0, s, parts, nb, 0, S, S, stop);
    launch_arnoldi_all<T, DIM, 1, M>(Z, N, q, P, S, parts, nb, s, stop);
    hipLaunchKernelGGL((k_gm_update<T, M>), dim3(nb), dim3(GM_BT), 0, s, u, Z, N, S, stop);
}

template <typename T, int DIM>
void launch_step_dim(int m, const LevelGeom &g, const Stencil<T> &P, const cx<T> *b, const cx<T> *q, cx<T> *u,
                     bool zero, cx<T> *Z, double *S, double *parts, hipStream_t s, const int *stop, bool fused)
{
    switch (m) {
    case 1: launch_step_m<T, DIM, 1>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 2: launch_step_m<T, DIM, 2>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 3: launch_step_m<T, DIM, 3>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 4: launch_step_m<T, DIM, 4>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 5: launch_step_m<T, DIM, 5>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 6: launch_step_m<T, DIM, 6>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    case 7: launch_step_m<T, DIM, 7>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    default: launch_step_m<T, DIM, 8>(g, P, b, q, u, zero, Z, S, parts, s, stop, fused); break;
    }
}

}  // namespace

// One GMRES(m) smoothing step in place on a level: Z holds m + 2 vectors of
// N points, S the step's scalars (GM_S doubles), parts the partial sums
// (GM_PARTS doubles).  zero: u is 0 on entry (not read).  fused: the
// m + 3-launch passes, else the reference passes.
template <typename T>
void launch_gmres_step(const LevelGeom &g, const Stencil<T> &P, const cx<T> *b, const cx<T> *q, cx<T> *u, bool zero,
                       int m, cx<T> *Z, double *S, double *parts, hipStream_t s, const int *stop, bool fused)
{
    if (g.dim == 3) launch_step_dim<T, 3>(m, g, P, b, q, u, zero, Z, S, parts, s, stop, fused);
    else launch_step_dim<T, 2>(m, g, P, b, q, u, zero, Z, S, parts, s, stop, fused);
}
template void launch_gmres_step<double>(const LevelGeom &, const Stencil<double> &, const cd *, const cd *, cd *, bool,
                                        int, cd *, double *, double *, hipStream_t, const int *, bool);
template void launch_gmres_step<float>(const LevelGeom &, const Stencil<float> &, const cf *, const cf *, cf *, bool,
                                       int, cf *, double *, double *, hipStream_t, const int *, bool);

}  // namespace ffmg
