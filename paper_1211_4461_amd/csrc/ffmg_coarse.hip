// ffmg_coarse.hip -- the exact inverse of the coarsest operator from its block
// structure.
//
// Along its longest axis the coarsest grid is a chain of nb slices of B points
// (B <= 56), and the contour operator couples neighbouring slices by the
// constant -c (c = e^{-2 i gamma} / h^2 of that axis) times the identity:
//   A = tridiag(-c I, D_i, -c I),  D_i the slice's own stencil.
// With the Schur complements from both ends,
//   S_0 = D_0,        S_i = D_i - c^2 S_{i-1}^{-1},
//   T_{nb-1} = D,     T_i = D_i - c^2 T_{i+1}^{-1},
// the inverse's blocks are
//   G_jj = (D_j - c^2 S_{j-1}^{-1} - c^2 T_{j+1}^{-1})^{-1},
//   G_ij = c S_i^{-1} G_{i+1,j} (i < j),  G_ij = c T_i^{-1} G_{i-1,j} (i > j).
// That is 2 nb + nb inversions of B x B blocks, of which only 2 x nb depend on
// each other (two chains that run side by side), and O(n^2 B) products, against
// n dependent pivot steps and O(n^3) for elimination on the whole matrix.  The
// blocks are inverted with partial pivoting; pivots are not exchanged between
// slices, so a chain whose leading slices are close to singular by themselves
// loses digits that the whole matrix has.  The result is therefore held to
// rounding, max |A X - I| <= CB_ROUND eps ||A|| max |X|, and a matrix on which it
// fails is inverted by the pivoted elimination of ffmg_stencil.hip instead.
// Measured in units of eps ||A|| max |X| over random operators (boxes, wavenumbers
// and contrasts over two decades): 7 x 7 at most 2.9 of 200, 15 x 15 3.2 of 100, 31 x 31
// 3.0 of 12, 7 x 7 x 7 median 2.7 and at most 6.4 of 200; the 31 x 31 ionisation
// operators 1.9.  With a first slice singular up to a relative shift of 1e-3, 1e-5,
// 1e-7 on 7 x 15 points 13, 1053, 109054 (elimination: 1).
//
// The two chains are bound by latency (B nb dependent pivot steps of 0.6 us for
// B = 31, 0.8 us for B = 49: a 64-lane arg-max, one reciprocal, one barrier).
// Measured, all kernels of the inverse: 31 x 31 grid 740 us (blocked
// elimination: 7100 us), 7 x 7 x 7 390 us (1350 us), 7 x 7 47 us (193 us).
#include <algorithm>
#include <cmath>

#include "ffmg_internal.hpp"
#include "ffmg_wave.hpp"

namespace ffmg {

namespace {

constexpr int CB_WAVES = 8;                     // waves that share a block's columns
constexpr int CB_MAX = CB_WAVES * 7;             // largest block: seven columns per wave
constexpr int CB_COLS = 8;                      // columns of G a workgroup carries along the chain
constexpr double CB_ROUND = 8.0;                // accepted max |A X - I| over eps ||A|| max |X|
constexpr double CB_TOL = 1e-9;                 // and in any case

// The coarsest grid as nb slices of B = n0 n1 points; point (i0, i1) of slice
// i has the flat index i0 s0 + i1 s1 + i so.
struct CoarseShape {
    int B, nb, n0, n1, s0, s1, so;
    cd c0, c1, co;      // stencil coefficients rot / h^2 of the three axes
    cd csum2;
    double k02;
};

__device__ __forceinline__ int cb_index(const CoarseShape &C, int p, int i)
{
    const int i1 = p / C.n0, i0 = p - i1 * C.n0;
    return i0 * C.s0 + i1 * C.s1 + i * C.so;
}

// Entry (r, k) of a slice's own stencil; qr: the contrast at point r.
__device__ __forceinline__ cd cb_entry(const CoarseShape &C, int r, int k, cd qr)
{
    if (r == k) return C.csum2 - cd{C.k02 + qr.re, qr.im};
    const int r1 = r / C.n0, r0 = r - r1 * C.n0, k1 = k / C.n0, k0 = k - k1 * C.n0;
    if (r1 == k1 && (r0 - k0 == 1 || k0 - r0 == 1)) return cd{-C.c0.re, -C.c0.im};
    if (r0 == k0 && (r1 - k1 == 1 || k1 - r1 == 1)) return cd{-C.c1.re, -C.c1.im};
    return cd{0.0, 0.0};
}

struct CbShared {
    cd f[2][64];        // the pivot column of a step, by row (two steps alternate)
    cd r[2];            // 1 / pivot
    int p[2];           // pivot row
    int perm[CB_MAX];   // pivot row of every step
};

// max over the wave of an unsigned value (0 is the identity)
__device__ __forceinline__ unsigned wave_max(unsigned v)
{
#define CB_STEP(ctrl) v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false))
    CB_STEP(0x111);     // row_shr:1, 2, 4, 8
    CB_STEP(0x112);
    CB_STEP(0x114);
    CB_STEP(0x118);
    CB_STEP(0x142);     // row_bcast:15, 31
    CB_STEP(0x143);
#undef CB_STEP
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ __forceinline__ cd readlane_cd(cd v, int lane) { return cd{lane_value(v.re, lane), lane_value(v.im, lane)}; }

// 1 / a: the hardware reciprocal with two Newton steps (a zero gives NaN).
__device__ __forceinline__ cd cb_recip(cd a)
{
    const double d = __builtin_fma(a.re, a.re, a.im * a.im);
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return cd{a.re * r, -(a.im * r)};
}

__device__ __forceinline__ cd cb_mul(cd a, cd b)
{
    return cd{__builtin_fma(a.re, b.re, -(a.im * b.im)), __builtin_fma(a.re, b.im, a.im * b.re)};
}

// c - a b
__device__ __forceinline__ cd cb_sub(cd c, cd a, cd b)
{
    return cd{__builtin_fma(-a.re, b.re, __builtin_fma(a.im, b.im, c.re)),
              __builtin_fma(-a.re, b.im, __builtin_fma(-a.im, b.re, c.im))};
}

// c + a b
__device__ __forceinline__ cd cb_add(cd c, cd a, cd b)
{
    return cd{__builtin_fma(a.re, b.re, __builtin_fma(-a.im, b.im, c.re)),
              __builtin_fma(a.re, b.im, __builtin_fma(a.im, b.re, c.im))};
}

// The pivot of step k from its column v (row = lane; rows already used are out):
// the largest max(|re|, |im|) to 17 bits, into sh's slot k & 1.
__device__ __forceinline__ void cb_pivot(cd v, bool used, int k, CbShared &sh)
{
    const int lane = threadIdx.x & 63, buf = k & 1;
    const float a = fmaxf(fabsf((float)v.re), fabsf((float)v.im));
    const unsigned key = used ? 0u : ((__float_as_uint(a) & ~63u) | (unsigned)(63 - lane));
    const int p = 63 - (int)(wave_max(key) & 63u);
    const cd r = cb_recip(readlane_cd(v, p));
    sh.f[buf][lane] = v;
    if (lane == 0) {
        sh.p[buf] = p;
        sh.r[buf] = r;
        sh.perm[k] = p;
    }
}

// In-place Gauss-Jordan inversion of a B x B block held by a workgroup of
// CB_WAVES waves: lane r of wave w holds row r's columns w, w + 8, ... in its NS
// slots.  Rows are not exchanged: step k takes its pivot among the rows not yet
// used; afterwards lane r holds row kown(r) (returned) of the inverse, its
// column slot k being column perm[k].  The wave that owns the next column
// updates that one first and finds its pivot before it updates the others.
template <int NS>
__device__ __forceinline__ int cb_invert(cd (&m)[NS], int B, CbShared &sh)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool used = lane >= B;
    int kown = -1;
    if (wave == 0) cb_pivot(m[0], used, 0, sh);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        for (int w = 0; w < CB_WAVES; ++w) {
            const int k = s * CB_WAVES + w, buf = k & 1;
            if (k >= B) break;
            __syncthreads();
            const int p = __builtin_amdgcn_readfirstlane(sh.p[buf]);
            const cd r = sh.r[buf], f = sh.f[buf][lane];
            const bool piv = lane == p;
            if (piv) {
                used = true;
                kown = k;
            }
            auto update = [&](cd &x, bool own) {
                if (own) {
                    const cd t = cb_mul(f, r);
                    x = piv ? r : cd{-t.re, -t.im};
                } else {
                    const cd sc = cb_mul(readlane_cd(x, p), r), y = cb_sub(x, f, sc);
                    x = piv ? sc : y;
                }
            };
            // column k + 1: slot s of the next wave, or slot s + 1 of the first one
            const bool nxt_s = wave == w + 1, nxt_s1 = w + 1 == CB_WAVES && wave == 0;
            if (nxt_s) update(m[s], false);
            if (s + 1 < NS && nxt_s1) update(m[s + 1 < NS ? s + 1 : s], false);
            if (k + 1 < B) {
                if (nxt_s) cb_pivot(m[s], used, k + 1, sh);
                if (s + 1 < NS && nxt_s1) cb_pivot(m[s + 1 < NS ? s + 1 : s], used, k + 1, sh);
            }
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                if ((j == s && nxt_s) || (j == s + 1 && nxt_s1)) continue;
                update(m[j], j == s && wave == w);
            }
        }
    }
    return kown;
}

// The largest magnitudes the check goes by, as FP32 bits: of the inverse's
// entries (the larger of |re| and |im|) and of the operator's diagonal.
struct CbScale {
    unsigned x, diag;
};

__device__ __forceinline__ float cb_abs(cd v) { return fmaxf(fabsf((float)v.re), fabsf((float)v.im)); }

// The two chains: block 0 the S_i from the first slice, block 1 the T_i from
// the last; c S_i^{-1} and c T_i^{-1} go to chain[dir][i] (row-major B x B).
template <int NS>
__global__ __launch_bounds__(64 * CB_WAVES) void k_coarse_chain(CoarseShape C, const cd *__restrict__ q,
                                                                cd *__restrict__ chain, CbScale *__restrict__ scale)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale = CbScale{0u, 0u};   // (the later launches add to it)
    __shared__ CbShared sh;
    __shared__ cd X[NS * CB_WAVES * NS * CB_WAVES];
    const int dir = blockIdx.x, B = C.B;   // B is odd: rows of B values fall on different banks
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool row = lane < B;
    cd *out = chain + (size_t)dir * C.nb * B * B;
    cd qn = row ? q[cb_index(C, lane, dir ? C.nb - 1 : 0)] : cd{0.0, 0.0};
    for (int i = 0; i < C.nb; ++i) {
        const int ib = dir ? C.nb - 1 - i : i;
        const cd qr = qn;
        if (i + 1 < C.nb && row) qn = q[cb_index(C, lane, dir ? ib - 1 : ib + 1)];
        cd m[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int col = j * CB_WAVES + wave;
            m[j] = cd{0.0, 0.0};
            if (row && col < B) {
                m[j] = cb_entry(C, lane, col, qr);
                if (i > 0) m[j] = m[j] - C.co * X[lane * B + col];
            }
        }
        const int kown = cb_invert(m, B, sh);
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int col = j * CB_WAVES + wave;
            if (kown >= 0 && col < B) {
                const cd v = C.co * m[j];
                const int cc = sh.perm[col];
                X[kown * B + cc] = v;
                out[((size_t)ib * B + kown) * B + cc] = v;
            }
        }
        __syncthreads();
    }
}

// The diagonal blocks G_jj of the inverse, one workgroup each.
template <int NS>
__global__ __launch_bounds__(64 * CB_WAVES) void k_coarse_diag(CoarseShape C, const cd *__restrict__ q,
                                                               const cd *__restrict__ chain, cd *__restrict__ G,
                                                               CbScale *__restrict__ scale)
{
    __shared__ CbShared sh;
    const int jb = blockIdx.x, B = C.B;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t BB = (size_t)B * B;
    cd m[NS];
    const cd qr = lane < B ? q[cb_index(C, lane, jb)] : cd{0.0, 0.0};
    if (wave == 0) {
        const unsigned d = wave_max(lane < B ? __float_as_uint(cb_abs(cb_entry(C, lane, lane, qr))) : 0u);
        if (lane == 0) atomicMax(&scale->diag, d);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int col = j * CB_WAVES + wave;
        m[j] = cd{0.0, 0.0};
        if (lane < B && col < B) {
            m[j] = cb_entry(C, lane, col, qr);
            if (jb > 0) m[j] = m[j] - C.co * chain[(jb - 1) * BB + (size_t)lane * B + col];
            if (jb + 1 < C.nb) m[j] = m[j] - C.co * chain[(C.nb + jb + 1) * BB + (size_t)lane * B + col];
        }
    }
    const int kown = cb_invert(m, B, sh);
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int col = j * CB_WAVES + wave;
        if (kown >= 0 && col < B) G[jb * BB + (size_t)kown * B + sh.perm[col]] = m[j];
    }
}

// CB_COLS columns of block column blockIdx.x / ngroups of the inverse, carried
// from the diagonal block towards the first slice (blockIdx.y = 0) or the last
// (1), into the right half of aug (n x 2n).  Lane r forms row r of 2 columns;
// the next slice's factor is loaded into registers during the current product
// and stored to the other of two LDS buffers after it.
__global__ __launch_bounds__(256) void k_coarse_cols(CoarseShape C, const cd *__restrict__ chain,
                                                     const cd *__restrict__ G, cd *__restrict__ aug, int ngroups,
                                                     CbScale *__restrict__ scale)
{
    constexpr int NL = (CB_MAX * CB_MAX + 255) / 256;
    __shared__ cd L[2][CB_MAX * CB_MAX];
    __shared__ cd g[2][64][CB_COLS];
    const int B = C.B, n = B * C.nb, dir = blockIdx.y;
    const int jb = blockIdx.x / ngroups, c0 = (blockIdx.x - jb * ngroups) * CB_COLS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int BB = B * B, lr = min(lane, B - 1);
    const cd zero = {0.0, 0.0};
    const cd *src = chain + (size_t)dir * C.nb * BB;
    cd l[NL];
    auto load = [&](int i) {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (256 * k < BB) l[k] = src[(size_t)i * BB + min(e, BB - 1)];
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (e < BB) L[buf][e] = l[k];
        }
    };
    const int step = dir ? 1 : -1;
    int i = jb + step;
    const bool any = i >= 0 && i < C.nb;
    if (any) load(i);
    int gcol[2];
    float big = 0.f;        // the largest entry this thread forms (rows and columns beyond B repeat others or are 0)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int c = wave * 2 + k, col = c0 + c;
        const cd v = (lane < B && col < B) ? G[(size_t)jb * BB + lane * B + col] : zero;
        big = fmaxf(big, cb_abs(v));
        g[0][lane][c] = v;
        gcol[k] = col < B ? cb_index(C, col, jb) : -1;
        if (dir == 0 && lane < B && gcol[k] >= 0) aug[(size_t)cb_index(C, lane, jb) * 2 * n + n + gcol[k]] = v;
    }
    if (any) stage(0);
    const int row0 = cb_index(C, lr, 0);
    for (int buf = 0; i >= 0 && i < C.nb; i += step, buf ^= 1) {
        __syncthreads();
        const bool more = i + step >= 0 && i + step < C.nb;
        if (more) load(i + step);
        cd a0 = zero, a1 = zero;
#pragma unroll 4
        for (int k = 0; k < B; ++k) {
            const cd x = L[buf][lr * B + k];
            a0 = cb_add(a0, x, g[buf][k][wave * 2]);
            a1 = cb_add(a1, x, g[buf][k][wave * 2 + 1]);
        }
        big = fmaxf(big, fmaxf(cb_abs(a0), cb_abs(a1)));
        g[buf ^ 1][lane][wave * 2] = a0;
        g[buf ^ 1][lane][wave * 2 + 1] = a1;
        if (lane < B) {
            const size_t row = (size_t)(row0 + i * C.so) * 2 * n + n;
            if (gcol[0] >= 0) aug[row + gcol[0]] = a0;
            if (gcol[1] >= 0) aug[row + gcol[1]] = a1;
        }
        if (more) stage(buf ^ 1);
    }
    const unsigned m = wave_max(__float_as_uint(big));
    if (lane == 0) atomicMax(&scale->x, m);
}

// info[0] = -1 if an entry of A X - I is not below its bound (a NaN is not);
// offdiag: the sum of the magnitudes of a row's other entries.
__global__ __launch_bounds__(256) void k_coarse_check(const cd *__restrict__ q, const cd *__restrict__ aug,
                                                      Stencil<double> P, double offdiag,
                                                      const CbScale *__restrict__ scale, int *__restrict__ info)
{
    const int mx = P.mx, my = P.my, mz = P.mz, n = mx * my * mz;
    const int i = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const int ix = i % mx, iy = (i / mx) % my, iz = i / (mx * my);
    const size_t W = 2 * (size_t)n;
    const cd *X = aug + n + j;
    const cd qi = q[i];
    cd r = (P.csum2 - cd{P.k02 + qi.re, qi.im}) * X[i * W];
    if (ix > 0) r = r - P.c[0] * X[(i - 1) * W];
    if (ix + 1 < mx) r = r - P.c[0] * X[(i + 1) * W];
    if (iy > 0) r = r - P.c[1] * X[(i - mx) * W];
    if (iy + 1 < my) r = r - P.c[1] * X[(i + mx) * W];
    if (iz > 0) r = r - P.c[2] * X[(i - mx * my) * W];
    if (iz + 1 < mz) r = r - P.c[2] * X[(i + mx * my) * W];
    if (i == j) r.re -= 1.0;
    const double norm = (double)__uint_as_float(scale->diag) + offdiag;
    const double tol = fmin(CB_ROUND * 0x1p-52 * norm * (double)__uint_as_float(scale->x), CB_TOL);
    if (!(fabs(r.re) < tol && fabs(r.im) < tol)) info[0] = -1;
}

CoarseShape coarse_shape(const LevelGeom &g, const Stencil<double> &P)
{
    int o = 0;
    for (int k = 1; k < 3; ++k)
        if (g.m[k] > g.m[o]) o = k;
    const int a = o == 0 ? 1 : 0, b = o == 2 ? 1 : 2;     // the other axes, the faster one first
    const int st[3] = {1, g.m[0], g.m[0] * g.m[1]};
    CoarseShape C;
    C.n0 = g.m[a];
    C.n1 = g.m[b];
    C.s0 = st[a];
    C.s1 = st[b];
    C.so = st[o];
    C.B = C.n0 * C.n1;
    C.nb = g.m[o];
    C.c0 = P.c[a];
    C.c1 = P.c[b];
    C.co = P.c[o];
    C.csum2 = P.csum2;
    C.k02 = P.k02;
    return C;
}

}  // namespace

// Workspace of launch_coarse_inverse in complex values; 0 where the slices are
// too large for it.
size_t coarse_inverse_ws(const LevelGeom &g)
{
    const int mo = std::max(g.m[0], std::max(g.m[1], g.m[2]));
    const size_t n = g.N(), B = n / mo;
    return B <= CB_MAX ? 3 * n * B + 1 : 0;
}

void launch_coarse_inverse(const LevelGeom &g, const Stencil<double> &P, const cd *q, cd *aug, cd *ws, int *info,
                           hipStream_t s)
{
    const CoarseShape C = coarse_shape(g, P);
    const int n = C.B * C.nb, groups = (C.B + CB_COLS - 1) / CB_COLS;
    cd *chain = ws, *G = ws + 2 * (size_t)n * C.B;
    CbScale *scale = reinterpret_cast<CbScale *>(ws + 3 * (size_t)n * C.B);
    double offdiag = 0.0;
    for (int k = 0; k < 3; ++k)
        if (g.m[k] > 1) offdiag += 2.0 * std::hypot(P.c[k].re, P.c[k].im);
    launch_gj_init(info, s);
#define CB_LAUNCH(NS)                                                                                          \
    do {                                                                                                       \
        hipLaunchKernelGGL(k_coarse_chain<NS>, dim3(2), dim3(64 * CB_WAVES), 0, s, C, q, chain, scale);        \
        hipLaunchKernelGGL(k_coarse_diag<NS>, dim3(C.nb), dim3(64 * CB_WAVES), 0, s, C, q, (const cd *)chain, G, \
                           scale);                                                                             \
    } while (0)
    if (C.B <= CB_WAVES) CB_LAUNCH(1);
    else if (C.B <= 2 * CB_WAVES) CB_LAUNCH(2);
    else if (C.B <= 4 * CB_WAVES) CB_LAUNCH(4);
    else CB_LAUNCH(7);
#undef CB_LAUNCH
    hipLaunchKernelGGL(k_coarse_cols, dim3(C.nb * groups, 2), dim3(256), 0, s, C, (const cd *)chain, (const cd *)G,
                       aug, groups, scale);
    hipLaunchKernelGGL(k_coarse_check, dim3((n + 255) / 256, n), dim3(256), 0, s, q, (const cd *)aug, P, offdiag,
                       (const CbScale *)scale, info);
}

}  // namespace ffmg
