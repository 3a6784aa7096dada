// ffmg_tail2d.hip -- the coarse end of the 2D V-cycle in one workgroup.
//
// Levels of a few thousand points are bound by latency: as launches of their
// own they take 4.5 to 5.5 us each whatever their size, four of them a level.
// k_tail2d runs all levels from the first with at most 4096 points down to the
// exact coarsest solve in one workgroup, on the grids the hierarchy has
// (m = 2^k - 1 points an axis), with
//   - a row of mx points padded to mx + 1 = 2^lp threads, so that a wave holds
//     whole rows, the x-neighbours of a point are the neighbouring lanes (DPP
//     moves, no memory) and the pad lane is the Dirichlet zero;
//   - each thread keeping its points of a level in registers through the
//     sweeps, the residual and the correction; only values that other rows'
//     threads read go through LDS (two arrays a level, alternating, so one
//     barrier a sweep);
//   - a first level of more than 1024 points (the "top") in strips of KS = 2 or
//     4 rows a thread, of which LDS sees the first and the last;
//   - every global load of the kernel issued at its start, the rows of the
//     coarsest inverse among them (up to 64 unknowns).
// Per point the arithmetic is that of the grid-wide kernels (same operation
// order, same summation order in the coarsest solve), so the iterates are the
// same bit for bit.
//
// Bound by the chain of dependent steps (six barriers a level) and, on the top
// level, by one CU's vector rate.  Measured per V-cycle launch, against a form
// that kept every field in LDS: FP64 from 31 x 31 11.6 us (17.3), FP32 from
// 63 x 31 11.6 us (22.1); FP32 from 63 x 63 14.9 us, where that form started at
// 31 x 31 (14.7 us) and the 63 x 63 level took two launches more (9.5 us).
#include <algorithm>

#include "ffmg_internal.hpp"
#include "ffmg_point.hpp"
#include "ffmg_wave.hpp"

namespace ffmg {

namespace {

// v where `in` holds, else 0 (by component: a conditional of the structs may
// become a load through a selected address).
template <typename T>
__device__ __forceinline__ cx<T> masked(bool in, cx<T> v)
{
    return {in ? v.re : T(0), in ? v.im : T(0)};
}

// The x-neighbours of the thread's value v.  Rows of more than 64 threads
// (lp > 6) cross waves: there the edge lanes read the array row that holds v by
// thread (at the row's ends that is a pad lane's zero).
template <typename T>
__device__ __forceinline__ void neighbours_x(cx<T> v, int lp, const cx<T> *row, cx<T> &w, cx<T> &e)
{
    w = {dpp_mov<DPP_WAVE_SHR1>(v.re), dpp_mov<DPP_WAVE_SHR1>(v.im)};
    e = {dpp_mov<DPP_WAVE_SHL1>(v.re), dpp_mov<DPP_WAVE_SHL1>(v.im)};
    if (lp > 6) {
        const int t = threadIdx.x;
        if ((t & 63) == 0 && t > 0) w = row[t - 1];
        if ((t & 63) == 63 && t + 1 < (int)blockDim.x) e = row[t + 1];
    }
}

// A level's place in LDS (levels of one point a thread): two arrays A and B of
// pitch x (my + 1) values, A after a lead of pitch + 1 zeros (row -1 and column
// -1 of what is interpolated from it; row -1 of B is A's last row, zeros too),
// then the right-hand side and q by thread.
template <typename T>
struct TailView {
    cx<T> *A, *B, *b, *q;
    int mx, my, lp, slots;
    __device__ __forceinline__ TailView(cx<T> *lds, const TailLevel<T> &L)
        : mx(L.mx), my(L.my), lp(L.lp), slots((L.my + 1) << L.lp)
    {
        A = lds + L.off + (1 << lp) + 1;
        B = A + slots;
        b = B + slots;
        q = b + slots;
    }
};

// Full weighting at coarse point (I, J) of the residual array R (row pitch 2^lp).
template <typename T>
__device__ __forceinline__ cx<T> full_weight(const cx<T> *R, int lp, int I, int J)
{
    const T w[3] = {T(0.25), T(0.5), T(0.25)};
    const cx<T> *c = R + ((2 * J + 1) << lp) + 2 * I + 1;
    cx<T> acc = {T(0), T(0)};
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
            T wgt = (w[dx + 1] * w[dy + 1]) * T(1);
            acc = acc + wgt * c[dy * (1 << lp) + dx];
        }
    return acc;
}

// The interpolated coarse correction at fine point (x, y), from the coarse
// level's array E (zeros around it); terms in the order of the one-operation
// kernel, zero-weight terms add 0.
template <typename T>
__device__ __forceinline__ cx<T> interp(const cx<T> *E, int clp, int x, int y)
{
    const int fx = x + 1, fy = y + 1;
    const cx<T> *e = E + (((fy >> 1) - 1) * (1 << clp)) + (fx >> 1) - 1;
    const T wx0 = (fx & 1) ? T(0.5) : T(1), wx1 = (fx & 1) ? T(0.5) : T(0);
    const T wy0 = (fy & 1) ? T(0.5) : T(1), wy1 = (fy & 1) ? T(0.5) : T(0);
    cx<T> acc = {T(0), T(0)};
    acc = acc + (wx0 * wy0 * T(1)) * e[0];
    acc = acc + (wx1 * wy0 * T(1)) * e[1];
    acc = acc + (wx0 * wy1 * T(1)) * e[1 << clp];
    acc = acc + (wx1 * wy1 * T(1)) * e[(1 << clp) + 1];
    return acc;
}

// Right-hand side of the next level from the residual array R of this one: by
// thread, or in flat order for the coarsest (its solve reads it across threads).
template <typename T>
__device__ __forceinline__ void restrict_to(const TailParams<T> &tp, cx<T> *lds, int i, const cx<T> *R, int lp)
{
    const TailView<T> c(lds, tp.lv[i]);
    const int tid = threadIdx.x, I = tid & ((1 << c.lp) - 1), J = tid >> c.lp;
    if (tid >= c.slots) return;
    const bool in = I < c.mx && J < c.my;
    const cx<T> v = masked(in, full_weight(R, lp, min(I, c.mx - 1), min(J, c.my - 1)));
    if (i + 1 < tp.nt) c.b[tid] = v;
    else if (in) c.b[J * c.mx + I] = v;
}

// The coarsest inverse (up to 64 unknowns) on its way to LDS, behind the levels.
// NT: the least number of threads.
constexpr int INV_MAX_N = 64;
template <int NT>
struct CoarseInverse {
    static constexpr int K = INV_MAX_N * INV_MAX_N / NT;
    cd a[K];
    __device__ __forceinline__ void load(const cd *__restrict__ aug, int n)
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            a[k] = cd{0.0, 0.0};
            const int e = min((int)(threadIdx.x + blockDim.x * k), n * n - 1), r = e / n;
            if ((int)blockDim.x * k < n * n) a[k] = aug[(size_t)r * 2 * n + n + e - r * n];
        }
    }
    __device__ __forceinline__ void store(cd *lds, int n) const
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = threadIdx.x + blockDim.x * k;
            if (e < n * n) lds[e] = a[k];
        }
    }
};
template <int KS>
constexpr int TAIL_NT = KS > 1 ? 1024 : 512;

// Coarsest level: u = A^{-1} b in FP64, eight lanes a row, lane m the columns
// m, m + 8, ...; summed over columns 64 apart, then over column distances 32,
// 16, 8, 4, 2, 1 (the order of the one-operation kernel).  ainv: the inverse in
// LDS, or null (then it is read from global memory).
template <typename T>
__device__ __forceinline__ void tail_coarsest(const TailParams<T> &tp, cx<T> *lds, const cd *ainv)
{
    const TailView<T> c(lds, tp.lv[tp.nt - 1]);
    const int n = tp.nc, m = threadIdx.x & 7;
    for (int row = threadIdx.x >> 3; row < n; row += blockDim.x >> 3) {
        double re[8], im[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) re[t] = im[t] = 0.0;
        auto add = [&](int t, int k, cd a) {
            const cx<T> bk = c.b[k];
            const double br = (double)bk.re, bi = (double)bk.im;
            re[t] += a.re * br - a.im * bi;
            im[t] += a.re * bi + a.im * br;
        };
        if (ainv) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int k = m + 8 * t;
                if (k < n) add(t, k, ainv[row * n + k]);
            }
        } else {
            const cd *g = tp.aug + (size_t)row * 2 * n + n;
            for (int k0 = m; k0 < n; k0 += 64) {
                cd a[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) a[t] = g[min(k0 + 8 * t, n - 1)];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (k0 + 8 * t < n) add(t, k0 + 8 * t, a[t]);
            }
        }
#pragma unroll
        for (int h = 4; h > 0; h >>= 1)
#pragma unroll
            for (int t = 0; t < h; ++t) {
                re[t] += re[t + h];
                im[t] += im[t + h];
            }
        double r = re[0], s = im[0];
        r += dpp_mov<DPP_ROW_SHL + 4>(r);
        s += dpp_mov<DPP_ROW_SHL + 4>(s);
        r += dpp_mov<DPP_ROW_SHL + 2>(r);
        s += dpp_mov<DPP_ROW_SHL + 2>(s);
        r += dpp_mov<DPP_ROW_SHL + 1>(r);
        s += dpp_mov<DPP_ROW_SHL + 1>(s);
        if (m == 0) {
            const int y = row / c.mx;
            c.A[(y << c.lp) + row - y * c.mx] = cx<T>{T(r), T(s)};
        }
    }
}

// One V-cycle from level i0 (one point a thread; its right-hand side in place;
// zero_top: from a zero guess, else from the guess in its array A): down to the
// coarsest level, every coarser level from a zero guess, and back up.  The
// result is in A of level i0, behind a barrier.  The sweep weight of a pad is 0,
// so its value stays 0.  KEEPQ: the levels are visited
// again, so their q stays (else the sweep weight takes its place).
template <typename T, bool KEEPQ>
__device__ __forceinline__ void tail_vcycle(const TailParams<T> &tp, cx<T> *lds, int i0, bool zero_top,
                                            const cd *ainv)
{
    const int nt = tp.nt, tid = threadIdx.x, nu1 = tp.nu1, nu2 = tp.nu2;
    const cx<T> zero = {T(0), T(0)};
#pragma unroll 1
    for (int i = i0; i + 1 < nt; ++i) {
        const TailLevel<T> &L = tp.lv[i];
        const TailView<T> v(lds, L);
        const int pitch = 1 << v.lp, x = tid & (pitch - 1), y = tid >> v.lp;
        const bool act = tid < v.slots, in = act && x < v.mx && y < v.my;
        const int north = y < v.my ? tid + pitch : tid;     // (the pad row has none)
        const bool from0 = zero_top || i > i0;
        cx<T> u = zero, b = zero, q = zero, w = zero;
        if (act) {
            b = v.b[tid];
            q = v.q[tid];
            w = masked(in, jweight(L.P, q));
        }
        int s = 0, cur = 0;     // cur: the array (0 A, 1 B) that holds u
        if (from0) {
            if (nu1 > 0) {
                u = jacobi0_w(b, w);
                s = 1;
            }
            if (act) v.A[tid] = u;
        } else if (act) {
            u = v.A[tid];
        }
        __syncthreads();
#pragma unroll 1
        for (; s < nu1; ++s) {
            const cx<T> *src = cur ? v.B : v.A;
            cx<T> *dst = cur ? v.A : v.B;
            cx<T> we, ea;
            neighbours_x(u, v.lp, src, we, ea);
            if (act) {
                u = jacobi_point<T>(L.P, u, we, ea, src[tid - pitch], src[north], b, w);
                dst[tid] = u;
            }
            cur ^= 1;
            __syncthreads();
        }
        {
            const cx<T> *src = cur ? v.B : v.A;
            cx<T> *R = cur ? v.A : v.B;
            cx<T> we, ea;
            neighbours_x(u, v.lp, src, we, ea);
            if (act) {
                const cx<T> r = resid_point<T>(L.P, u, we, ea, src[tid - pitch], src[north], b, q);
                R[tid] = masked(in, r);
                if (!KEEPQ) v.q[tid] = w;
            }
            __syncthreads();
            restrict_to(tp, lds, i + 1, R, v.lp);
        }
    }
    __syncthreads();
    tail_coarsest(tp, lds, ainv);
    __syncthreads();
#pragma unroll 1
    for (int i = nt - 2; i >= i0; --i) {
        const TailLevel<T> &L = tp.lv[i];
        const TailView<T> v(lds, L), c(lds, tp.lv[i + 1]);
        const int pitch = 1 << v.lp, x = tid & (pitch - 1), y = tid >> v.lp;
        const bool act = tid < v.slots, in = act && x < v.mx && y < v.my;
        const int north = y < v.my ? tid + pitch : tid;     // (the pad row has none)
        // where the pre-smoothing left u: its writes alternate from A (zero
        // guess) or from B (the guess was in A)
        const bool from0 = zero_top || i > i0;
        const int at = nu1 == 0 ? 0 : from0 ? (nu1 - 1) & 1 : nu1 & 1;
        cx<T> u = zero, b = zero, w = zero;
        if (act) {
            const cx<T> *at_u = at ? v.B : v.A;
            u = at_u[tid];
            b = v.b[tid];
            const cx<T> qw = v.q[tid];
            if (KEEPQ) w = masked(in, jweight(L.P, qw));
            else w = qw;
        }
        if (in) u = u + interp(c.A, c.lp, x, y);
        int cur = nu2 & 1;      // so that the last sweep writes A
        cx<T> *first = cur ? v.B : v.A;
        if (act) first[tid] = u;
        __syncthreads();
#pragma unroll 1
        for (int s = 0; s < nu2; ++s) {
            const cx<T> *src = cur ? v.B : v.A;
            cx<T> *dst = cur ? v.A : v.B;
            cx<T> we, ea;
            neighbours_x(u, v.lp, src, we, ea);
            if (act) {
                u = jacobi_point<T>(L.P, u, we, ea, src[tid - pitch], src[north], b, w);
                dst[tid] = u;
            }
            cur ^= 1;
            __syncthreads();
        }
    }
}

// The first level when it has 2048 or 4096 padded points: thread (strip, x)
// holds KS consecutive rows of column x.  Two LDS buffers take the strips'
// first and last rows by turns; the residual array overlays both.
template <typename T, int KS>
struct TailTop {
    static constexpr int NT = 1024;
    cx<T> u[KS], b[KS], w[KS], q[KS];
    cx<T> *buf;
    int mx, my, lp, x, strip;

    __device__ __forceinline__ TailTop(cx<T> *lds, const TailLevel<T> &L) : mx(L.mx), my(L.my), lp(L.lp)
    {
        buf = lds + L.off;
        x = threadIdx.x & ((1 << lp) - 1);
        strip = threadIdx.x >> lp;
    }
    __device__ __forceinline__ bool in(int r) const { return x < mx && strip * KS + r < my; }
    __device__ __forceinline__ void publish(int k)
    {
        buf[2 * k * NT + threadIdx.x] = u[0];
        buf[(2 * k + 1) * NT + threadIdx.x] = u[KS - 1];
    }
    // row r of the strips in buffer k (KS = 2: every row is there; only these
    // have rows of more than 64 threads)
    __device__ __forceinline__ const cx<T> *row(int k, int r) const { return buf + (2 * k + (r > 0)) * NT; }
    // the row before the strip and the row after it
    __device__ __forceinline__ void edges(int k, cx<T> &s, cx<T> &n) const
    {
        const int pitch = 1 << lp, t = threadIdx.x;
        s = n = cx<T>{T(0), T(0)};
        if (t >= pitch) s = buf[(2 * k + 1) * NT + t - pitch];
        if (t + pitch < NT) n = buf[2 * k * NT + t + pitch];
    }
    __device__ __forceinline__ void sweep(const Stencil<T> &P, int k)
    {
        cx<T> s, n;
        edges(k, s, n);
#pragma unroll
        for (int r = 0; r < KS; ++r) {
            const cx<T> uc = u[r], up = r + 1 < KS ? u[r + 1 < KS ? r + 1 : r] : n;
            cx<T> we, ea;
            neighbours_x(uc, lp, row(k, r), we, ea);
            u[r] = jacobi_point<T>(P, uc, we, ea, s, up, b[r], w[r]);
            s = uc;
        }
    }
    // pre-smoothing (zero: from a zero guess, else from u), the residual and
    // its full weighting into level 1's right-hand side
    __device__ __forceinline__ void down(const TailParams<T> &tp, cx<T> *lds, bool from0)
    {
        const Stencil<T> &P = tp.lv[0].P;
        int s = 0, k = 0;
        if (from0) {
#pragma unroll
            for (int r = 0; r < KS; ++r) u[r] = masked(tp.nu1 > 0, jacobi0_w(b[r], w[r]));
            s = 1;
        } else {
            __syncthreads();    // the buffer may still be read
        }
        publish(0);
        __syncthreads();
#pragma unroll 1
        for (; s < tp.nu1; ++s) {
            sweep(P, k);
            k ^= 1;
            publish(k);
            __syncthreads();
        }
        cx<T> so, n, res[KS];
        edges(k, so, n);
#pragma unroll
        for (int r = 0; r < KS; ++r) {
            const cx<T> uc = u[r], up = r + 1 < KS ? u[r + 1 < KS ? r + 1 : r] : n;
            cx<T> we, ea;
            neighbours_x(uc, lp, row(k, r), we, ea);
            res[r] = resid_point<T>(P, uc, we, ea, so, up, b[r], q[r]);   // (a pad's is not read)
            so = uc;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KS; ++r) buf[((strip * KS + r) << lp) + x] = res[r];
        __syncthreads();
        restrict_to(tp, lds, 1, buf, lp);
    }
    // the correction from level 1 and post-smoothing
    __device__ __forceinline__ void up(const TailParams<T> &tp, cx<T> *lds, bool add)
    {
        const TailView<T> c(lds, tp.lv[1]);
#pragma unroll
        for (int r = 0; r < KS; ++r) {
            const cx<T> e = interp(c.A, c.lp, x, strip * KS + r);
            u[r] = masked(in(r), add ? cx<T>{u[r].re + e.re, u[r].im + e.im} : e);
        }
        if (!add) return;
        int k = 0;
#pragma unroll 1
        for (int s = 0; s < tp.nu2; ++s) {
            publish(k);
            __syncthreads();
            sweep(tp.lv[0].P, k);
            k ^= 1;
        }
    }
};

// What every thread loads from global memory at the kernel's start besides the
// first level's fields: q of the levels with one point a thread, and its part of
// the coarsest inverse.  While the loads are in flight, clear() writes the zeros
// around the levels' arrays; store() then puts the values in place.
template <typename T>
__device__ __forceinline__ cx<T> load_point(const cx<T> *p, const TailLevel<T> &L)
{
    const int t = threadIdx.x, x = t & ((1 << L.lp) - 1), y = t >> L.lp;
    return ld_masked(p, (size_t)(y * L.mx + x), x < L.mx && y < L.my);
}

template <typename T, int KS>
struct TailLoads {
    static constexpr int FIRST = KS > 1;    // the top level keeps its q in registers
    cx<T> q[TAIL_MAX_LEVELS];
    CoarseInverse<TAIL_NT<KS>> ci;

    // cycles: whether V-cycles follow (the coarsest solve alone needs no q)
    __device__ __forceinline__ void load(const TailParams<T> &tp, const cd *ainv, bool cycles = true)
    {
#pragma unroll
        for (int i = FIRST; i < TAIL_MAX_LEVELS; ++i)
            if (cycles && i + 1 < tp.nt) q[i] = load_point(tp.lv[i].q, tp.lv[i]);
        if (ainv) ci.load(tp.aug, tp.nc);
    }
    // (the coarsest level's whole array: its solve writes the interior only)
    __device__ __forceinline__ void clear(const TailParams<T> &tp, cx<T> *lds)
    {
#pragma unroll 1
        for (int i = FIRST; i < tp.nt; ++i) {
            const TailView<T> v(lds, tp.lv[i]);
            const int lead = (1 << v.lp) + 1, n = i + 1 < tp.nt ? lead : lead + v.slots;
            for (int j = threadIdx.x; j < n; j += blockDim.x) v.A[j - lead] = cx<T>{T(0), T(0)};
        }
    }
    __device__ __forceinline__ void store(const TailParams<T> &tp, cx<T> *lds, cd *ainv, bool cycles = true)
    {
#pragma unroll
        for (int i = FIRST; i < TAIL_MAX_LEVELS; ++i)
            if (cycles && i + 1 < tp.nt) {
                const TailView<T> v(lds, tp.lv[i]);
                if ((int)threadIdx.x < v.slots) v.q[threadIdx.x] = q[i];
            }
        if (ainv) ci.store(ainv, tp.nc);
    }
};

// Where the coarsest inverse goes in LDS; null where it stays in global memory.
template <typename T>
__device__ __forceinline__ cd *inverse_at(const TailParams<T> &tp, cx<T> *lds)
{
    return tp.nc <= INV_MAX_N ? reinterpret_cast<cd *>(lds + tp.inv_off) : nullptr;
}

// One V-cycle of the tail: b_top, u_top the first level's right-hand side and
// correction (zero: from a zero guess, u_top is only written).
template <typename T, int KS>
__device__ __forceinline__ void tail2d_body(const TailParams<T> &tp, const cx<T> *__restrict__ b_top,
                                            cx<T> *__restrict__ u_top, bool zero, const int *__restrict__ stop,
                                            cx<T> *lds)
{
    const int st = stop ? *stop : 0;
    TailLoads<T, KS> ld;
    const TailLevel<T> &L0 = tp.lv[0];
    cd *ainv = inverse_at(tp, lds);
    if constexpr (KS > 1) {
        TailTop<T, KS> top(lds, L0);
#pragma unroll
        for (int r = 0; r < KS; ++r) {
            const size_t j = (size_t)(top.strip * KS + r) * L0.mx + top.x;
            top.b[r] = ld_masked(b_top, j, top.in(r));
            top.q[r] = ld_masked(L0.q, j, top.in(r));
            if (!zero) top.u[r] = ld_masked((const cx<T> *)u_top, j, top.in(r));
        }
        ld.load(tp, ainv);
        ld.clear(tp, lds);
        if (st) return;
        ld.store(tp, lds, ainv);
#pragma unroll
        for (int r = 0; r < KS; ++r) top.w[r] = masked(top.in(r), jweight(L0.P, top.q[r]));
        top.down(tp, lds, zero);
        tail_vcycle<T, false>(tp, lds, 1, true, ainv);
        top.up(tp, lds, true);
#pragma unroll
        for (int r = 0; r < KS; ++r)
            if (top.in(r)) u_top[(size_t)(top.strip * KS + r) * L0.mx + top.x] = top.u[r];
    } else {
        const TailView<T> v(lds, L0);
        const int t = threadIdx.x, x = t & ((1 << v.lp) - 1), y = t >> v.lp;
        const cx<T> b = load_point(b_top, L0);
        cx<T> u = {T(0), T(0)};
        if (!zero) u = load_point((const cx<T> *)u_top, L0);
        ld.load(tp, ainv);
        ld.clear(tp, lds);
        if (st) return;
        ld.store(tp, lds, ainv);
        if (t < v.slots) {
            v.b[t] = b;
            if (!zero) v.A[t] = u;
        }
        __syncthreads();    // the zeros
        tail_vcycle<T, false>(tp, lds, 0, zero, ainv);
        if (x < v.mx && y < v.my) u_top[(size_t)y * v.mx + x] = v.A[t];
    }
}

// Full multigrid start on the tail's levels: b of the first level from b_top,
// injected down to the coarsest, exact solve there, then on each level up to the
// first the interpolated coarser solution as the guess and k V-cycles; u_top
// receives the first level's solution.
template <typename T, int KS>
__device__ __forceinline__ void tail2d_fmg_body(const TailParams<T> &tp, const cx<T> *__restrict__ b_top,
                                                cx<T> *__restrict__ u_top, int k, const int *__restrict__ stop,
                                                cx<T> *lds)
{
    if (stop && *stop) return;
    const int nt = tp.nt, tid = threadIdx.x;
    const TailLevel<T> &L0 = tp.lv[0];
    constexpr int first = KS > 1 ? 1 : 0;
    cd *ainv = inverse_at(tp, lds);
    {
        TailLoads<T, KS> ld;
        ld.load(tp, ainv, k > 0);
        ld.clear(tp, lds);
        ld.store(tp, lds, ainv, k > 0);
    }
    // point (x, y) of level i is point (2^i (x + 1) - 1, 2^i (y + 1) - 1) of level
    // 0; without cycles only the coarsest level's right-hand side is read
#pragma unroll 1
    for (int i = k > 0 ? first : nt - 1; i < nt; ++i) {
        const TailView<T> v(lds, tp.lv[i]);
        const int x = tid & ((1 << v.lp) - 1), y = tid >> v.lp;
        const bool in = x < v.mx && y < v.my;
        const cx<T> bi = ld_masked(b_top, (size_t)(((y + 1) << i) - 1) * L0.mx + ((x + 1) << i) - 1, in);
        if (i + 1 < nt) {
            if (tid < v.slots) v.b[tid] = bi;
        } else if (in) {
            v.b[y * v.mx + x] = bi;
        }
    }
    TailTop<T, (KS > 1 ? KS : 2)> top(lds, L0);
    __syncthreads();
    tail_coarsest(tp, lds, ainv);
    __syncthreads();
#pragma unroll 1
    for (int i = nt - 2; i >= 0; --i) {
        const bool at_top = KS > 1 && i == 0;
        if (at_top) {
            if constexpr (KS > 1) {
#pragma unroll
                for (int r = 0; r < KS; ++r) {
                    if (k == 0) break;
                    const size_t j = (size_t)(top.strip * KS + r) * L0.mx + top.x;
                    top.b[r] = ld_masked(b_top, j, top.in(r));
                    top.q[r] = ld_masked(L0.q, j, top.in(r));
                    top.w[r] = masked(top.in(r), jweight(L0.P, top.q[r]));
                }
                top.up(tp, lds, false);
            }
        } else {
            const TailView<T> v(lds, tp.lv[i]), c(lds, tp.lv[i + 1]);
            const int x = tid & ((1 << v.lp) - 1), y = tid >> v.lp;
            if (tid < v.slots) {
                cx<T> u = {T(0), T(0)};
                if (x < v.mx && y < v.my) u = interp(c.A, c.lp, x, y);
                v.A[tid] = u;
            }
        }
#pragma unroll 1
        for (int c2 = 0; c2 < k; ++c2) {
            if constexpr (KS > 1) {
                if (at_top) top.down(tp, lds, false);
            }
            tail_vcycle<T, true>(tp, lds, at_top ? 1 : i, at_top, ainv);
            if constexpr (KS > 1)
                if (at_top) top.up(tp, lds, true);
        }
        if (k == 0) __syncthreads();    // (a V-cycle ends with one)
    }
    if constexpr (KS > 1) {
#pragma unroll
        for (int r = 0; r < KS; ++r)
            if (top.in(r)) u_top[(size_t)(top.strip * KS + r) * L0.mx + top.x] = top.u[r];
    } else {
        const TailView<T> v(lds, L0);
        const int x = tid & ((1 << v.lp) - 1), y = tid >> v.lp;
        if (x < v.mx && y < v.my) u_top[(size_t)y * v.mx + x] = v.A[tid];
    }
}

template <typename T>
__device__ __forceinline__ cx<T> *tail_lds()
{
    extern __shared__ __attribute__((aligned(16))) unsigned char tail_lds_bytes[];
    return reinterpret_cast<cx<T> *>(tail_lds_bytes);
}

template <typename T, int KS>
__global__ __launch_bounds__(1024) void k_tail2d(TailParams<T> tp, const cx<T> *__restrict__ b_top,
                                                 cx<T> *__restrict__ u_top, bool zero, const int *__restrict__ stop)
{
    tail2d_body<T, KS>(tp, b_top, u_top, zero, stop, tail_lds<T>());
}

template <typename T, int KS>
__global__ __launch_bounds__(1024) void k_tail2d_fmg(TailParams<T> tp, const cx<T> *__restrict__ b_top,
                                                     cx<T> *__restrict__ u_top, int k)
{
    tail2d_fmg_body<T, KS>(tp, b_top, u_top, k, nullptr, tail_lds<T>());
}

// one workgroup per instance
template <typename T, int KS>
__global__ __launch_bounds__(1024) void k_tail2d_batch(const TailJob<T> *__restrict__ jobs)
{
    const TailJob<T> &J = jobs[blockIdx.x];
    tail2d_body<T, KS>(J.tp, J.b_top, J.u_top, true, J.stop, tail_lds<T>());
}

template <typename T, int KS>
__global__ __launch_bounds__(1024) void k_tail2d_fmg_batch(const TailJob<T> *__restrict__ jobs, int k)
{
    const TailJob<T> &J = jobs[blockIdx.x];
    tail2d_fmg_body<T, KS>(J.tp, J.b_top, J.u_top, k, J.stop, tail_lds<T>());
}

int tail_slots(int mx, int my) { return (mx + 1) * (my + 1); }

// rows a thread holds of the first level
template <typename T>
int tail_ks(const TailParams<T> &tp)
{
    const int s = tail_slots(tp.lv[0].mx, tp.lv[0].my);
    return s > 2048 ? 4 : s > 1024 ? 2 : 1;
}

// 1024 threads, or 512 where no level has more than 512 padded points
template <typename T>
int tail_threads(const TailParams<T> &tp)
{
    return tail_slots(tp.lv[0].mx, tp.lv[0].my) > 512 ? 1024 : 512;
}

// The 160 KB limit of a kernel's dynamic LDS, raised once per kernel (a
// thread-safe static initialisation).
template <typename K>
bool raise_lds(K *kernel)
{
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, TAIL_LDS_BUDGET);
    return true;
}
#define TAIL_RAISED(kernel)                        \
    do {                                           \
        static const bool raised = raise_lds(kernel); \
        (void)raised;                              \
    } while (0)

}  // namespace

size_t tail_level_elems(int mx, int my, bool first)
{
    const int s = tail_slots(mx, my);
    if (first && s > 1024) return 4 * 1024;
    return 4 * (size_t)s + mx + 2;
}

// Levels of up to 1024 padded points; in FP32 the first one up to 4096 (2048
// with rows of more than 64).  Measured per V-cycle on 63 x 63: FP32 13.2 us in
// the tail against 9.1 us of the tail from 31 x 31 and two launches of 4.7 us
// for the level; FP64 28.8 against 10.8 and two of 5.5 (one CU's FP64 rate binds).
bool tail_level_fits(int mx, int my, bool first, bool fp32)
{
    const int s = tail_slots(mx, my);
    if (s <= 1024) return mx <= 255;
    return first && fp32 && (mx <= 63 ? s <= 4096 : mx <= 255 && s <= 2048);
}

template <typename T>
size_t tail_layout(TailParams<T> &tp)
{
    size_t off = 0;
    const size_t inv = tp.nc <= INV_MAX_N ? (size_t)tp.nc * tp.nc : 0;
    for (int i = 0; i < tp.nt; ++i) {
        TailLevel<T> &L = tp.lv[i];
        L.lp = 0;
        while ((1 << L.lp) < L.mx + 1) ++L.lp;
        L.off = (int)off;
        off += tail_level_elems(L.mx, L.my, i == 0);
    }
    off += off & 1;         // (the inverse is FP64: 16-byte aligned)
    tp.inv_off = (int)off;
    off += inv * (sizeof(cd) / sizeof(cx<T>));
    return off * sizeof(cx<T>);
}
template size_t tail_layout<double>(TailParams<double> &);
template size_t tail_layout<float>(TailParams<float> &);

template <typename T>
void launch_tail2d(const TailParams<T> &tp, size_t lds_bytes, const cx<T> *b_top, cx<T> *u_top, bool zero,
                   hipStream_t s, const int *stop)
{
#define TAIL_GO(KS)                                                                                             \
    do {                                                                                                        \
        TAIL_RAISED((k_tail2d<T, KS>));                                                                         \
        hipLaunchKernelGGL((k_tail2d<T, KS>), dim3(1), dim3(tail_threads(tp)), lds_bytes, s, tp, b_top, u_top,  \
                           zero, stop);                                                                         \
    } while (0)
    const int ks = tail_ks(tp);
    if constexpr (sizeof(T) == 4) {
        if (ks == 4) TAIL_GO(4);
        else if (ks == 2) TAIL_GO(2);
        else TAIL_GO(1);
    } else {
        TAIL_GO(1);
    }
#undef TAIL_GO
}
template void launch_tail2d<double>(const TailParams<double> &, size_t, const cd *, cd *, bool, hipStream_t,
                                    const int *);
template void launch_tail2d<float>(const TailParams<float> &, size_t, const cf *, cf *, bool, hipStream_t,
                                   const int *);

template <typename T>
void launch_tail2d_fmg(const TailParams<T> &tp, size_t lds_bytes, const cx<T> *b_top, cx<T> *u_top, int k,
                       hipStream_t s)
{
#define TAIL_GO(KS)                                                                                              \
    do {                                                                                                         \
        TAIL_RAISED((k_tail2d_fmg<T, KS>));                                                                      \
        hipLaunchKernelGGL((k_tail2d_fmg<T, KS>), dim3(1), dim3(tail_threads(tp)), lds_bytes, s, tp, b_top, u_top, \
                           k);                                                                                   \
    } while (0)
    const int ks = tail_ks(tp);
    if constexpr (sizeof(T) == 4) {
        if (ks == 4) TAIL_GO(4);
        else if (ks == 2) TAIL_GO(2);
        else TAIL_GO(1);
    } else {
        TAIL_GO(1);
    }
#undef TAIL_GO
}
template void launch_tail2d_fmg<double>(const TailParams<double> &, size_t, const cd *, cd *, int, hipStream_t);
template void launch_tail2d_fmg<float>(const TailParams<float> &, size_t, const cf *, cf *, int, hipStream_t);

// tp: any job's parameters (the jobs' levels have the same shapes); njobs = 0
// only raises the kernels' LDS limit (before a stream capture).
template <typename T>
void launch_tail2d_batch(const TailParams<T> &tp, const TailJob<T> *jobs, int njobs, size_t lds_bytes, hipStream_t s)
{
#define TAIL_GO(KS)                                                                                            \
    do {                                                                                                       \
        TAIL_RAISED((k_tail2d_batch<T, KS>));                                                                  \
        if (njobs > 0)                                                                                         \
            hipLaunchKernelGGL((k_tail2d_batch<T, KS>), dim3(njobs), dim3(tail_threads(tp)), lds_bytes, s, jobs); \
    } while (0)
    const int ks = tail_ks(tp);
    if constexpr (sizeof(T) == 4) {
        if (ks == 4) TAIL_GO(4);
        else if (ks == 2) TAIL_GO(2);
        else TAIL_GO(1);
    } else {
        TAIL_GO(1);
    }
#undef TAIL_GO
}
template void launch_tail2d_batch<float>(const TailParams<float> &, const TailJob<float> *, int, size_t, hipStream_t);

template <typename T>
void launch_tail2d_fmg_batch(const TailParams<T> &tp, const TailJob<T> *jobs, int njobs, int k, size_t lds_bytes,
                             hipStream_t s)
{
#define TAIL_GO(KS)                                                                                                \
    do {                                                                                                           \
        TAIL_RAISED((k_tail2d_fmg_batch<T, KS>));                                                                  \
        if (njobs > 0)                                                                                             \
            hipLaunchKernelGGL((k_tail2d_fmg_batch<T, KS>), dim3(njobs), dim3(tail_threads(tp)), lds_bytes, s, jobs, \
                               k);                                                                                 \
    } while (0)
    const int ks = tail_ks(tp);
    if constexpr (sizeof(T) == 4) {
        if (ks == 4) TAIL_GO(4);
        else if (ks == 2) TAIL_GO(2);
        else TAIL_GO(1);
    } else {
        TAIL_GO(1);
    }
#undef TAIL_GO
}
template void launch_tail2d_fmg_batch<float>(const TailParams<float> &, const TailJob<float> *, int, int, size_t,
                                             hipStream_t);

}  // namespace ffmg
