// ffmg_learned.hip -- the learned smoother: a three-layer 3x3 complex
// convolutional network that replaces the weighted-Jacobi sweeps of the
// finest level (the paper smooths with weighted Jacobi, Sec. 4, and notes
// that other smoothers can take its place).  One smoothing step is
//
//   u <- u + s h^2 N(r / s, kappa h^2) = u + h^2 N(r, kappa h^2),
//   r = b - A u,  s = RMS(r) (the training data are scaled by s),
//   N:  a = W1[., ., 0] * r~,  m = W1[., ., 1] * kappa~,  x1 = a (1 + m),
//       x2 = W2 * x1,  N = W3 * x2,
//
// with 1 + 1 -> 16 -> 16 -> 1 complex channels and 3x3 taps (tap t =
// 3 (dy + 1) + (dx + 1) reads the point (y + dy, x + dx); zero outside the
// grid).  N is complex-linear in r~ (a learned radius-3 stencil whose weights
// the coefficient gate 1 + m adapts), so the smoothing step is a linear
// iteration.  Weights and activations are stored in BF16, products are
// accumulated in FP32.
//
// Training (on patches of (residual, error) pairs from plain V-cycle
// iterates): loss = mean over the patch interior of |L5 (e~ - N)|^2 +
// LOSS_ALPHA max(0, ||e~ - N||^2 / ||e~||^2 - 1) with e~ = e / (s h^2) and
// L5 the 5-point Laplacian stencil (4, -1, -1, -1, -1): the high-frequency
// part of the error left by the smoothing step, plus a penalty on growth of
// the patch's error (smooth error, which L5 does not see, must not be
// amplified).  One
// workgroup per 32 x 32 patch runs the forward pass, the loss and the whole
// backward pass in LDS and writes that patch's weight gradient; a second
// kernel averages them over the minibatch in a fixed order; Adam updates the
// FP32 master weights and refreshes the BF16 copies.
//
// Complex gradients use g = dL/dRe + i dL/dIm; for y = W x this gives
// dL/dW = g_y conj(x) and g_x = conj(W) g_y.
#include <math.h>

#include "ffmg_internal.hpp"
#include "ffmg_learned.hpp"

#include <algorithm>

namespace ffmg {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// Hardware round-to-nearest-even pair FP32 -> BF16 (v_cvt_pk_bf16_f32).
typedef float fv2 __attribute__((ext_vector_type(2)));
typedef __bf16 bv2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector(fv2{lo, hi}, bv2));
}

// ---------------------------------------------------------------------------
// BF16 helpers: round-to-nearest-even of a finite FP32, and complex values
// packed as (bf16 re) | (bf16 im) << 16.
__host__ __device__ __forceinline__ unsigned bf16_bits(float f)
{
    unsigned u = __builtin_bit_cast(unsigned, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__host__ __device__ __forceinline__ float bf16_round(float f)
{
    return __builtin_bit_cast(float, bf16_bits(f) << 16);
}
__device__ __forceinline__ unsigned pack_c(float re, float im) { return bf16_bits(re) | (bf16_bits(im) << 16); }
__device__ __forceinline__ float2 unpack_c(unsigned v)
{
    return make_float2(__builtin_bit_cast(float, v << 16), __builtin_bit_cast(float, v & 0xFFFF0000u));
}

// acc += conj(w) x
__device__ __forceinline__ void cmac_cw(float2 &acc, float2 w, float2 x)
{
    acc.x = fmaf(w.x, x.x, acc.x);
    acc.x = fmaf(w.y, x.y, acc.x);
    acc.y = fmaf(w.x, x.y, acc.y);
    acc.y = fmaf(-w.y, x.x, acc.y);
}
__device__ __forceinline__ constexpr int tap_dy(int t) { return t / 3 - 1; }
__device__ __forceinline__ constexpr int tap_dx(int t) { return t % 3 - 1; }

// ---------------------------------------------------------------------------
// Training: one 1024-thread workgroup per 32 x 32 patch, a point per thread in
// the point-wise steps.  Every product of two BF16 arrays (layers 1 to 3, the
// gradients of x1 and of all weights) is a GEMM on v_mfma_f32_16x16x32_bf16
// (operand layout as in the inference kernel below) with FP32 accumulators, so
// the products are exact and the precision is that of FP32 sums; the gradient
// g_N of the output is FP32 and enters the weight gradient of layer 3 as three
// BF16 parts (24 bits).
//   convolutions: rows = 16 points, K = the 16 complex channels of a tap as 32
//     real slots (a packed activation is two of them), columns = 16 output
//     channels, one product for the real and one for the imaginary parts;
//   weight gradients sum_p g(p) conj(x(p + d)): K = 16 points x (re, im), the
//     packed dwords of both operands as they are for the real part, g's as
//     (im, -re) for the imaginary part.
// A row of a point's 16 packed channels is 64 bytes in LDS; its four 16-byte
// chunks are permuted by the point (chunk c of point p at c ^ (p / 4 % 4)), so
// that the 16-point operand reads spread over all banks.  Points outside the
// patch read row TPP, which is zero.
// Bound by LDS latency and the vector unit between the GEMMs (which take about
// 8 us at the matrix rate).  Measured, 256 patches: 77 us; with one FP32 vector
// product per weight and point in 256-thread workgroups it took 879 us.
constexpr float LOSS_ALPHA = 1.f;   // weight of the error-growth penalty
constexpr int TP = 32;              // patch side
constexpr int TPP = TP * TP;        // points per patch
constexpr int TRAIN_SETS = 8;       // partial sums kept in LDS for a weight gradient

struct alignas(16) TrainLds {
    unsigned x1[(TPP + 1) * 16];    // layer-1 output, later its gradient, later that of a
    unsigned x2[(TPP + 1) * 16];    // layer-2 output, later its gradient, later that of m
    unsigned r0[TPP + 4], k0[TPP + 4];  // inputs r~, kappa~, BF16 complex
    float2 d[TPP];                  // e~ - N, later g_N
    union {
        unsigned w2[9 * 256];       // packed W2
        float2 z[TPP];              // mask L5 (e~ - N)
        unsigned gp[3][TPP];        // g_N as three BF16 parts
    };
};
static_assert(offsetof(TrainLds, z) == offsetof(TrainLds, d) + sizeof(float2) * TPP && sizeof(TrainLds) <= 160 * 1024,
              "d and what follows it serve as one buffer of partial sums");
static_assert(TRAIN_SETS * 288 * sizeof(float2) <= sizeof(float2) * TPP + 3 * sizeof(unsigned) * TPP, "partial sums");
static_assert(TRAIN_SETS * 144 * sizeof(float2) <= 3 * sizeof(unsigned) * TPP, "partial sums");

__device__ __forceinline__ bool in_patch(int y, int x) { return (unsigned)y < (unsigned)TP && (unsigned)x < (unsigned)TP; }
__device__ __forceinline__ int point_or_zero(int y, int x) { return in_patch(y, x) ? y * TP + x : TPP; }
// dword of channel c of point p, and the 16-byte chunk c of it
__device__ __forceinline__ int act_at(int p, int c) { return p * 16 + (((c >> 2) ^ ((p >> 2) & 3)) << 2) + (c & 3); }
__device__ __forceinline__ bf8 act_chunk(const unsigned *x, int p, int c)
{
    return __builtin_bit_cast(bf8, *reinterpret_cast<const uint4 *>(x + p * 16 + ((c ^ ((p >> 2) & 3)) << 2)));
}
__device__ __forceinline__ unsigned swap_halves(unsigned v) { return __builtin_amdgcn_alignbit(v, v, 16); }
__device__ __forceinline__ bf8 as_bf8(unsigned a, unsigned b, unsigned c, unsigned d)
{
    return __builtin_bit_cast(bf8, make_uint4(a, b, c, d));
}
// BF16-rounded weights: the upper halves of their FP32 bits are exact
__device__ __forceinline__ unsigned pack_weight(float2 w)
{
    return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, w.y), __builtin_bit_cast(unsigned, w.x), 0x07060302u);
}
constexpr unsigned NEG_HI = 0x80000000u, NEG_LO = 0x8000u;

// The four row tiles (16 points each: half a patch row) of a wave.
struct TrainTile {
    int py, px;     // of the lane's point as an operand row
    int p0;         // of the tile's first point
    __device__ __forceinline__ TrainTile(int wave, int q)
    {
        const int rt = wave * 4 + q;
        py = rt >> 1;
        px = 16 * (rt & 1) + (threadIdx.x & 15);
        p0 = py * TP + 16 * (rt & 1);
    }
};

// acc[q] = the 3x3 convolution of x with W2 (16 -> 16 channels) at the wave's
// tiles, real and imaginary parts; TR: with the conjugate transposed weights.
template <bool TR>
__device__ __forceinline__ void conv16(const unsigned *x, const unsigned *w2, int wave, f4 (&acc)[4][2])
{
    const int j = threadIdx.x & 15, kq = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q][0] = acc[q][1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 3
    for (int t = 0; t < 9; ++t) {
        const int dy = TR ? -tap_dy(t) : tap_dy(t), dx = TR ? -tap_dx(t) : tap_dx(t);
        unsigned w[4];
        if (TR) {
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = w2[(t * 16 + 4 * kq + e) * 16 + j];
        } else {
            const uint4 v = *reinterpret_cast<const uint4 *>(w2 + (t * 16 + j) * 16 + 4 * kq);
            w[0] = v.x;
            w[1] = v.y;
            w[2] = v.z;
            w[3] = v.w;
        }
        unsigned re[4], im[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            re[e] = TR ? w[e] : w[e] ^ NEG_HI;                              // (wr, wi) or (wr, -wi)
            im[e] = TR ? swap_halves(w[e]) ^ NEG_LO : swap_halves(w[e]);    // (-wi, wr) or (wi, wr)
        }
        const bf8 bre = as_bf8(re[0], re[1], re[2], re[3]), bim = as_bf8(im[0], im[1], im[2], im[3]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const TrainTile T(wave, q);
            const bf8 a = act_chunk(x, point_or_zero(T.py + dy, T.px + dx), kq);
            acc[q][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bre, acc[q][0], 0, 0, 0);
            acc[q][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bim, acc[q][1], 0, 0, 0);
        }
    }
}

// Layer 1 at the wave's tile: a (from r~) and m (from kappa~), real and
// imaginary parts; K = 9 taps x (re, im), lanes 16 kq.. the taps 4 kq .. + 3.
struct Layer1 {
    bf8 are, aim, mre, mim;
    __device__ __forceinline__ explicit Layer1(const float2 *__restrict__ W1)
    {
        const int j = threadIdx.x & 15, kq = (threadIdx.x & 63) >> 4;
        unsigned a[4], m[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * kq + e, s = min(t, 8);
            const float4 w = *reinterpret_cast<const float4 *>(W1 + (s * 16 + j) * 2);
            a[e] = t < 9 ? pack_weight(make_float2(w.x, w.y)) : 0u;
            m[e] = t < 9 ? pack_weight(make_float2(w.z, w.w)) : 0u;
        }
        are = as_bf8(a[0] ^ NEG_HI, a[1] ^ NEG_HI, a[2] ^ NEG_HI, a[3] ^ NEG_HI);
        aim = as_bf8(swap_halves(a[0]), swap_halves(a[1]), swap_halves(a[2]), swap_halves(a[3]));
        mre = as_bf8(m[0] ^ NEG_HI, m[1] ^ NEG_HI, m[2] ^ NEG_HI, m[3] ^ NEG_HI);
        mim = as_bf8(swap_halves(m[0]), swap_halves(m[1]), swap_halves(m[2]), swap_halves(m[3]));
    }
    __device__ __forceinline__ void at(const TrainLds &S, const TrainTile &T, f4 (&a)[2], f4 (&m)[2]) const
    {
        const int kq = (threadIdx.x & 63) >> 4;
        unsigned r[4], k[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * kq + e, ty = t / 3;
            const int p = t < 9 ? point_or_zero(T.py + ty - 1, T.px + t - 3 * ty - 1) : TPP;
            r[e] = S.r0[p];
            k[e] = S.k0[p];
        }
        const bf8 ar = as_bf8(r[0], r[1], r[2], r[3]), ak = as_bf8(k[0], k[1], k[2], k[3]);
        const f4 z = {0.f, 0.f, 0.f, 0.f};
        a[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar, are, z, 0, 0, 0);
        a[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar, aim, z, 0, 0, 0);
        m[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, mre, z, 0, 0, 0);
        m[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, mim, z, 0, 0, 0);
    }
};

// The 5-point Laplacian stencil of v at (y, x), zero outside the patch.
__device__ __forceinline__ float2 lap5(const float2 *v, int y, int x)
{
    const float2 c = v[y * TP + x];
    float2 s = make_float2(4.f * c.x, 4.f * c.y);
    const int nb[4][2] = {{0, -1}, {0, 1}, {-1, 0}, {1, 0}};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int yy = y + nb[m][0], xx = x + nb[m][1];
        if (in_patch(yy, xx)) {
            const float2 w = v[yy * TP + xx];
            s.x -= w.x;
            s.y -= w.y;
        }
    }
    return s;
}

__device__ __forceinline__ void stage_w2(TrainLds &S, const float2 *__restrict__ W2)
{
    for (int k = threadIdx.x; k < 9 * 256; k += 1024) S.w2[k] = pack_weight(W2[k]);
}

__global__ __launch_bounds__(1024) void k_train_patch(const float2 *__restrict__ rt, const float2 *__restrict__ kt,
                                                      const float2 *__restrict__ et, const float2 *__restrict__ W,
                                                      float2 *__restrict__ dW_part, float *__restrict__ loss_part,
                                                      int border)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    TrainLds &S = *reinterpret_cast<TrainLds *>(lds_raw);
    const float2 *W1 = W + NET_W1, *W2 = W + NET_W2, *W3 = W + NET_W3;
    const size_t base = (size_t)blockIdx.x * TPP;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kq = lane >> 4;
    const int py = tid / TP, px = tid % TP;
    // inputs, rounded to BF16; the zero rows
    {
        const float2 r = rt[base + tid], k = kt[base + tid];
        S.r0[tid] = pack_bf16(r.x, r.y);
        S.k0[tid] = pack_bf16(k.x, k.y);
        if (tid < 16) S.x1[TPP * 16 + tid] = S.x2[TPP * 16 + tid] = 0u;
        if (tid == 0) S.r0[TPP] = S.k0[TPP] = 0u;
        stage_w2(S, W2);
    }
    const float2 e = et[base + tid];
    __syncthreads();
    // layer 1: a gated by 1 + m
    {
        const Layer1 l1(W1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const TrainTile T(wave, q);
            f4 a[2], m[2];
            l1.at(S, T, a, m);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float cr = 1.f + m[0][r], ci = m[1][r];
                S.x1[act_at(T.p0 + 4 * kq + r, j)] =
                    pack_bf16(a[0][r] * cr - a[1][r] * ci, a[0][r] * ci + a[1][r] * cr);
            }
        }
    }
    __syncthreads();
    // layer 2: 16 -> 16
    {
        f4 acc[4][2];
        conv16<false>(S.x1, S.w2, wave, acc);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const TrainTile T(wave, q);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                S.x2[act_at(T.p0 + 4 * kq + r, j)] = pack_bf16(acc[q][0][r], acc[q][1][r]);
        }
    }
    __syncthreads();
    // layer 3: 16 -> 1 (columns 0 and 1: real and imaginary part); d = e~ - N
    {
        f4 acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 3
        for (int t = 0; t < 9; ++t) {
            unsigned w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const unsigned v = pack_weight(W3[t * 16 + 4 * kq + c]);
                w[c] = j == 0 ? v ^ NEG_HI : j == 1 ? swap_halves(v) : 0u;
            }
            const bf8 b = as_bf8(w[0], w[1], w[2], w[3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const TrainTile T(wave, q);
                const bf8 a = act_chunk(S.x2, point_or_zero(T.py + tap_dy(t), T.px + tap_dx(t)), kq);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[q], 0, 0, 0);
            }
        }
        if (j < 2) {
            float *d = reinterpret_cast<float *>(S.d);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const TrainTile T(wave, q);
#pragma unroll
                for (int r = 0; r < 4; ++r) d[2 * (T.p0 + 4 * kq + r) + j] = acc[q][r];
            }
        }
    }
    __syncthreads();
    S.d[tid] = make_float2(e.x - S.d[tid].x, e.y - S.d[tid].y);
    __syncthreads();
    // z = mask L5 d; loss; patch sums of |e~|^2 and |d|^2 for the growth penalty
    const int lo = border, hi = TP - border;
    const float cnt = (float)((hi - lo) * (hi - lo));
    const bool inner = py >= lo && py < hi && px >= lo && px < hi;
    const float2 dv = S.d[tid];
    float v[3] = {0.f, 0.f, 0.f};
    {
        float2 z = make_float2(0.f, 0.f);
        if (inner) {
            z = lap5(S.d, py, px);
            v[0] = z.x * z.x + z.y * z.y;
            v[1] = e.x * e.x + e.y * e.y;
            v[2] = dv.x * dv.x + dv.y * dv.y;
        }
        S.z[tid] = z;
    }
    __shared__ float red[3][16];
    __shared__ float tot[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_down(v[q], off, 64);
        if (lane == 0) red[q][wave] = v[q];
    }
    __syncthreads();
    if (tid < 3) {
        float s = 0.f;
        for (int w = 0; w < 16; ++w) s += red[tid][w];
        tot[tid] = s;
    }
    // g_N = -(2 / cnt) L5 z - (growth) 2 LOSS_ALPHA mask d / E  (into d)
    const float2 lz = lap5(S.z, py, px);
    __syncthreads();
    const float E = tot[1], D = tot[2];
    const bool grow = E > 0.f && D > E;
    if (tid == 0) loss_part[blockIdx.x] = tot[0] / cnt + (grow ? LOSS_ALPHA * (D / E - 1.f) : 0.f);
    {
        const float sc = -2.f / cnt;
        float2 gn = make_float2(sc * lz.x, sc * lz.y);
        if (grow && inner) {
            const float f = -2.f * LOSS_ALPHA / E;
            gn.x += f * dv.x;
            gn.y += f * dv.y;
        }
        S.d[tid] = gn;
        // three parts of 8 bits (z is dead: every thread has read it)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const unsigned u = pack_bf16(gn.x, gn.y);
            const float2 part = unpack_c(u);
            S.gp[k][tid] = u;
            gn.x -= part.x;
            gn.y -= part.y;
        }
    }
    __syncthreads();
    float2 *dW = dW_part + (size_t)blockIdx.x * NET_NW;
    // dW3[t][i] = sum_p g_N(p) conj(x2_i(p + d_t)): rows 0..2 the parts of g_N
    // for the real part, 3..5 for the imaginary part; each wave two patch rows
    {
        f4 acc[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
        const unsigned *g = S.gp[j < 3 ? j : j < 6 ? j - 3 : 0];
#pragma unroll 1
        for (int s = 0; s < 4; ++s) {
            const int y = 2 * wave + (s >> 1), x0 = 16 * (s & 1) + kq;
            unsigned a[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const unsigned u = g[y * TP + x0 + 4 * c];
                a[c] = j < 3 ? u : j < 6 ? swap_halves(u) ^ NEG_HI : 0u;
            }
            const bf8 av = as_bf8(a[0], a[1], a[2], a[3]);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                unsigned b[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    b[c] = S.x2[act_at(point_or_zero(y + tap_dy(t), x0 + 4 * c + tap_dx(t)), j)];
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, as_bf8(b[0], b[1], b[2], b[3]), acc[t], 0, 0, 0);
            }
        }
        // lanes 0..15 hold rows 0..3, lanes 16..31 rows 4 and 5
        float2 part[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            part[t].x = (acc[t][2] + acc[t][1]) + acc[t][0];
            part[t].y = __shfl_down(acc[t][1] + acc[t][0], 16, 64) + acc[t][3];
        }
        __syncthreads();    // gp is dead
        float2 *sum = S.z;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (wave / TRAIN_SETS == half && lane < 16) {
                float2 *at = sum + (wave % TRAIN_SETS) * 144 + lane;
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    float2 s = part[t];
                    if (half) {
                        s.x += at[16 * t].x;
                        s.y += at[16 * t].y;
                    }
                    at[16 * t] = s;
                }
            }
            __syncthreads();
        }
        if (tid < 144) {
            float2 s = make_float2(0.f, 0.f);
            for (int k = 0; k < TRAIN_SETS; ++k) {
                s.x += sum[k * 144 + tid].x;
                s.y += sum[k * 144 + tid].y;
            }
            dW[NET_W3 + tid] = s;
        }
    }
    // g_x2 = (conj(W3) * g_N, transposed), in place of x2
    {
        float2 g[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) g[i] = make_float2(0.f, 0.f);
#pragma unroll 1
        for (int t = 0; t < 9; ++t) {
            const int dy = t / 3 - 1, y = py - dy, x = px - (t - 3 * (dy + 1) - 1);
            const bool in = in_patch(y, x);
            float2 gn = S.d[in ? y * TP + x : 0];
            gn = make_float2(in ? gn.x : 0.f, in ? gn.y : 0.f);
#pragma unroll
            for (int i = 0; i < 16; ++i) cmac_cw(g[i], W3[t * 16 + i], gn);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) S.x2[act_at(tid, i)] = pack_bf16(g[i].x, g[i].y);
    }
    __syncthreads();
    // dW2[t][o][i] = sum_p g_x2_o(p) conj(x1_i(p + d_t)): a tap per wave
    if (wave < 9) {
        const int dy = wave / 3 - 1, dx = wave - 3 * (dy + 1) - 1;
        f4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int y = max(0, -dy); y < TP - max(0, dy); ++y) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                unsigned a[4], b[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int x = 16 * h + 4 * c + kq;
                    a[c] = S.x2[act_at(y * TP + x, j)];
                    b[c] = S.x1[act_at(point_or_zero(y + dy, x + dx), j)];
                }
                const bf8 bv = as_bf8(b[0], b[1], b[2], b[3]);
                re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(a[0], a[1], a[2], a[3]), bv, re, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = swap_halves(a[c]) ^ NEG_HI;
                im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(a[0], a[1], a[2], a[3]), bv, im, 0, 0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) dW[NET_W2 + (wave * 16 + 4 * kq + r) * 16 + j] = make_float2(re[r], im[r]);
    } else {
        for (int k = tid - 9 * 64; k < 9 * 256; k += 7 * 64) S.w2[k] = pack_weight(W2[k]);   // (the sums are dead)
    }
    __syncthreads();
    // g_x1 = (conj(W2) * g_x2, transposed), in place of x1
    {
        f4 acc[4][2];
        conv16<true>(S.x2, S.w2, wave, acc);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const TrainTile T(wave, q);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                S.x1[act_at(T.p0 + 4 * kq + r, j)] = pack_bf16(acc[q][0][r], acc[q][1][r]);
        }
    }
    __syncthreads();
    // through the gate x1 = a c, c = 1 + m (a, m recomputed from the
    // inputs): g_a = conj(c) g_x1 into x1, g_m = conj(a) g_x1 into x2
    {
        const Layer1 l1(W1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const TrainTile T(wave, q);
            f4 a[2], m[2];
            l1.at(S, T, a, m);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int at = act_at(T.p0 + 4 * kq + r, j);
                const float2 g = unpack_c(S.x1[at]);
                float2 ga = make_float2(0.f, 0.f), gm = make_float2(0.f, 0.f);
                cmac_cw(ga, make_float2(1.f + m[0][r], m[1][r]), g);
                cmac_cw(gm, make_float2(a[0][r], a[1][r]), g);
                S.x1[at] = pack_bf16(ga.x, ga.y);
                S.x2[at] = pack_bf16(gm.x, gm.y);
            }
        }
    }
    __syncthreads();
    // dW1[t][o][0] = sum_p g_a_o(p) conj(r~(p + d_t)), dW1[t][o][1] likewise from
    // g_m and kappa~ (columns = taps); each wave two patch rows
    {
        f4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][0] = acc[i][1] = f4{0.f, 0.f, 0.f, 0.f};
        const int ty = j / 3;
#pragma unroll 1
        for (int s = 0; s < 4; ++s) {
            const int y = 2 * wave + (s >> 1), x0 = 16 * (s & 1) + kq;
            int p[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                p[c] = j < 9 ? point_or_zero(y + ty - 1, x0 + 4 * c + j - 3 * ty - 1) : TPP;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned *in = i ? S.k0 : S.r0, *gr = i ? S.x2 : S.x1;
                unsigned a[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = gr[act_at(y * TP + x0 + 4 * c, j)];
                const bf8 bv = as_bf8(in[p[0]], in[p[1]], in[p[2]], in[p[3]]);
                acc[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(a[0], a[1], a[2], a[3]), bv, acc[i][0], 0, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = swap_halves(a[c]) ^ NEG_HI;
                acc[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(a[0], a[1], a[2], a[3]), bv, acc[i][1], 0, 0, 0);
            }
        }
        float2 *sum = S.d;      // d and what follows it are dead
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (wave / TRAIN_SETS == half && j < 9)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float2 *at = sum + (wave % TRAIN_SETS) * 288 + (j * 16 + 4 * kq + r) * 2 + i;
                        float2 s = make_float2(acc[i][0][r], acc[i][1][r]);
                        if (half) {
                            s.x += at->x;
                            s.y += at->y;
                        }
                        *at = s;
                    }
            __syncthreads();
        }
        if (tid < 288) {
            float2 s = make_float2(0.f, 0.f);
            for (int k = 0; k < TRAIN_SETS; ++k) {
                s.x += sum[k * 288 + tid].x;
                s.y += sum[k * 288 + tid].y;
            }
            dW[NET_W1 + tid] = s;
        }
    }
}

// Adam on the real and imaginary parts of weight k (step >= 1); refreshes the
// BF16-rounded copy used by the training forward pass.
struct AdamArgs {
    float2 *Wm, *Wq, *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamArgs &A, int k, float2 g)
{
    float2 mk = A.m[k], vk = A.v[k], w = A.Wm[k];
    mk.x = A.b1 * mk.x + (1.f - A.b1) * g.x;
    mk.y = A.b1 * mk.y + (1.f - A.b1) * g.y;
    vk.x = A.b2 * vk.x + (1.f - A.b2) * g.x * g.x;
    vk.y = A.b2 * vk.y + (1.f - A.b2) * g.y * g.y;
    w.x -= A.lr * (mk.x / A.c1) / (sqrtf(vk.x / A.c2) + A.eps);
    w.y -= A.lr * (mk.y / A.c1) / (sqrtf(vk.y / A.c2) + A.eps);
    A.m[k] = mk;
    A.v[k] = vk;
    A.Wm[k] = w;
    A.Wq[k] = make_float2(bf16_round(w.x), bf16_round(w.y));
}

// Mean of the per-patch gradients, 64 weights a block (every 16th patch a wave,
// then the waves in order), where ADAM with the update of those weights; the last
// block takes the mean of the losses, written to the host's page-locked word.
// (One thread a weight over all patches is a chain of dependent loads: 61 us for
// 256 patches.)  5 us for 256 patches; as launches of their own the loss, the
// update and the copy of the loss took 4.7, 5.2 and 4.1 us more.
constexpr int NB_GRADS = (NET_NW + 63) / 64;

template <bool ADAM>
__global__ __launch_bounds__(1024) void k_reduce_grads(const float2 *__restrict__ dW_part, int count,
                                                       float2 *__restrict__ grad,
                                                       const float *__restrict__ loss_part, float *__restrict__ loss,
                                                       AdamArgs A)
{
    __shared__ float2 part[16][64];
    if (blockIdx.x == NB_GRADS) {
        float *red = &part[0][0].x;
        if (threadIdx.x < 256) {
            float s = 0.f;
            for (int p = threadIdx.x; p < count; p += 256) s += loss_part[p];
            red[threadIdx.x] = s;
        }
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = red[0] / (float)count;
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane, kk = min(k, NET_NW - 1);
    float2 s = make_float2(0.f, 0.f);
#pragma unroll 4
    for (int p = wave; p < count; p += 16) {
        const float2 v = dW_part[(size_t)p * NET_NW + kk];
        s.x += v.x;
        s.y += v.y;
    }
    part[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && k < NET_NW) {
        for (int w = 1; w < 16; ++w) {
            s.x += part[w][lane].x;
            s.y += part[w][lane].y;
        }
        const float inv = 1.f / (float)count;
        const float2 g = make_float2(s.x * inv, s.y * inv);
        grad[k] = g;
        if (ADAM) adam_update(A, k, g);
    }
}

__global__ __launch_bounds__(256) void k_round_weights(const float2 *__restrict__ Wm, float2 *__restrict__ Wq)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < NET_NW) Wq[k] = make_float2(bf16_round(Wm[k].x), bf16_round(Wm[k].y));
}

size_t train_lds_bytes() { return sizeof(TrainLds); }

void launch_train_patches(const float2 *rt, const float2 *kt, const float2 *et, const float2 *Wq, float2 *dW_part,
                          float *loss_part, int count, int border, hipStream_t s)
{
    // once (a thread-safe static initialisation)
    static const bool attr = [] {
        (void)hipFuncSetAttribute((const void *)k_train_patch, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)sizeof(TrainLds));
        return true;
    }();
    (void)attr;
    hipLaunchKernelGGL(k_train_patch, dim3(count), dim3(1024), sizeof(TrainLds), s, rt, kt, et, Wq, dW_part,
                       loss_part, border);
}

void launch_reduce_grads(const float2 *dW_part, int count, float2 *grad, const float *loss_part, float *loss,
                         hipStream_t s)
{
    hipLaunchKernelGGL(k_reduce_grads<false>, dim3(NB_GRADS + 1), dim3(1024), 0, s, dW_part, count, grad, loss_part,
                       loss, AdamArgs());
}

void launch_reduce_grads_adam(const float2 *dW_part, int count, float2 *grad, const float *loss_part, float *loss,
                              float2 *Wm, float2 *Wq, float2 *m, float2 *v, float lr, float b1, float b2, float eps,
                              int step, hipStream_t s)
{
    const AdamArgs A = {Wm, Wq, m, v, lr, b1, b2, eps, 1.f - powf(b1, (float)step), 1.f - powf(b2, (float)step)};
    hipLaunchKernelGGL(k_reduce_grads<true>, dim3(NB_GRADS + 1), dim3(1024), 0, s, dW_part, count, grad, loss_part,
                       loss, A);
}

void launch_round_weights(const float2 *Wm, float2 *Wq, hipStream_t s)
{
    hipLaunchKernelGGL(k_round_weights, dim3((NET_NW + 255) / 256), dim3(256), 0, s, Wm, Wq);
}



// ---------------------------------------------------------------------------
// Inference on a grid with the BF16 MFMA v_mfma_f32_16x16x32_bf16 (A[i][k]
// from lane i + 16 (k / 8), element k % 8; B[k][j] likewise with j; D[i][j]
// in lane j + 16 (i / 4), register i % 4).  Each convolution is an implicit
// GEMM over points: rows are the real output channels (Re / Im of each complex
// channel), columns 16 points of a region, K the (tap, real input channel)
// pairs.  A complex weight w acts on (Re x, Im x) as the real 2 x 2 block
// [[Re w, -Im w], [Im w, Re w]].
//   layer 1: K = 9 taps x 2 (Re / Im), padded to 32, one k-step, a product
//            for a and one for m (accumulator started at 1 for Re m); a lane
//            holds Re and Im of both for its channels, so the gate
//            x1 = a (1 + m) needs no exchange between lanes
//   layer 2: K = 32 channels per tap, one k-step per tap
//   layer 3: one output channel, so the 9 taps go to the rows instead:
//            Z_t = W3[t] x2 per point (K = 32, rows 2 t + part, 18 of 32
//            used), then N(p) = sum_t Z_t(p + d_t) by a gather from LDS
// With the points in the columns a lane's two accumulators are 8 channels of
// one point: layer 1 writes them with one 128-bit store and layer 2's are
// layer 3's operand as they are, so x2 never leaves the registers.
// A 16 x 16 output tile needs layer-2 values on 18 x 18 points, layer-1
// values on 20 x 20 and the inputs on 22 x 22 (zero outside the grid); the
// activations live in LDS as BF16 [point][channel].  The weight fragments
// (prepared on the host by pack_net_mfma) stay in registers.
typedef unsigned short us8 __attribute__((ext_vector_type(8)));

constexpr int IT = 16;                       // output tile side
constexpr int R1 = IT + 4, R2 = IT + 2;      // layer-1 / layer-2 region sides
constexpr int R0 = IT + 6;                   // input region side
constexpr int NR1 = (R1 * R1 + 15) / 16;     // row tiles of the layer-1 region
constexpr int IN_PER_THREAD = (R0 * R0 + 255) / 256;

// Activations: 32 BF16 channel slots per point, padded to 40 (80 bytes): the
// 8 lanes a 128-bit LDS read serves together then start 20 dwords apart and
// cover all 32 banks once.  Slot s holds row 16 (s & 1) + (s >> 1) of the
// producing layer: the lanes of group lg, which hold rows 4 lg .. 4 lg + 3 of
// both row tiles, write slots 8 lg .. 8 lg + 7.  Row j is Re (j even) or Im
// (j odd) of channel j / 2.
constexpr int XS = 40;
// Per-tap layer-3 products: 18 floats per point, rows of 20 (80 bytes).
constexpr int ZS = 20;
struct alignas(16) InferLds {
    unsigned r0[R0 * R0], k0[R0 * R0];       // r~, kappa~ (packed re, im)
    unsigned short x1[NR1 * 16][XS];
    float z[R2 * R2][ZS];
};

__device__ __forceinline__ bf8 as_bf8(us8 v) { return __builtin_bit_cast(bf8, v); }

// Point (y, x) of row-major region of width R for index p.
struct RegionPos {
    int y, x;
};
template <int R>
__device__ __forceinline__ RegionPos region_pos(int p)
{
    return RegionPos{p / R, p - (p / R) * R};
}
// Inputs of one tile's 22 x 22 region (origin oy - 3, ox - 3), held in
// registers between their global load and their LDS store so that the next
// tile's loads overlap the current tile's layers.
struct TileInput {
    cd r[IN_PER_THREAD];
    unsigned k[IN_PER_THREAD];
};

// Position of input i of this thread in the region; past its end the origin.
__device__ __forceinline__ RegionPos input_pos(int i)
{
    const int p = threadIdx.x + 256 * i;
    return region_pos<R0>(p < R0 * R0 ? p : 0);
}

// Whether the region of the tile at (oy, ox) lies inside the grid.
__device__ __forceinline__ bool input_interior(int mx, int my, int oy, int ox)
{
    return oy >= 3 && ox >= 3 && oy + IT + 3 <= my && ox + IT + 3 <= mx;
}

__device__ __forceinline__ bool input_in_grid(RegionPos q, int mx, int my, int oy, int ox)
{
    const int gy = oy - 3 + q.y, gx = ox - 3 + q.x;
    return gy >= 0 && gy < my && gx >= 0 && gx < mx;
}

// Issues the loads only (points outside the grid read element 0 and are
// zeroed when stored), so that nothing waits for them before the store.
__device__ __forceinline__ void load_tile_input(TileInput &in, const cd *__restrict__ r,
                                                const unsigned *__restrict__ kh2, int mx, int my, int oy, int ox)
{
    const bool inside = input_interior(mx, my, oy, ox);
    const long long origin = (long long)(oy - 3) * mx + (ox - 3);
#pragma unroll
    for (int i = 0; i < IN_PER_THREAD; ++i) {
        const RegionPos q = input_pos(i);
        const long long at = origin + (q.y * mx + q.x);
        const size_t j = inside || input_in_grid(q, mx, my, oy, ox) ? (size_t)at : 0;
        in.r[i] = r[j];
        in.k[i] = kh2[j];
    }
}

__device__ __forceinline__ void store_tile_input(InferLds &S, const TileInput &in, int mx, int my, int oy, int ox)
{
    const bool inside = input_interior(mx, my, oy, ox);
#pragma unroll
    for (int i = 0; i < IN_PER_THREAD; ++i) {
        const int p = threadIdx.x + 256 * i;
        unsigned r = pack_bf16((float)in.r[i].re, (float)in.r[i].im), k = in.k[i];
        if (!inside && !input_in_grid(input_pos(i), mx, my, oy, ox)) r = k = 0u;
        if (p < R0 * R0) {
            S.r0[p] = r;
            S.k0[p] = k;
        }
    }
}

// The network's weight fragments, the same for every tile.
struct NetFrags {
    bf8 a1[2], m1[2], w2[9][2], w3[2];
};

// The 8 channels of a point that a lane's two accumulators hold, as the slots
// 8 lg .. 8 lg + 7.
__device__ __forceinline__ uint4 pack_slots(const float (&x0)[4], const float (&x1)[4])
{
    return make_uint4(pack_bf16(x0[0], x1[0]), pack_bf16(x0[1], x1[1]), pack_bf16(x0[2], x1[2]), pack_bf16(x0[3], x1[3]));
}

// Layers 2 and 3 of one wave: the points (y0 .. y0 + NR - 1, x = 0 .. 15) of the
// 18 x 18 region, a row a column tile, and where SIDE the points 16 k .. 16 k +
// 15 of the 36 of its last two columns.  A row's layer-1 values are read once for
// the up to three rows whose taps they are (3 (NR + 2) reads for 9 NR k-steps), a
// row of reads ahead of their products; the taps of a point are added in the
// order 0 .. 8.  Each stage is issued for all column tiles before the next, so
// that no product waits for the one before it.
template <bool EDGE, int NR, bool SIDE>
__device__ __forceinline__ void layers23(InferLds &S, const NetFrags &W, int mx, int my, int oy, int ox, int y0, int k)
{
    constexpr int NT = NR + (SIDE ? 1 : 0);   // column tiles
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const f4 z = f4{0.f, 0.f, 0.f, 0.f};
    f4 acc[NT][2];
#pragma unroll
    for (int r = 0; r < NT; ++r) acc[r][0] = acc[r][1] = z;
    const int e = min(16 * k + li, 2 * R2 - 1), sy = e >> 1, sx = 16 + (e & 1);   // SIDE
    const us8 *base = reinterpret_cast<const us8 *>(&S.x1[y0 * R1 + li][8 * lg]);
    const us8 *side = reinterpret_cast<const us8 *>(&S.x1[sy * R1 + sx][8 * lg]);
    us8 x[2][3], xs[9];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) x[0][dx] = base[dx * (XS / 8)];
#pragma unroll
    for (int yy = 0; yy < NR + 2; ++yy) {
        if (yy + 1 < NR + 2) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) x[(yy + 1) & 1][dx] = base[((yy + 1) * R1 + dx) * (XS / 8)];
        } else if (SIDE) {
#pragma unroll
            for (int t = 0; t < 9; ++t) xs[t] = side[((t / 3) * R1 + t % 3) * (XS / 8)];
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int r = yy - dy;
                if (r < 0 || r >= NR) continue;
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    acc[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w2[3 * dy + dx][nt], as_bf8(x[yy & 1][dx]),
                                                                         acc[r][nt], 0, 0, 0);
            }
    }
    if (SIDE) {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                acc[NT - 1][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w2[t][nt], as_bf8(xs[t]), acc[NT - 1][nt],
                                                                          0, 0, 0);
    }
    // layer 3's operand: the accumulators as they are, zero outside the grid
    uint4 b[NT];
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        const float c0[4] = {acc[r][0][0], acc[r][0][1], acc[r][0][2], acc[r][0][3]};
        const float c1[4] = {acc[r][1][0], acc[r][1][1], acc[r][1][2], acc[r][1][3]};
        b[r] = pack_slots(c0, c1);
        if (EDGE) {
            const int gy = oy - 1 + (r < NR ? y0 + r : sy), gx = ox - 1 + (r < NR ? li : sx);
            if (!(gy >= 0 && gy < my && gx >= 0 && gx < mx)) b[r] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
#pragma unroll
    for (int r = 0; r < NT; ++r)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
            acc[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w3[nt], as_bf8(b[r].x, b[r].y, b[r].z, b[r].w), z,
                                                                 0, 0, 0);
#pragma unroll
    for (int r = 0; r < NT; ++r) {
        float *zp = S.z[r < NR ? (y0 + r) * R2 + li : sy * R2 + sx];
        if (r < NR || 16 * k + li < 2 * R2) *reinterpret_cast<f4 *>(zp + 4 * lg) = acc[r][0];
    }
    if (lg == 0) {
#pragma unroll
        for (int r = 0; r < NT; ++r) {
            float *zp = S.z[r < NR ? (y0 + r) * R2 + li : sy * R2 + sx];
            if (r < NR || 16 * k + li < 2 * R2)
                *reinterpret_cast<float2 *>(zp + 16) = make_float2(acc[r][1][0], acc[r][1][1]);
        }
    }
}

// Layer 1 on the column tiles rt, rt + 4, .. (NR of them) of the 20 x 20
// region (origin -2), each stage issued for all of them before the next.
template <bool EDGE, int NR>
__device__ __forceinline__ void layer1(InferLds &S, const NetFrags &W, int mx, int my, int oy, int ox, int rt)
{
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    // operand: lane group lg holds taps 4 lg .. 4 lg + 3; taps 9 .. 15 are zero
    // padding whose weights are zero, so they may read any (finite) slot: the
    // point itself
    int off1[4];
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) {
        const int t = 4 * lg + hh;
        off1[hh] = t < 9 ? (t / 3 - 1) * R0 + (t % 3 - 1) : 0;
    }
    unsigned r[NR][4], k[NR][4];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const RegionPos P = region_pos<R1>((rt + 4 * i) * 16 + li);
        const int at = (P.y + 1) * R0 + P.x + 1;
#pragma unroll
        for (int hh = 0; hh < 4; ++hh) {
            r[i][hh] = S.r0[at + off1[hh]];
            k[i][hh] = S.k0[at + off1[hh]];
        }
    }
    f4 A[NR][2], M[NR][2];   // rows (Re, Im) of two channels
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const bf8 br = as_bf8(r[i][0], r[i][1], r[i][2], r[i][3]), bk = as_bf8(k[i][0], k[i][1], k[i][2], k[i][3]);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            A[i][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.a1[nt], br, f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            M[i][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.m1[nt], bk, f4{1.f, 0.f, 1.f, 0.f}, 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        float x[2][4];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int c = 0; c < 4; c += 2) {
                x[nt][c] = fmaf(A[i][nt][c], M[i][nt][c], -(A[i][nt][c + 1] * M[i][nt][c + 1]));
                x[nt][c + 1] = fmaf(A[i][nt][c + 1], M[i][nt][c], A[i][nt][c] * M[i][nt][c + 1]);
            }
        uint4 val = pack_slots(x[0], x[1]);
        const int p = (rt + 4 * i) * 16 + li;
        if (EDGE) {
            const RegionPos P = region_pos<R1>(p);
            const int gy = oy - 2 + P.y, gx = ox - 2 + P.x;
            if (!(gy >= 0 && gy < my && gx >= 0 && gx < mx)) val = make_uint4(0u, 0u, 0u, 0u);
        }
        *reinterpret_cast<uint4 *>(&S.x1[p][8 * lg]) = val;
    }
}

// Layers of one 16 x 16 output tile (origin oy, ox) whose inputs are in
// S.r0, S.k0; leaves layer 3's per-tap products in S.z.  EDGE: the tile's layer-1
// region reaches outside the grid, so activations there are set to zero
// (interior tiles skip the test).
template <bool EDGE>
__device__ __forceinline__ void net_layers(InferLds &S, int mx, int my, int oy, int ox, const NetFrags &W, int wave)
{
    static_assert(NR1 == 25, "column tiles of layer 1: 6 a wave and one");
    layer1<EDGE, 3>(S, W, mx, my, oy, ox, wave);
    layer1<EDGE, 3>(S, W, mx, my, oy, ox, wave + 12);
    if (wave == 1) layer1<EDGE, 1>(S, W, mx, my, oy, ox, 24);
    __syncthreads();
    // layers 2 and 3 on the 18 x 18 region (origin -1): rows 5, 5, 4, 4 a wave,
    // and the three column tiles of the last two columns
    if (wave == 0) layers23<EDGE, 5, true>(S, W, mx, my, oy, ox, 0, 2);
    else if (wave == 1) layers23<EDGE, 5, false>(S, W, mx, my, oy, ox, 5, 0);
    else layers23<EDGE, 4, true>(S, W, mx, my, oy, ox, 4 * wave + 2, wave - 2);
}

// Layer 3, second part, for this thread's output point (py, px) of the tile:
// N = sum over the 9 taps of Z_t at the neighbour p + d_t (region origin -1).
__device__ __forceinline__ float2 layer3_gather(const InferLds &S, int py, int px)
{
    float2 y = make_float2(0.f, 0.f);
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int q = (py + 1 + tap_dy(t)) * R2 + (px + 1 + tap_dx(t));
        const float2 zt = *reinterpret_cast<const float2 *>(&S.z[q][2 * t]);
        y.x += zt.x;
        y.y += zt.y;
    }
    return y;
}

// N is complex-linear in its residual input, so s h^2 N(r / s) = h^2 N(r)
// for any scale s; BF16 has the exponent range of FP32, so the residual is
// fed unscaled and no global reduction precedes the step.  Persistent
// workgroups: each loads the weight fragments once and works through a
// contiguous range of tiles (ranges of neighbouring workgroups sit on one
// XCD); the inputs of the next tile are loaded while the current one is
// computed, and u is updated by all threads, one point each.
//
// 520 matrix instructions a tile, 4160 cycles for a SIMD's two waves; the
// stages' LDS latency and three barriers a tile are not all hidden behind them
// (the weights in registers leave room for two waves a SIMD).  1023 x 1023:
// 43 us a step; with the points in the rows (674 instructions a tile: a and m
// twice in layer 1, idle column tiles in layer 2; x2 through LDS, a read for each
// k-step) 69 us.
__global__ __launch_bounds__(256, 2) void k_net_apply(const cd *__restrict__ r, const unsigned *__restrict__ kh2,
                                                   cd *__restrict__ u, int mx, int my, int tiles_x, int ntiles,
                                                   int per_block, const us8 *__restrict__ wfrag, double h2,
                                                   const int *__restrict__ stop)
{
    if (stop && *stop) return;
    __shared__ InferLds S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    NetFrags W;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        W.a1[nt] = as_bf8(wfrag[nt * 64 + lane]);
        W.m1[nt] = as_bf8(wfrag[128 + nt * 64 + lane]);
        W.w3[nt] = as_bf8(wfrag[256 + 1152 + nt * 64 + lane]);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) W.w2[t][nt] = as_bf8(wfrag[256 + (t * 2 + nt) * 64 + lane]);
    const int first = xcd_tile(blockIdx.x, gridDim.x) * per_block;
    const int last = min(first + per_block, ntiles);
    if (first >= last) return;
    TileInput in;
    load_tile_input(in, r, kh2, mx, my, (first / tiles_x) * IT, (first % tiles_x) * IT);
    // this thread's output point of the tile
    const int py = tid >> 4, px = tid & 15;
    for (int tile = first; tile < last; ++tile) {
        const int oy = (tile / tiles_x) * IT, ox = (tile % tiles_x) * IT;
        store_tile_input(S, in, mx, my, oy, ox);
        __syncthreads();
        if (tile + 1 < last)
            load_tile_input(in, r, kh2, mx, my, ((tile + 1) / tiles_x) * IT, ((tile + 1) % tiles_x) * IT);
        const int gy = oy + py, gx = ox + px;
        const bool mine = gy < my && gx < mx;
        const size_t j = mine ? (size_t)gy * mx + gx : 0;
        const cd uv = u[j];
        // the layer-1 region (origin -2, side 20) lies inside the grid
        const bool interior = oy >= 2 && ox >= 2 && oy + IT + 2 <= my && ox + IT + 2 <= mx;
        if (interior)
            net_layers<false>(S, mx, my, oy, ox, W, wave);
        else
            net_layers<true>(S, mx, my, oy, ox, W, wave);
        __syncthreads();
        if (mine) {
            const float2 yv = layer3_gather(S, py, px);
            u[j] = cd{uv.re + h2 * (double)yv.x, uv.im + h2 * (double)yv.y};
        }
        // the next tile's layers 2 and 3 start two barriers on, so S.z is not
        // overwritten before it is read here
    }
}

// Channel and Re / Im part held in activation slot s (see InferLds).
static int slot_channel(int s) { return (16 * (s & 1) + (s >> 1)) / 2; }
static int slot_part(int s) { return (s >> 1) & 1; }

// MFMA A-operand fragments of the three layers from the complex weights
// (rounded to BF16): 64 lanes x 8 values per fragment, in the order read by
// k_net_apply.
void pack_net_mfma(const float *w, unsigned short *out)
{
    auto W = [&](int off, int idx, int part) { return w[2 * (off + idx) + part]; };
    // real weight of complex weight (re, im) from real input part pi to output part po
    auto real_block = [](float re, float im, int po, int pi) {
        return po == 0 ? (pi == 0 ? re : -im) : (pi == 0 ? im : re);
    };
    auto bf = [](float f) { return (unsigned short)bf16_bits(f); };
    size_t o = 0;
    // layer 1, k = 2 tap + part (k < 18), row j part j % 2 of channel j / 2: of
    // a (from the r~ weights), then of m (from the kappa~ weights)
    for (int in = 0; in < 2; ++in)
        for (int nt = 0; nt < 2; ++nt)
            for (int lane = 0; lane < 64; ++lane)
                for (int e = 0; e < 8; ++e) {
                    const int k = 8 * (lane / 16) + e, j = 16 * nt + lane % 16;
                    float v = 0.f;
                    if (k < 18) {
                        const int idx = ((k / 2) * 16 + j / 2) * 2 + in;
                        v = real_block(W(NET_W1, idx, 0), W(NET_W1, idx, 1), j % 2, k % 2);
                    }
                    out[o++] = bf(v);
                }
    for (int t = 0; t < 9; ++t)
        for (int nt = 0; nt < 2; ++nt)
            for (int lane = 0; lane < 64; ++lane)
                for (int e = 0; e < 8; ++e) {
                    const int slot = 8 * (lane / 16) + e, j = 16 * nt + lane % 16;
                    const int i = slot_channel(slot), pi = slot_part(slot), oc = j / 2, po = j % 2;
                    const int idx = (t * 16 + oc) * 16 + i;
                    out[o++] = bf(real_block(W(NET_W2, idx, 0), W(NET_W2, idx, 1), po, pi));
                }
    // layer 3: row c = 16 nt + lane % 16 is part c % 2 of tap c / 2 (< 9)
    for (int nt = 0; nt < 2; ++nt)
        for (int lane = 0; lane < 64; ++lane)
            for (int e = 0; e < 8; ++e) {
                const int slot = 8 * (lane / 16) + e, c = 16 * nt + lane % 16;
                const int t = c / 2, po = c % 2;
                float v = 0.f;
                if (t < 9) {
                    const int i = slot_channel(slot), pi = slot_part(slot);
                    const int idx = t * 16 + i;
                    v = real_block(W(NET_W3, idx, 0), W(NET_W3, idx, 1), po, pi);
                }
                out[o++] = bf(v);
            }
}

size_t net_mfma_frag_count() { return (size_t)(4 + 18 + 2) * 64 * 8; }

// kappa h^2 as packed BF16 complex
__global__ __launch_bounds__(256) void k_kappa_h2(const cd *__restrict__ q, double k02, double h2, size_t N,
                                                  unsigned *__restrict__ out)
{
    for (size_t j = (size_t)blockIdx.x * 256 + threadIdx.x; j < N; j += (size_t)gridDim.x * 256) {
        const cd qj = q[j];
        out[j] = pack_c((float)((k02 + qj.re) * h2), (float)(qj.im * h2));
    }
}

void launch_kappa_h2(const cd *q, double k02, double h2, size_t N, unsigned *out, hipStream_t s)
{
    size_t nb = std::min<size_t>((N + 255) / 256, 65536);
    hipLaunchKernelGGL(k_kappa_h2, dim3((unsigned)nb), dim3(256), 0, s, q, k02, h2, N, out);
}

void launch_net_apply(const cd *r, const unsigned *kh2, cd *u, int mx, int my, const unsigned short *wfrag,
                      double h2, hipStream_t st, const int *stop)
{
    const int tx = (mx + IT - 1) / IT, ty = (my + IT - 1) / IT, nt = tx * ty;
    const int blocks = std::min(nt, 256 * 2);   // two resident workgroups per CU
    const int per = (nt + blocks - 1) / blocks;
    const int nb = (nt + per - 1) / per;
    hipLaunchKernelGGL(k_net_apply, dim3(nb), dim3(256), 0, st, r, kh2, u, mx, my, tx, nt, per,
                       reinterpret_cast<const us8 *>(wfrag), h2, stop);
}

}  // namespace ffmg

// ===========================================================================
// C ABI: the network object (weights, Adam state, training buffers).
#include <stdarg.h>
#include <stdio.h>

#include <string>
#include <vector>

#include "../../include/ffmg.h"

struct ffmg_net {
    hipStream_t stream = nullptr;
    float2 *Wm = nullptr, *Wq = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
    float2 *dW_part = nullptr;
    float *loss_part = nullptr, *h_loss = nullptr;   // h_loss: page-locked, written by the device
    int part_cap = 0;
    int step = 0;
    std::string err;
    std::vector<void *> allocs;
};

namespace {

ffmg_status net_fail(ffmg_net *n, ffmg_status s, const char *fmt, ...)
{
    if (n) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        n->err = buf;
    }
    return s;
}

#define NCHK(n, x)                                                                                                   \
    do {                                                                                                             \
        hipError_t e_ = (x);                                                                                         \
        if (e_ != hipSuccess)                                                                                        \
            return net_fail((n), e_ == hipErrorOutOfMemory ? FFMG_ENOMEM : FFMG_EDEVICE, "%s: %s", #x,              \
                            hipGetErrorString(e_));                                                                  \
    } while (0)

template <typename P>
ffmg_status net_alloc(ffmg_net *n, P **p, size_t bytes)
{
    void *q = nullptr;
    NCHK(n, hipMalloc(&q, bytes));
    n->allocs.push_back(q);
    *p = (P *)q;
    return FFMG_OK;
}

ffmg_status check_finite(ffmg_net *n, const float *w)
{
    for (int k = 0; k < 2 * ffmg::NET_NW; ++k)
        if (!isfinite(w[k])) return net_fail(n, FFMG_ENAN, "weight %d is not finite", k / 2);
    return FFMG_OK;
}

// Losses and gradients of the patches; lr > 0: and the Adam step with that rate.
ffmg_status train_common(ffmg_net *n, const void *rt, const void *kt, const void *et, int count, int border,
                         float lr)
{
    if (!rt || !kt || !et || count < 1) return net_fail(n, FFMG_EINVAL, "null patches or count < 1");
    if (border < 1 || border > 12) return net_fail(n, FFMG_EINVAL, "border must lie in [1, 12]");
    if (n->part_cap < count) {
        if (n->dW_part) {
            (void)hipFree(n->dW_part);
            (void)hipFree(n->loss_part);
            n->allocs.erase(std::remove(n->allocs.begin(), n->allocs.end(), (void *)n->dW_part), n->allocs.end());
            n->allocs.erase(std::remove(n->allocs.begin(), n->allocs.end(), (void *)n->loss_part), n->allocs.end());
            n->dW_part = nullptr;
            n->loss_part = nullptr;
            n->part_cap = 0;
        }
        ffmg_status s = net_alloc(n, &n->dW_part, (size_t)count * ffmg::NET_NW * sizeof(float2));
        if (s != FFMG_OK) return s;
        s = net_alloc(n, &n->loss_part, (size_t)count * sizeof(float));
        if (s != FFMG_OK) return s;
        n->part_cap = count;
    }
    ffmg::launch_train_patches((const float2 *)rt, (const float2 *)kt, (const float2 *)et, n->Wq, n->dW_part,
                               n->loss_part, count, border, n->stream);
    if (lr > 0.f)
        ffmg::launch_reduce_grads_adam(n->dW_part, count, n->grad, n->loss_part, n->h_loss, n->Wm, n->Wq, n->m, n->v,
                                       lr, 0.9f, 0.999f, 1e-8f, n->step + 1, n->stream);
    else
        ffmg::launch_reduce_grads(n->dW_part, count, n->grad, n->loss_part, n->h_loss, n->stream);
    NCHK(n, hipGetLastError());
    if (lr > 0.f) n->step += 1;
    return FFMG_OK;
}

}  // namespace

extern "C" {

ffmg_status ml_net_create(const float *w, void *stream, ffmg_net **out)
{
    if (!out || !w) return FFMG_EINVAL;
    *out = nullptr;
    ffmg_net *n = new ffmg_net();
    n->stream = (hipStream_t)stream;
    ffmg_status s = check_finite(n, w);
    const size_t bytes = ffmg::NET_NW * sizeof(float2);
    if (s == FFMG_OK) s = net_alloc(n, &n->Wm, bytes);
    if (s == FFMG_OK) s = net_alloc(n, &n->Wq, bytes);
    if (s == FFMG_OK) s = net_alloc(n, &n->m, bytes);
    if (s == FFMG_OK) s = net_alloc(n, &n->v, bytes);
    if (s == FFMG_OK) s = net_alloc(n, &n->grad, bytes);
    if (s == FFMG_OK && hipHostMalloc((void **)&n->h_loss, sizeof(float), hipHostMallocDefault) != hipSuccess)
        s = net_fail(n, FFMG_ENOMEM, "hipHostMalloc failed");
    if (s == FFMG_OK) s = ml_net_set_weights(n, w);
    if (s != FFMG_OK) {
        ml_net_destroy(n);
        return s;
    }
    *out = n;
    return FFMG_OK;
}

ffmg_status ml_net_set_weights(ffmg_net *n, const float *w)
{
    if (!n || !w) return FFMG_EINVAL;
    ffmg_status s = check_finite(n, w);
    if (s != FFMG_OK) return s;
    const size_t bytes = ffmg::NET_NW * sizeof(float2);
    NCHK(n, hipMemcpyAsync(n->Wm, w, bytes, hipMemcpyHostToDevice, n->stream));
    ffmg::launch_round_weights(n->Wm, n->Wq, n->stream);
    NCHK(n, hipMemsetAsync(n->m, 0, bytes, n->stream));
    NCHK(n, hipMemsetAsync(n->v, 0, bytes, n->stream));
    n->step = 0;
    NCHK(n, hipStreamSynchronize(n->stream));
    return FFMG_OK;
}

ffmg_status ml_net_get_weights(ffmg_net *n, float *w)
{
    if (!n || !w) return FFMG_EINVAL;
    NCHK(n, hipMemcpyAsync(w, n->Wm, ffmg::NET_NW * sizeof(float2), hipMemcpyDeviceToHost, n->stream));
    NCHK(n, hipStreamSynchronize(n->stream));
    return FFMG_OK;
}

ffmg_status ml_loss_grad(ffmg_net *n, const void *rt, const void *kt, const void *et, int count, int border,
                         float *loss, float *grad)
{
    if (!n) return FFMG_EINVAL;
    ffmg_status s = train_common(n, rt, kt, et, count, border, 0.f);
    if (s != FFMG_OK) return s;
    if (grad) NCHK(n, hipMemcpyAsync(grad, n->grad, ffmg::NET_NW * sizeof(float2), hipMemcpyDeviceToHost, n->stream));
    NCHK(n, hipStreamSynchronize(n->stream));
    if (loss) *loss = *n->h_loss;
    return FFMG_OK;
}

ffmg_status ml_train_step(ffmg_net *n, const void *rt, const void *kt, const void *et, int count, int border,
                          float lr, float *loss)
{
    if (!n) return FFMG_EINVAL;
    if (!(lr > 0.f) || !isfinite(lr)) return net_fail(n, FFMG_EINVAL, "lr must be positive");
    ffmg_status s = train_common(n, rt, kt, et, count, border, lr);
    if (s != FFMG_OK) return s;
    if (loss) {
        NCHK(n, hipStreamSynchronize(n->stream));
        *loss = *n->h_loss;
    }
    return FFMG_OK;
}

const char *ml_net_last_error(const ffmg_net *n) { return n ? n->err.c_str() : "null network"; }

void ml_net_destroy(ffmg_net *n)
{
    if (!n) return;
    if (n->stream) (void)hipStreamSynchronize(n->stream);
    else (void)hipDeviceSynchronize();
    for (void *p : n->allocs) (void)hipFree(p);
    if (n->h_loss) (void)hipHostFree(n->h_loss);
    delete n;
}

}  // extern "C"
