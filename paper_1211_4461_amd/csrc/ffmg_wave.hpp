// ffmg_wave.hpp -- lane moves and sums within a wave of 64.
#pragma once

#include "ffmg_internal.hpp"

namespace ffmg {

// A value moved between the lanes of a wave by a DPP control; 0 where there is
// no source lane.
template <int CTRL>
__device__ __forceinline__ unsigned dpp_u32(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float, dpp_u32<CTRL>(__builtin_bit_cast(unsigned, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = dpp_u32<CTRL>((unsigned)b), hi = dpp_u32<CTRL>((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// the lane below (x - 1), the lane above (x + 1); within rows of 16 lanes: the
// lane n above, and a rotation by n
constexpr int DPP_WAVE_SHR1 = 0x138, DPP_WAVE_SHL1 = 0x130, DPP_ROW_SHL = 0x100, DPP_ROW_ROR = 0x120;

// The value of one lane, the same in all lanes.
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Two values a wave apart folded into one register: the lower half of the
// wave (HALF32), or the even rows of 16 lanes, get a + a moved down by 32 (16)
// lanes, the other half the same of b.
template <bool HALF32>
__device__ __forceinline__ double fold_pair(double a, double b)
{
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32), yl = (unsigned)y, yh = (unsigned)(y >> 32);
    unsigned al, ah, bl, bh;
    if constexpr (HALF32) {
        const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
        al = l[0], bl = l[1], ah = h[0], bh = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
        al = l[0], bl = l[1], ah = h[0], bh = h[1];
    }
    return __builtin_bit_cast(double, ((unsigned long long)ah << 32) | al)
         + __builtin_bit_cast(double, ((unsigned long long)bh << 32) | bl);
}

// Sums over the wave of NV doubles a lane, each by halving (32, 16, 8, 4, 2, 1
// lanes apart: the order of a tree of shuffles).  Four values share the adds of
// a register: s[h] holds in all lanes of row r of 16 the sum of value
// 4 h + wave_sum_value(r) (value 4 h + v: lane wave_sum_lane(v)); rows beyond
// the last value repeat others.  For four values 9 adds and no memory, where a
// tree of shuffles each takes 24 adds and 48 moves through LDS.
__device__ __forceinline__ constexpr int wave_sum_value(int row) { return ((row & 1) << 1) | (row >> 1); }
__device__ __forceinline__ constexpr int wave_sum_lane(int v) { return 16 * (((v & 1) << 1) | ((v >> 1) & 1)); }
template <int NV>
__device__ __forceinline__ void wave_sums(const double (&a)[NV], double (&s)[(NV + 3) / 4])
{
#pragma unroll
    for (int h = 0; h < (NV + 3) / 4; ++h) {
        constexpr auto at = [](int i) { return i < NV ? i : NV - 1; };
        const double x = fold_pair<true>(a[4 * h], a[at(4 * h + 1)]);
        double r = x;
        if (4 * h + 2 < NV) r = fold_pair<true>(a[at(4 * h + 2)], a[at(4 * h + 3)]);
        r = fold_pair<false>(x, r);
        r += dpp_mov<DPP_ROW_ROR + 8>(r);
        r += dpp_mov<DPP_ROW_ROR + 4>(r);
        r += dpp_mov<DPP_ROW_ROR + 2>(r);
        r += dpp_mov<DPP_ROW_ROR + 1>(r);
        s[h] = r;
    }
}

// Sums over a workgroup of NW waves (a power of two, at most 16), in s as
// wave_sums leaves them, the same in every wave: the waves' sums through red
// (LDS, behind which one barrier stands), then by halving.  red must not be one
// that a wave may still read: two used in turn, with a barrier between the
// uses, do.
template <int NV, int NW>
__device__ __forceinline__ void block_sums(const double (&a)[NV], double (&s)[(NV + 3) / 4], double *red)
{
    static_assert(NW <= 16 && (NW & (NW - 1)) == 0, "waves of a workgroup");
    wave_sums<NV>(a, s);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int v0 = wave_sum_value(lane >> 4);
#pragma unroll
    for (int h = 0; h < (NV + 3) / 4; ++h)
        if ((lane & 15) == 0 && 4 * h + v0 < NV) red[(4 * h + v0) * NW + wv] = s[h];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < (NV + 3) / 4; ++h) {
        double r = red[min(4 * h + v0, NV - 1) * NW + (lane & (NW - 1))];
        if (NW > 8) r += dpp_mov<DPP_ROW_ROR + 8>(r);
        if (NW > 4) r += dpp_mov<DPP_ROW_ROR + 4>(r);
        if (NW > 2) r += dpp_mov<DPP_ROW_ROR + 2>(r);
        if (NW > 1) r += dpp_mov<DPP_ROW_ROR + 1>(r);
        s[h] = r;
    }
}

}  // namespace ffmg
