// Rotations, inner products, sums and extremes across the lanes of a wave, on DPP
// operands.
//
// The lanes of a row of 16 hold four index bits; the lane number is the XOR of
// the masks 1, 2, 7, 15 of the bits that are set, so that a bit's partner lane
// is one DPP step away (quad_perm, row_half_mirror, row_mirror). The compiler
// does not fold a DPP move into a fused multiply-add, which would cost a move
// per operand, so the blocks below are written out. Each starts with the two
// wait states that a DPP read needs after the last vector write of its source,
// and reads nothing by DPP that it has written within the two instructions
// before. All 64 lanes must be active.
#pragma once

#include "common.h"

namespace pq {

__device__ inline float2 cmul(float2 a, float2 b)
{
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__host__ __device__ constexpr uint32_t row_lanes(uint32_t bits)
{
    return (bits & 1u ? 1u : 0u) ^ (bits & 2u ? 2u : 0u) ^ (bits & 4u ? 7u : 0u) ^ (bits & 8u ? 15u : 0u);
}
// the inverse: index bits of a lane of the row
__host__ __device__ constexpr uint32_t row_bits(uint32_t lane)
{
    const uint32_t a = lane & 8u ? lane ^ 15u : lane;  // without bit 3's mask
    const uint32_t b = a & 4u ? a ^ 7u : a;
    return (lane & 8u) | (a & 4u) | (b & 3u);
}

#define PQ_DPP0 "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
#define PQ_DPP1 "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
#define PQ_DPP2 "row_half_mirror row_mask:0xf bank_mask:0xf"
#define PQ_DPP3 "row_mirror row_mask:0xf bank_mask:0xf"

// the value of the lane that differs in row bit K
template <int K>
__device__ inline float across(float x)
{
    constexpr int CTRL = K == 0 ? 0xB1 : K == 1 ? 0x4E : K == 2 ? 0x141 : 0x140;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// x += t * (partner's y), y -= t * (partner's old x), four amplitudes
#define PQ_RX_LANE(D)                                                                                            \
    asm("s_nop 1\n\t"                                                                                            \
        "v_mov_b32 %8, %0\n\t"                                                                                   \
        "v_mov_b32 %9, %2\n\t"                                                                                   \
        "v_mov_b32 %10, %4\n\t"                                                                                  \
        "v_mov_b32 %11, %6\n\t"                                                                                  \
        "v_fmac_f32_dpp %0, %1, %12 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %2, %3, %12 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %4, %5, %12 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %6, %7, %12 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %1, %8, %13 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %3, %9, %13 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %5, %10, %13 " D "\n\t"                                                                  \
        "v_fmac_f32_dpp %7, %11, %13 " D                                                                         \
        : "+v"(v[r].x), "+v"(v[r].y), "+v"(v[r + 1].x), "+v"(v[r + 1].y), "+v"(v[r + 2].x), "+v"(v[r + 2].y),    \
          "+v"(v[r + 3].x), "+v"(v[r + 3].y), "=&v"(s0), "=&v"(s1), "=&v"(s2), "=&v"(s3)                         \
        : "v"(t), "v"(-t))

// rotation (I - i t X) of row bit K
template <int K, int R>
__device__ inline void rx_lane(float2 (&v)[R], float t)
{
    if constexpr (R % 4 == 0) {
#pragma unroll
        for (int r = 0; r < R; r += 4) {
            float s0, s1, s2, s3;
            if constexpr (K == 0) PQ_RX_LANE(PQ_DPP0);
            else if constexpr (K == 1) PQ_RX_LANE(PQ_DPP1);
            else if constexpr (K == 2) PQ_RX_LANE(PQ_DPP2);
            else PQ_RX_LANE(PQ_DPP3);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float px = across<K>(v[r].x), py = across<K>(v[r].y);
            v[r] = make_float2(fmaf(py, t, v[r].x), fmaf(px, -t, v[r].y));
        }
    }
}

// per amplitude la.x * (partner's ps.y) - la.y * (partner's ps.x), which cancel, one
// after the other into a (even registers) or b (odd ones)
#define PQ_XB_LANE(D)                                                                                            \
    asm("s_nop 1\n\t"                                                                                            \
        "v_fmac_f32_dpp %0, %3, %10 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %1, %5, %12 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %0, %2, -%11 " D "\n\t"                                                                  \
        "v_fmac_f32_dpp %1, %4, -%13 " D "\n\t"                                                                  \
        "v_fmac_f32_dpp %0, %7, %14 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %1, %9, %16 " D "\n\t"                                                                   \
        "v_fmac_f32_dpp %0, %6, -%15 " D "\n\t"                                                                  \
        "v_fmac_f32_dpp %1, %8, -%17 " D                                                                         \
        : "+&v"(a), "+&v"(b)                                                                                     \
        : "v"(ps[r].x), "v"(ps[r].y), "v"(ps[r + 1].x), "v"(ps[r + 1].y), "v"(ps[r + 2].x), "v"(ps[r + 2].y),    \
          "v"(ps[r + 3].x), "v"(ps[r + 3].y), "v"(la[r].x), "v"(la[r].y), "v"(la[r + 1].x), "v"(la[r + 1].y),    \
          "v"(la[r + 2].x), "v"(la[r + 2].y), "v"(la[r + 3].x), "v"(la[r + 3].y))

// sum over the lane's amplitudes of Im conj(lam(z)) psi(z ^ row bit K)
template <int K, int R>
__device__ inline float xb_lane(const float2 (&ps)[R], const float2 (&la)[R])
{
    float a = 0.f, b = 0.f;
    if constexpr (R % 4 == 0) {
#pragma unroll
        for (int r = 0; r < R; r += 4) {
            if constexpr (K == 0) PQ_XB_LANE(PQ_DPP0);
            else if constexpr (K == 1) PQ_XB_LANE(PQ_DPP1);
            else if constexpr (K == 2) PQ_XB_LANE(PQ_DPP2);
            else PQ_XB_LANE(PQ_DPP3);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float& x = r & 1 ? b : a;
            x = fmaf(across<K>(ps[r].y), la[r].x, x);
            x = fmaf(-across<K>(ps[r].x), la[r].y, x);
        }
    }
    return a + b;
}

// exchanges lane bit 4 (H = 16) or 5 (H = 32) of a pair of registers: afterwards
// a holds the values of both registers' lower halves and b those of the upper
template <int H>
__device__ inline void swap_halves(float& a, float& b)
{
    const uint32_t x = __float_as_uint(a), y = __float_as_uint(b);
    if constexpr (H == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        a = __uint_as_float(s[0]);
        b = __uint_as_float(s[1]);
    } else {
        const auto s = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        a = __uint_as_float(s[0]);
        b = __uint_as_float(s[1]);
    }
}

// Sum over the wave in every lane, without LDS (a butterfly of lane
// permutations has six LDS latencies in a chain).
template <int K>
__device__ inline double across(double x)
{
    const uint64_t u = __double_as_longlong(x);
    const uint32_t lo = __float_as_uint(across<K>(__uint_as_float((uint32_t)u)));
    const uint32_t hi = __float_as_uint(across<K>(__uint_as_float((uint32_t)(u >> 32))));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <int H>
__device__ inline double halves_sum(double x)
{
    const uint64_t u = __double_as_longlong(x);
    float l0 = __uint_as_float((uint32_t)u), h0 = __uint_as_float((uint32_t)(u >> 32)), l1 = l0, h1 = h0;
    swap_halves<H>(l0, l1);
    swap_halves<H>(h0, h1);
    const double a = __longlong_as_double((long long)(((uint64_t)__float_as_uint(h0) << 32) | __float_as_uint(l0)));
    const double b = __longlong_as_double((long long)(((uint64_t)__float_as_uint(h1) << 32) | __float_as_uint(l1)));
    return a + b;
}
__device__ inline double wave_total(double x)
{
    x += across<0>(x);
    x += across<1>(x);
    x += across<2>(x);
    x += across<3>(x);
    return halves_sum<32>(halves_sum<16>(x));
}

// the wave's largest / smallest value, by lane permutations that need no LDS
template <typename F>
__device__ inline uint32_t wave_fold(uint32_t x, F pick)
{
    x = pick(x, __float_as_uint(across<0>(__uint_as_float(x))));
    x = pick(x, __float_as_uint(across<1>(__uint_as_float(x))));
    x = pick(x, __float_as_uint(across<2>(__uint_as_float(x))));
    x = pick(x, __float_as_uint(across<3>(__uint_as_float(x))));
    float a = __uint_as_float(x), c = a;
    swap_halves<16>(a, c);
    x = pick(__float_as_uint(a), __float_as_uint(c));
    a = c = __uint_as_float(x);
    swap_halves<32>(a, c);
    return pick(__float_as_uint(a), __float_as_uint(c));
}
__device__ inline uint32_t wave_max(uint32_t x)
{
    return wave_fold(x, [](uint32_t a, uint32_t c) { return a > c ? a : c; });
}
__device__ inline uint32_t wave_min(uint32_t x)
{
    return wave_fold(x, [](uint32_t a, uint32_t c) { return a < c ? a : c; });
}

}  // namespace pq
