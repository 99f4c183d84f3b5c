// Products of binary32 matrices on the fp16 MFMA: a value is a scaled pair of halves, a product three MFMAs.  Shared by the Hessian
// product and the GPTQ sweep's update.
#pragma once

#include "device_util.hpp"

namespace fp4mr {

// An operand lies in stages of 32 along the contraction; the other index goes in blocks of sixteen, in which lane (c, q) holds
// element c at 8 q .. 8 q + 7 of the contraction: the high halves of the 64 lanes, then the low ones.
constexpr int kPairBytes = 2048;

// A value y is (h + l) 2^(e - 14), e an exponent that some neighbourhood shares and in which |y| < 2^(e + 1): h the nearest fp16
// of y's share, l that of what is left -- y itself or, where the remainder's 13th bit is set, y but for 2^-23 of it, down to
// 2^(e - 17) (below, l has a fixed last place: 2^(e - 39)).  Exponents are biased, 14 at least (2^(14 - e) is a normal number then,
// also where e says infinity).  A sum of products takes up the row's as an integer, in v_ldexp_f32, and the column's as a factor, in the
// fused multiply-add onto what is there: results may have any size of binary32, whatever the two sides' exponents are (the first step
// overflows where a row's values reach 2^118 or more; what it loses below 2^-149 is 2^-38 of the largest product).
__device__ __forceinline__ uint32_t pair_exponent(float largest) { return max(__float_as_uint(largest) >> 23, 14u); }
__device__ __forceinline__ float pair_up(uint32_t e) { return __uint_as_float((268u - e) << 23); }
constexpr int kPairRow = 127 + 27;   // the row's step: its exponent less this
__device__ __forceinline__ float pair_column(uint32_t e) { return __uint_as_float((e - 1u) << 23); }   // the column's factor, for the other 2^-1 of 2^-28

__device__ __forceinline__ void pair_split(float y, float up, _Float16& h, _Float16& l)
{
    const float s = y * up;
    h = (_Float16)s;
    l = (_Float16)(s - (float)h);
}

// of the column's and the row's two parts: the products that count, small ones first (low times low is 2^-23 of the whole)
__device__ constexpr int kPairParts[3][2] = {{1, 0}, {0, 1}, {0, 0}};

// A wave's 16 NT x 16 NT sums.  The three products of 32 terms are summed from zero in the MFMA (which cuts off what an addition
// leaves over), a few such sums in t, and those, with their exponents, in acc.  The column operand is the MFMA's A, so that a
// lane owns four neighbouring columns of a row.
template <int NT>
struct PairSums {
    v4f acc[NT][NT], t[NT][NT];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    }

    template <bool FIRST>
    __device__ __forceinline__ void add(int i, int j, v4f sum)
    {
        if constexpr (FIRST) t[i][j] = sum;
        else t[i][j] += sum;
    }

    // one stage, the FIRST of those that are added up in t or another; rows, cols: the wave's first block of either operand in LDS
    template <bool FIRST>
    __device__ __forceinline__ void multiply(const char* rows, const char* cols)
    {
        const int lane = threadIdx.x & 63;
        auto block = [&](const char* s, int i, int part) { return *(reinterpret_cast<const v8h*>(s + i * kPairBytes + part * 1024) + lane); };
        v8h u[2][NT], next[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) next[k] = block(rows, 0, k);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) u[k][j] = block(cols, j, k);
        v4f sum[2][NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const v8h e[2] = {next[0], next[1]};
            if (i + 1 < NT) {
#pragma unroll
                for (int k = 0; k < 2; ++k) next[k] = block(rows, i + 1, k);
            }
            __builtin_amdgcn_sched_barrier(0);
            // (the sums of the row block before are added up between the products of this one)
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    v4f& d = sum[i & 1][j];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_f16(u[kPairParts[s][0]][j], e[kPairParts[s][1]], s ? d : v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    if (i && s == 0) add<FIRST>(i - 1, j, sum[(i - 1) & 1][j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) add<FIRST>(NT - 1, j, sum[(NT - 1) & 1][j]);
    }

    // t onto acc; row: the step of the lane's row in row block i, col: the factors of the four columns in column block j
    template <typename Row, typename Col>
    __device__ __forceinline__ void scale(Row row, Col col)
    {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int e = row(i);
                const v4f f = col(j);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = fmaf(__builtin_amdgcn_ldexpf(t[i][j][v], e), f[v], acc[i][j][v]);
            }
    }
};

}  // namespace fp4mr
