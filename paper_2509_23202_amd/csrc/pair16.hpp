// Products of binary32 matrices on the fp16 MFMA: a value is a scaled pair of halves, a product three MFMAs.  Shared by the Hessian
// product and the GPTQ sweep's update.
#pragma once

#include "device_util.hpp"

#include <type_traits>
#include <utility>

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

// 16 bytes a lane to LDS, one behind the other from dst (in a function of its own: these builtins are not known to the host's compiler)
__device__ __forceinline__ void copy_to_lds(__amdgpu_buffer_rsrc_t from, char* dst, uint32_t lane_at, int at)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (lds_void*)dst, 16, lane_at, at, 0, 0);
}

// f(0) .. f(N - 1), of constants
template <int... I, class F>
__device__ __forceinline__ void each(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void each(F f) { each(std::make_integer_sequence<int, N>{}, f); }

// a wave's share of a stage in registers: its blocks of either operand, their high and low halves
template <int NT>
struct PairOperands {
    v8h rows[2][NT], cols[2][NT];

    // the first block of either in LDS
    __device__ __forceinline__ void fetch(const char* r, const char* c)
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                rows[k][i] = *(reinterpret_cast<const v8h*>(r + i * kPairBytes + k * 1024) + lane);
                cols[k][i] = *(reinterpret_cast<const v8h*>(c + i * kPairBytes + k * 1024) + lane);
            }
    }
};

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
            // (the sums of the row block before are added up between the products of this one, one or two behind each: sixteen behind its first
            // four, the Hessian of 1408 rows, K = 8192 took 341 us, now 325, and the GPTQ sweep of [6144, 4096] 9 us more)
#pragma unroll
            for (int m = 0; m < 3 * NT; ++m) {
                const int s = m / NT, j = m % NT;
                v4f& d = FIRST ? t[i][j] : sum[i & 1][j];
                d = __builtin_amdgcn_mfma_f32_16x16x32_f16(u[kPairParts[s][0]][j], e[kPairParts[s][1]], s ? d : v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (!FIRST && i) {
#pragma unroll
                    for (int v = m * 4 / 3; v < (m + 1) * 4 / 3; ++v) t[i - 1][v / 4][v % 4] += sum[(i - 1) & 1][v / 4][v % 4];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!FIRST) {
#pragma unroll
            for (int j = 0; j < NT; ++j) t[NT - 1][j] += sum[(NT - 1) & 1][j];
        }
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

// The same sums of stages whose operands are in registers, with the additions spread between the MFMAs: a wave that has its SIMD's issue to
// itself hides one vector instruction or two behind an MFMA, not sixteen behind a dozen (48 MFMAs of 16 cycles and 64 additions: 1320
// cycles in a row, 850 spread).  So the additions of a row of blocks go between the MFMAs of the next one, the last row's between the first of the stage
// behind (PENDING).  The FIRST stage of a group is summed in t itself, row by row behind the last group's step onto acc, which goes
// between the MFMAs of the row before; the first row's, in begin(), runs while another wave multiplies.
template <int NT>
struct PairChain {
    v4f acc[NT][NT], t[NT][NT], sum[2][NT];
    int row[NT];   // of the last group: the step of a lane's row, the factors of its columns
    v4f col[NT];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = t[i][j] = sum[1][j] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    // nothing of a group is left to be added
    __device__ __forceinline__ void restart()
    {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) t[i][j] = sum[1][j] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void step(int i, int j, int v) { acc[i][j][v] = fmaf(__builtin_amdgcn_ldexpf(t[i][j][v], row[i]), col[j][v], acc[i][j][v]); }

    // between two groups, of which the first has more than one stage or none, in NT + 2 parts; Row, Col: its exponents, as of PairSums::scale
    static constexpr int kBegin = NT + 2;
    template <int PART, class Row, class Col>
    __device__ __forceinline__ void begin(Row r, Col c)
    {
        static_assert(NT % 2 == 0, "sum[1] is the last row's");
        if constexpr (PART < 2) {
#pragma unroll
            for (int j = PART * NT / 2; j < (PART + 1) * NT / 2; ++j) {
                row[j] = r(j);
                col[j] = c(j);
            }
        } else {
            constexpr int j = PART - 2;
            t[NT - 1][j] += sum[1][j];
#pragma unroll
            for (int v = 0; v < 4; ++v) step(0, j, v);
        }
    }
    // behind the last one
    template <class Row, class Col>
    __device__ __forceinline__ void end(Row r, Col c)
    {
        each<kBegin>([&](auto part) { begin<part.value>(r, c); });
#pragma unroll
        for (int i = 1; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) step(i, j, v);
    }

    template <bool FIRST, bool PENDING>
    __device__ __forceinline__ void multiply(const PairOperands<NT>& x)
    {
        constexpr int MFMAS = 3 * NT, VALUES = 4 * NT;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int m = 0; m < MFMAS; ++m) {
                const int s = m / NT, j = m % NT;
                v4f& d = FIRST ? t[i][j] : sum[i & 1][j];
                d = __builtin_amdgcn_mfma_f32_16x16x32_f16(x.cols[kPairParts[s][0]][j], x.rows[kPairParts[s][1]][i], s ? d : v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = m * VALUES / MFMAS; e < (m + 1) * VALUES / MFMAS; ++e) {
                    if (FIRST && i + 1 < NT) step(i + 1, e / 4, e % 4);
                    if (!FIRST && (i || PENDING)) t[i ? i - 1 : NT - 1][e / 4][e % 4] += sum[(i + 1) & 1][e / 4][e % 4];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
    }
};

// Eight waves that go through the stages of a product in two fours, each with an output of its own: while one four multiplies a stage that
// it holds in registers (MFMAs and the additions between them), the other reads its next one from LDS and requests copies; then they change
// over.  Every SIMD has a wave of either, so its matrix core works all the time, where waves that do both by themselves wait for the LDS
// together.  Both read the same stages, four 0 stage n in phase 2 n, four 1 in phase 2 n + 1, and multiply them in the phase behind.
//   issue(n, between):       this wave's share (COPIES of them) of copying stage n into slot n % 3, between(c) behind the c-th but the last; n past
//                            the end: anything, never read
//   begin(c):                what is to be done between two groups, in COPIES - 1 parts (the copies keep the wave waiting)
//   fetch(n, i), multiply(i):   stage n, the i-th of a group (a constant)
// In phase 2 n four 0 requests its share of stage n + 2, in phase 2 n + 1 four 1, into the slot that was read last in phase 2 n - 1; they are read from
// phase 2 n + 4 on.  The wait leaves a wave's latest request on its way: the one before has landed by the end of phase 2 n + 2 or 2 n + 3.
template <int COPIES, int GROUP, class Issue, class Begin, class Fetch, class Multiply>
__device__ __forceinline__ void pair_alternate(int four, int groups, Issue issue, Begin begin, Fetch fetch, Multiply multiply)
{
    auto nothing = [](auto) {};
    auto change = [] {
        __builtin_amdgcn_sched_barrier(0);
        block_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    issue(0, nothing);
    issue(1, nothing);
    wait_vmcnt<COPIES>();
    change();
    if (four == 1) change();
    auto stage = [&](int n, auto i) {
        fetch(n, i);
        if constexpr (i.value == 0) {
            issue(n + 2, [&](auto c) {
                __builtin_amdgcn_sched_barrier(0);
                begin(c);
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            issue(n + 2, nothing);
        }
        wait_lgkmcnt0();
        wait_vmcnt<COPIES>();
        change();
        __builtin_amdgcn_s_setprio(1);
        multiply(i);
        __builtin_amdgcn_s_setprio(0);
        change();
    };
#pragma unroll 1
    for (int n = 0; n < groups * GROUP; n += GROUP) each<GROUP>([&](auto i) { stage(n + i, i); });
    if (four == 0) change();
    wait_vmcnt<0>();
}

}  // namespace fp4mr
