// MR-GPTQ weight quantizer, the part that runs over the weight matrix (arXiv 2509.23202, Section 4: GPTQ quantizes
// all rows in one fixed column order and, after rounding a column, moves the columns not yet rounded by the
// optimal-brain update; Section 4.1: on rotated weights, with the scales fixed beforehand in the original column
// order and the columns visited in a static activation order).
//
// Given U, the upper-triangular factor of the damped inverse Hessian in visiting order (U^T U = Hinv), column j costs
//     q = Q(w_j / s),   e = (w_j - q s) / U[j,j],   w_k -= e U[j,k]  for every later column k.
// Rows never interact, so the sweep is data-parallel over the N rows and strictly sequential along K.  It is blocked
// 64 columns at a time inside outer blocks of 512: a workgroup owns 16 rows of an outer block, its working weights in LDS, and
// sweeps block by block, moving every block's errors onto the later ones (outer kernel, one launch per outer block); a
// finished outer block updates everything behind it in one rank-512 product (update kernel).  Working weights live in visiting
// order in an fp32 scratch matrix, codes in a byte-per-code scratch matrix, and a last kernel packs them back to the original
// column positions.
#include "device_util.hpp"
#include "internal.hpp"
#include "pair16.hpp"

#include <algorithm>
#include <cmath>

namespace fp4mr {
namespace {

constexpr int kB = 64;       // columns per block of the sequential sweep
constexpr int kOuter = 512;  // columns per outer block: later columns receive its errors in one rank-512 update

struct GptqArgs {
    const uint16_t* w;      // [N,K] bf16
    const float* U;         // [K,K] fp32, upper triangle used
    const int* perm;        // [K] or null
    int* iperm;             // [K] scratch
    float* wp;              // [N,K] scratch: working weights, visiting order
    uint8_t* q;             // [N,K] scratch: one code per byte, visiting order
    // scratch, the operands of an outer block's update as scaled pairs of halves (pair16.hpp), 16 stages along the contraction:
    char* e_pairs;          // errors, [stage][16 rows]
    int* e_scales;          // [kOuter / kB][rows]: their exponents: of a row's errors of 64 columns
    char* u_pairs;          // rows of U, [stage][16 columns]
    float* u_scales;        // [kOuter / kB][K]: of a column's entries in 64 rows, as factors
    float* err;             // ... or, in a workspace without room for those, the errors as they are, [N, kOuter]; else null
    int Np;                 // N rounded up to 16
    const uint8_t* scales;  // [N,K/G] canonical
    const float* s_T;       // NVFP4 tensor scale (device), else null
    const float* table;     // 256 scale values indexed by the scale byte (fitted scale range), else null
    uint8_t* codes;         // [N,K/2] canonical
    int N, K, b, G;
    float c_hi, c_lo;       // 1/sqrt(b) in two floats
    float factor;           // 4/3 for scales that leave that factor out, else 1
};

__device__ __forceinline__ int visit_col(const GptqArgs& a, int j)
{
    // an entry outside [0, K) (not a permutation: caller error) is clamped, so that no access leaves the buffers
    const int c = a.perm ? a.perm[j] : j;
    return min(max(c, 0), a.K - 1);
}

// wp[n, j] = (W H_b)[n, perm[j]]: the rotated weight of the column visited j-th.  One workgroup per row.  A thread rotates sixteen
// neighbouring columns in registers -- butterflies, the levels above sixteen across lanes (fp32 sums of b bf16 values, exact while
// the values' exponents spread over no more than 16 - log2(b) bits: 9 at b = 128, 12 at 16; beyond, every level rounds, log2(b)
// roundings where a sequential sum has b), then one multiplication by 1/sqrt(b) carried in two floats -- and the
// row is read back from LDS in visiting order for whole-line stores.  With a sum over the block per column, from LDS, [6144, 4096]
// took 91 us at b = 16 and 486 at b = 128; now 39 at either.  The first workgroup inverts the order as well (an entry that is no
// column's position, where the order is not a permutation, names a column all the same).
__global__ __launch_bounds__(256) void gptq_rotate_gather_kernel(GptqArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float rowbuf[];  // K floats
    if (blockIdx.x == 0) {
        for (int j = threadIdx.x; j < a.K; j += 256) a.iperm[j] = j;
        __syncthreads();
        for (int j = threadIdx.x; j < a.K; j += 256) a.iperm[visit_col(a, j)] = j;
    }
    const int n = blockIdx.x, levels = a.b <= 16 ? 0 : (a.b == 32 ? 1 : a.b == 64 ? 2 : 3);
    const uint4* src = reinterpret_cast<const uint4*>(a.w + (int64_t)n * a.K);
    // (K is a multiple of 64 and of b, so the lanes that exchange values are in or out of the row together)
    for (int c = threadIdx.x; c < a.K / 16; c += 256) {
        const uint4 lo = src[2 * c], hi = src[2 * c + 1];
        const uint32_t raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        float v[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[2 * i] = __uint_as_float(raw[i] << 16);
            v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
        }
        if (a.b > 1) {
#pragma unroll
            for (int d = 1; d < 16; d <<= 1)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (!(i & d)) {
                        const float x = v[i], y = v[i + d];
                        v[i] = x + y;
                        v[i + d] = x - y;
                    }
            for (int l = 0; l < levels; ++l) {
                const bool upper = (threadIdx.x >> l) & 1;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float o = __shfl_xor(v[i], 1 << l);
                    v[i] = upper ? o - v[i] : v[i] + o;
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = __fmaf_rn(v[i], a.c_hi, v[i] * a.c_lo);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) reinterpret_cast<float4*>(rowbuf)[4 * c + i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
    __syncthreads();
    float4* dst = reinterpret_cast<float4*>(a.wp + (int64_t)n * a.K);
    for (int j = threadIdx.x; j < a.K / 4; j += 256)
        dst[j] = make_float4(rowbuf[visit_col(a, 4 * j)], rowbuf[visit_col(a, 4 * j + 1)], rowbuf[visit_col(a, 4 * j + 2)], rowbuf[visit_col(a, 4 * j + 3)]);
}

template <int FMT>
__device__ __forceinline__ float decode_scale(uint32_t byte, float s_T, float factor)
{
    if constexpr (FMT == 0) {
        // 2^(byte - 127); byte 0 is 2^-127 (a subnormal in binary32, formed exactly)
        const float p = byte ? __uint_as_float(byte << 23) : __uint_as_float(0x00400000u);
        return p * factor;
    } else {
        return e4m3_decode<false>(byte) * s_T;
    }
}

// One outer block (columns o .. oe-1 in visiting order) of 16 rows in one workgroup, its working weights in LDS for as long
// as it lasts.  Columns are strictly sequential, so what bounds this is the chain from column to column; everything else is
// taken out of it.  Four waves sweep: sixteen lanes share a row, lane `part` holding the working weights of the columns
// 4 part .. 4 part + 3 of the current 64-column block, so that a column costs a lane four updates; the column's weight is
// broadcast along the sixteen lanes and all of them round it and form its error.  Four waves push: while block b is swept
// they move the errors of block b - 1 onto the blocks behind b (whose turn is not yet) and fetch block b + 1's triangle of U
// and scales; between two sweeps they only move block b's errors onto block b + 1, whose factor is in registers by then.  A push
// is a [16 x 64] x [64 x 16] product per 16 columns on the fp32 MFMA (v_mfma_f32_16x16x4_f32), summed from zero and
// subtracted once.  Blocks receive the pushes in ascending order.
// [6144, 4096]: 149 us per outer block with one wave per 16 rows doing all of this in turn, its weights in global memory.
// The rounding uses the converting instructions (round-to-nearest-even onto E2M1, saturating; decode back to fp32); the two
// divisions of the definition are multiplications by reciprocals formed once (exact for power-of-two scales and a unit
// diagonal).
typedef float v2f_t __attribute__((ext_vector_type(2)));

constexpr int kStages = kOuter / 32;
// 16-wide block `block` of a stage of an operand of `blocks` blocks
__device__ __forceinline__ int64_t pairs_at(int stage, int blocks, int block) { return ((int64_t)stage * blocks + block) * kPairBytes; }

// the largest |v| that is finite (an infinite error or NaN must not take its neighbours' scale)
__device__ __forceinline__ float largest_finite(float a, float v)
{
    const float f = fabsf(v);
    return f < INFINITY ? fmaxf(a, f) : a;
}

// The power of two next to U[j,j], from its reciprocal: column j's errors are multiplied by it where they become operands of the update,
// row j of U by its inverse.  Errors are as large as the channel is loud, (w - q) / U[j,j], and channels that have nothing to do with the
// loud ones among their 64 need all bits of theirs; the products of both factors then have the size of w - q.
__device__ __forceinline__ float error_factor(float r)
{
    return __uint_as_float((254u - min(max(__float_as_uint(r) >> 23 & 255u, 1u), 253u)) << 23);
}
__device__ __forceinline__ float inverse_power(float p) { return __uint_as_float(0x7f000000u - __float_as_uint(p)); }

// A lane's values of sixteen rows or columns by two stages into both, `step` bytes apart; the lane's row's exponent.
__device__ __forceinline__ uint32_t put_pairs(const float (&v)[2][8], char* dst, int64_t step)
{
    float top = 0.0f;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) top = largest_finite(top, v[s][i]);
    top = fmaxf(top, __shfl_xor(top, 16));
    top = fmaxf(top, __shfl_xor(top, 32));
    const uint32_t e = pair_exponent(top);
    const float up = pair_up(e);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        v8h h, l;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            _Float16 hi, lo;
            pair_split(v[s][i], up, hi, lo);
            h[i] = hi;
            l[i] = lo;
        }
        v8h* d = reinterpret_cast<v8h*>(dst + s * step) + (threadIdx.x & 63);
        d[0] = h;
        d[64] = l;
    }
    return e;
}

// a lane's share of 64 rows of U from row j0 of the outer block at o, in column col; Rp: the block's error factors
__device__ __forceinline__ void factor_rows(const GptqArgs& a, int o, int j0, int col, const float* Rp, float (&v)[2][8])
{
    const int r = j0 + 8 * (threadIdx.x >> 4 & 3);
    const float* src = a.U + (int64_t)(o + r) * a.K + col;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[s][i] = src[(int64_t)(32 * s + i) * a.K];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[s][i] *= inverse_power(Rp[r + 32 * s + i]);
}

// Rows o .. o + 511 of U, columns 16 cb .. 16 cb + 15, for the update behind the outer block; eight waves, 64 rows each.
__device__ __forceinline__ void pack_u(const GptqArgs& a, int o, int cb, const float* Rp)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15;
    float v[2][8];
    factor_rows(a, o, 64 * wave, cb * 16 + l16, Rp, v);
    const uint32_t e = put_pairs(v, a.u_pairs + pairs_at(2 * wave, a.K / 16, cb), pairs_at(1, a.K / 16, 0));
    if (lane < 16) a.u_scales[wave * a.K + cb * 16 + l16] = pair_column(e);
}

constexpr int kWStride = kOuter + 4;   // floats per row of working weights in LDS: rows start four banks apart
constexpr int kEStride = kB + 4;

// a weight rounded onto the grid of its scale: the code and the grid value (e2m1), before the scale
__device__ __forceinline__ float round_e2m1(float wj, float inv_scale, uint32_t& packed)
{
    const float t = wj * inv_scale;
    packed = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(packed, t, t, 1.0f, 0);   // (writes the low byte; the rest is not looked at)
    return __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(packed, 1.0f, 0)[0];
}

// what four columns of the sweep read from LDS: scale and reciprocal (0 for a zero scale), 1 / U[j,j], the lane's part of row j
// of the triangle.  The triangle is zero on and below the diagonal: a column that has been visited keeps the weight that was rounded,
// from which its lane makes code and error once more when the block is done -- two selects per column less in the chain.
// (As long as errors are finite: an infinite or NaN one times zero takes the visited columns of its row with it.  A block that
// comes out with a weight that is not finite is swept once more with KEEP, which puts every weight aside as it is rounded: to do so
// always costs 4 us per 512 columns of [6144, 4096].)
struct SweepOperands {
    v2f_t sc[4];
    float4 ru, u[4];
};

__device__ __forceinline__ SweepOperands sweep_operands(const float* Us, const float* Ru, const v2f_t* Sc, int p, int row, int part)
{
    SweepOperands x;
    x.ru = *reinterpret_cast<const float4*>(Ru + p * 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x.sc[i] = Sc[(p * 4 + i) * 16 + row];
        x.u[i] = *reinterpret_cast<const float4*>(Us + (p * 4 + i) * kB + part * 4);
    }
    return x;
}

// the four columns 4 P .. 4 P + 3 of the block, the next four's operands on their way meanwhile
template <int P, bool KEEP>
__device__ __forceinline__ void sweep_part(float (&w)[4], float (&kept)[4], uint32_t packed, const SweepOperands& x, const float* Us, const float* Ru, const v2f_t* Sc, int row, int part)
{
    SweepOperands next = x;
    if constexpr (P + 1 < 16) next = sweep_operands(Us, Ru, Sc, P + 1, row, part);
    __builtin_amdgcn_sched_barrier(0);
    const float ru[4] = {x.ru.x, x.ru.y, x.ru.z, x.ru.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        constexpr int ctrl = 0x150 + P;     // row_newbcast: the sixteen lanes of a row read lane P
        const float wj = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w[i]), ctrl, 0xf, 0xf, true));
        const float e = __fmaf_rn(-round_e2m1(wj, x.sc[i][1], packed), x.sc[i][0], wj) * ru[i];
        if (KEEP && part == P) kept[i] = wj;
        w[0] = __fmaf_rn(-e, x.u[i].x, w[0]);
        w[1] = __fmaf_rn(-e, x.u[i].y, w[1]);
        w[2] = __fmaf_rn(-e, x.u[i].z, w[2]);
        w[3] = __fmaf_rn(-e, x.u[i].w, w[3]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (P + 1 < 16) sweep_part<P + 1, KEEP>(w, kept, packed, next, Us, Ru, Sc, row, part);
}

// Barrier of the waves that share the working weights: LDS only (the sweep's stores to memory, and what the others have requested
// from there, need not have arrived: 500 cycles a time).
__device__ __forceinline__ void lds_barrier()
{
    wait_lgkmcnt0();
    block_barrier();
}

// The errors also go to memory, as operands of the update of everything behind the outer block; workgroups behind the first `rows16`
// prepare the other operand meanwhile.
template <int FMT>
__global__ __launch_bounds__(512, 4) void gptq_outer_kernel(GptqArgs a, int o, int oe, int rows16)
{
    __shared__ __attribute__((aligned(16))) float W[16 * kWStride];      // working weights of the outer block
    __shared__ __attribute__((aligned(16))) float Us[kB * kB];           // the block's triangle of U, zero on and below the diagonal
    __shared__ __attribute__((aligned(16))) v2f_t Sc[kB * 16];           // [column][row]: the block's scales and their reciprocals
    __shared__ __attribute__((aligned(16))) float Es[16 * kEStride];     // the block's errors
    __shared__ __attribute__((aligned(16))) uint8_t Sb[kOuter * 16];     // [column][row]: scale bytes of the outer block
    __shared__ __attribute__((aligned(16))) float Rd[kOuter];            // 1 / U[j,j]
    __shared__ __attribute__((aligned(16))) float Rp[kOuter];            // error_factor
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < oe - o) {
        Rd[tid] = 1.0f / a.U[(int64_t)(o + tid) * a.K + o + tid];
        Rp[tid] = error_factor(Rd[tid]);
    }
    if ((int)blockIdx.x >= rows16) {
        __syncthreads();
        pack_u(a, o, oe / 16 + (int)blockIdx.x - rows16, Rp);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.x * 16, width = oe - o, blocks = width / kB;
    const float* __restrict__ Ug = a.U;
    const float s_T = (FMT == 1) ? *a.s_T : 1.0f;

    // rows past the end shadow the last one and store nothing
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = wave * 2 + h;
        const float* src = a.wp + (int64_t)min(n0 + row, a.N - 1) * a.K + o;
        for (int c = lane * 4; c < width; c += 256) *reinterpret_cast<float4*>(&W[row * kWStride + c]) = *reinterpret_cast<const float4*>(src + c);
    }
    if (tid < width) {
        const int gshift = (a.G == 32) ? 5 : 4;
        const int group = visit_col(a, o + tid) >> gshift, groups = a.K >> gshift;
        uint32_t bytes[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 16; ++r) bytes[r >> 2] |= (uint32_t)a.scales[(int64_t)min(n0 + r, a.N - 1) * groups + group] << (8 * (r & 3));
        *reinterpret_cast<uint4*>(&Sb[tid * 16]) = make_uint4(bytes[0], bytes[1], bytes[2], bytes[3]);
    }

    // Two barriers per block, the same for the sweeping and the pushing waves: behind the sweep (its errors are in LDS), and
    // behind the push onto the next block (its weights, triangle and scales are).
    if (wave < 4) {
        __builtin_amdgcn_s_setprio(3);   // (the chain; the other four work beside it)
        lds_barrier();
        lds_barrier();
        const int row = wave * 4 + q, part = l16, n = n0 + row;
        for (int b = 0; b < blocks; ++b) {
            const float4 w4 = *reinterpret_cast<const float4*>(&W[row * kWStride + b * kB + part * 4]);
            float w[4] = {w4.x, w4.y, w4.z, w4.w}, e[4];
            const float* const Ru = Rd + b * kB;
            sweep_part<0, false>(w, w, 0u, sweep_operands(Us, Ru, Sc, 0, row, part), Us, Ru, Sc, row, part);
            if (__builtin_expect(__any(!(fabsf(w[0]) + fabsf(w[1]) + fabsf(w[2]) + fabsf(w[3]) < INFINITY)), 0)) {
                float again[4] = {w4.x, w4.y, w4.z, w4.w};
                sweep_part<0, true>(again, w, 0u, sweep_operands(Us, Ru, Sc, 0, row, part), Us, Ru, Sc, row, part);
            }
            // the lane's own four columns: w is what was rounded
            uint32_t codes = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v2f_t sc = Sc[(part * 4 + i) * 16 + row];
                uint32_t packed = 0u;
                e[i] = __fmaf_rn(-round_e2m1(w[i], sc[1], packed), sc[0], w[i]) * Ru[part * 4 + i];
                if (sc[0] > 0.0f) codes |= (packed & 15u) << (8 * i);
            }
            const float4 e4 = make_float4(e[0], e[1], e[2], e[3]);
            *reinterpret_cast<float4*>(&Es[row * kEStride + part * 4]) = e4;
            lds_barrier();
            if (n < a.N) *reinterpret_cast<uint32_t*>(a.q + (int64_t)n * a.K + o + b * kB + part * 4) = codes;
            if (oe < a.K) {   // (rows past the end too: what they hold is not stored)
                float top = 0.0f;
                const float4 f4 = *reinterpret_cast<const float4*>(&Rp[b * kB + part * 4]);
                const float f[4] = {f4.x, f4.y, f4.z, f4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    e[i] *= f[i];
                    top = largest_finite(top, e[i]);
                }
                if (a.err) {
                    if (n < a.N) *reinterpret_cast<float4*>(a.err + (int64_t)n * kOuter + b * kB + part * 4) = make_float4(e[0], e[1], e[2], e[3]);
                } else {
                    // the sixteen lanes of the row: rotations by 8, 4, 2, 1
                    top = fmaxf(top, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(top), 0x128, 0xf, 0xf, true)));
                    top = fmaxf(top, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(top), 0x124, 0xf, 0xf, true)));
                    top = fmaxf(top, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(top), 0x122, 0xf, 0xf, true)));
                    top = fmaxf(top, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(top), 0x121, 0xf, 0xf, true)));
                    const uint32_t ex = pair_exponent(top);
                    const float up = pair_up(ex);
                    typedef _Float16 v4h __attribute__((ext_vector_type(4)));
                    v4h h, l;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        _Float16 hi, lo;
                        pair_split(e[i], up, hi, lo);
                        h[i] = hi;
                        l[i] = lo;
                    }
                    // columns 4 part .. 4 part + 3 of 64: stage part / 8, there half of lane (row, (part % 8) / 2)
                    char* dst = a.e_pairs + pairs_at(2 * b + (part >> 3), a.Np / 16, blockIdx.x) + (((part & 7) >> 1) * 16 + row) * 16 + (part & 1) * 8;
                    *reinterpret_cast<v4h*>(dst) = h;
                    *reinterpret_cast<v4h*>(dst + 1024) = l;
                    if (part == 0) a.e_scales[b * a.Np + n] = (int)ex;
                }
            }
            lds_barrier();
        }
        return;
    }

    const int pt = tid - 256, pw = wave - 4;
    float4 tri[4];   // on its way to LDS for the next block
    float ea[16];    // errors of the last block (B operand: row l16, terms 4 ks + q)
    auto fetch_tri = [&](int b) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = it * 16 + (pt >> 4), c = (pt & 15) * 4;
            const float4 u = *reinterpret_cast<const float4*>(Ug + (int64_t)(o + b * kB + row) * a.K + o + b * kB + c);
            tri[it] = make_float4(c > row ? u.x : 0.0f, c + 1 > row ? u.y : 0.0f, c + 2 > row ? u.z : 0.0f, c + 3 > row ? u.w : 0.0f);
        }
    };
    v2f_t scn[4];
    auto decode_scales = [&](int b) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const uint32_t byte = Sb[b * kB * 16 + it * 256 + pt];
            const float sv = a.table ? a.table[byte] : decode_scale<FMT>(byte, s_T, a.factor);
            scn[it] = v2f_t{sv, sv > 0.0f ? 1.0f / sv : 0.0f};
        }
    };
    auto stash = [&](int it) {   // a quarter
        *reinterpret_cast<float4*>(&Us[(it * 16 + (pt >> 4)) * kB + (pt & 15) * 4]) = tri[it];
        Sc[it * 256 + pt] = scn[it];
    };
    // A operand of a push onto 16 columns: rows 4 ks + q of block b.  (Through a buffer resource: one lane offset for all
    // loads, the rest scalar; sixteen 64-bit addresses would not leave the registers for two factors in flight.)
    const int u_lane = (q * a.K + l16) * 4;
    auto fetch_u = [&](float (&u)[16], int b, int c) {
        const int64_t first = (int64_t)(o + b * kB) * a.K + o, bytes = ((int64_t)a.K * a.K - first) * 4;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Ug + first), 0, (int)(uint32_t)(bytes > 0xffffffffll ? 0xffffffffll : bytes), 0x00020000);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) u[ks] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, u_lane, (ks * 4 * a.K + c) * 4, 0));
    };
    auto push = [&](const float (&u)[16], int c) {   // (a lane owns four neighbouring columns of row l16)
        v4f sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) sum = __builtin_amdgcn_mfma_f32_16x16x4f32(u[ks], ea[ks], sum, 0, 0, 0);
        v4f* dst = reinterpret_cast<v4f*>(&W[l16 * kWStride + c + 4 * q]);
        *dst = *dst - sum;
    };
    fetch_tri(0);
    lds_barrier();
    decode_scales(0);
#pragma unroll
    for (int it = 0; it < 4; ++it) stash(it);
    lds_barrier();
    for (int b = 0; b < blocks; ++b) {
        float un[16];
        if (b + 1 < blocks) {
            fetch_tri(b + 1);
            fetch_u(un, b, (b + 1) * kB + pw * 16);
            if (b > 0) {
                // from the next block on, 16 columns at a time, the next factor on its way under the current product
                float u0[16], u1[16];
                int c = (b + 1) * kB + pw * 16;
                fetch_u(u0, b - 1, c);
                for (; c < width; c += 2 * kB) {
                    const bool second = c + kB < width;
                    if (second) fetch_u(u1, b - 1, c + kB);
                    push(u0, c);
                    if (!second) break;
                    if (c + 2 * kB < width) fetch_u(u0, b - 1, c + 2 * kB);
                    push(u1, c + kB);
                }
            }
            decode_scales(b + 1);
        }
        lds_barrier();
        if (b + 1 < blocks) {
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) ea[ks] = Es[l16 * kEStride + ks * 4 + q];
            // the push onto the next block, its triangle and scales written to LDS under the products
            v4f* dst = reinterpret_cast<v4f*>(&W[l16 * kWStride + (b + 1) * kB + pw * 16 + 4 * q]);
            const v4f old = *dst;
            v4f sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) {
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(un[ks], ea[ks], sum, 0, 0, 0);
                if (ks % 4 == 0) stash(ks / 4);
                __builtin_amdgcn_sched_barrier(0);
            }
            *dst = old - sum;
        }
        lds_barrier();
    }
}

// wp[n, c] -= sum_{j < kOuter} e[n, j] * U[o + j, c] for the columns c_begin <= c < K (visiting order): a dense fp32
// contraction, [N x 512] . [512 x columns], of the pairs of halves that the outer kernel left.  A row's errors have scales of
// their own (rows do not interact), and so have a column's entries of U; 64 terms are added to the accumulator at a time.
// 128 x 128 output tile per workgroup, a 64 x 64 quarter per wave, a stage of 32 terms copied into LDS while the one before is
// multiplied; two workgroups per compute unit.  [6144, 4096] behind its first outer block 95 us (157 with six bf16 products of
// operands that every workgroup split for itself, 308 on the fp32 MFMA), of which wp is 24 at the rate of a large copy; codes that differ from
// a sweep in 64 bits, 32 layers of K = 2048 and 4096: 9616 of 50 million (9830 with the bf16 products).
constexpr int kUpdateStage = 16 * kPairBytes;   // 8 row blocks, then 8 column blocks
constexpr int kUpdateLds = 2 * (kUpdateStage + 1024), kUpdateLdsUnpacked = kUpdateLds + kOuter * 4;   // two stages and their exponents; error factors
//
// PACKED == false: the workspace has no room for the pairs, every workgroup makes its own, 64 terms at a time, from the errors and from U.
// The results are the same bit for bit.
template <bool PACKED>
__global__ __launch_bounds__(256, 2) void gptq_update_kernel(GptqArgs a, int c_begin)
{
    constexpr int T = 128, NT = 4;
    extern __shared__ __attribute__((aligned(1024))) char St[];
    int* const Sc = reinterpret_cast<int*>(St + 2 * kUpdateStage);   // for two groups of 64 terms: exponents of 128 rows, factors of 128 columns
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wr = (wave >> 1) * NT, wc = (wave & 1) * NT;   // first block of rows / columns of the wave's quarter
    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of tiles, which share rows
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7, p = xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3);
    const int tiles = (a.K - c_begin + T - 1) / T;
    const int n0 = p / tiles * T, c0 = c_begin + p % tiles * T;
    PairSums<NT> sums;
    sums.clear();
    auto scale_sums = [&](const int* sc) {
        sums.scale([&](int i) { return sc[(wr + i) * 16 + l16] - kPairRow; }, [&](int j) { return *reinterpret_cast<const v4f*>(sc + 128 + (wc + j) * 16 + 4 * q); });
    };
    if constexpr (PACKED) {
        const int row_blocks = a.Np / 16, col_blocks = a.K / 16;
        // Blocks past the end are the last one again: they only feed outputs that are not stored.
        const uint32_t scale_at = 4u * (uint32_t)(wave < 2 ? min(n0 + wave * 64 + lane, a.Np - 1) : min(c0 + (wave - 2) * 64 + lane, a.K - 1));
        auto issue = [&](int s) {
            const int slot = s & 1;
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(a.e_pairs + pairs_at(s, row_blocks, n0 / 16), 0, min(row_blocks - n0 / 16, 8) * kPairBytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t cols = __builtin_amdgcn_make_buffer_rsrc(a.u_pairs + pairs_at(s, col_blocks, c0 / 16), 0, min(col_blocks - c0 / 16, 8) * kPairBytes, 0x00020000);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = (wave & 1) * 8 + i;   // 1 KB: half a block; two waves for either operand
                char* const dst = St + slot * kUpdateStage + wave * 8192 + i * 1024;
                if (wave < 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (lds_void*)dst, 16, lane * 16, min(c >> 1, row_blocks - 1 - n0 / 16) * kPairBytes + (c & 1) * 1024, 0, 0);
                else __builtin_amdgcn_raw_ptr_buffer_load_lds(cols, (lds_void*)dst, 16, lane * 16, min(c >> 1, col_blocks - 1 - c0 / 16) * kPairBytes + (c & 1) * 1024, 0, 0);
            }
            if (s % 2 == 0) {
                const __amdgpu_buffer_rsrc_t rs = wave < 2 ? __builtin_amdgcn_make_buffer_rsrc(a.e_scales + (int64_t)(s / 2) * a.Np, 0, 4 * a.Np, 0x00020000)
                                                           : __builtin_amdgcn_make_buffer_rsrc(a.u_scales + (int64_t)(s / 2) * a.K, 0, 4 * a.K, 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(Sc + (s / 2 & 1) * 256 + wave * 64), 4, scale_at, 0, 0, 0);
            }
        };
        issue(0);
        for (int s = 0; s < kStages; ++s) {
            wait_vmcnt<0>();
            wait_lgkmcnt0();
            block_barrier();   // stage s has landed, stage s - 1 has been read
            if (s + 1 < kStages) issue(s + 1);
            const char* base = St + (s & 1) * kUpdateStage;
            if (s & 1) {
                sums.multiply<false>(base + wr * kPairBytes, base + (8 + wc) * kPairBytes);
                scale_sums(Sc + (s / 2 & 1) * 256);
            } else {
                sums.multiply<true>(base + wr * kPairBytes, base + (8 + wc) * kPairBytes);
            }
        }
    } else {
        float* const Rp = reinterpret_cast<float*>(St + kUpdateLds);
        const int o = c_begin - kOuter;
        for (int j = tid; j < kOuter; j += 256) Rp[j] = error_factor(1.0f / a.U[(int64_t)(o + j) * a.K + o + j]);
        for (int j0 = 0; j0 < kOuter; j0 += kB) {
            __syncthreads();
            for (int block = wave; block < 16; block += 4) {
                float v[2][8];
                if (block < 8) {
                    const float* src = a.err + (int64_t)min(n0 + block * 16 + l16, a.N - 1) * kOuter + j0 + 8 * q;
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[s][i] = src[32 * s + i];
                } else {
                    factor_rows(a, o, j0, min(c0 + (block - 8) * 16 + l16, a.K - 1), Rp, v);
                }
                const uint32_t e = put_pairs(v, St + block * kPairBytes, kUpdateStage);
                if (lane < 16) Sc[block * 16 + l16] = block < 8 ? (int)e : __float_as_int(pair_column(e));
            }
            __syncthreads();
            sums.multiply<true>(St + wr * kPairBytes, St + (8 + wc) * kPairBytes);
            sums.multiply<false>(St + kUpdateStage + wr * kPairBytes, St + kUpdateStage + (8 + wc) * kPairBytes);
            scale_sums(Sc);
        }
    }
    // a lane holds columns 4 q .. 4 q + 3 of row l16 of every 16 x 16 tile (K is a multiple of 64)
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int row = n0 + (wr + i) * 16 + l16;
        if (row >= a.N) continue;
        float* dst = a.wp + (int64_t)row * a.K + c0 + wc * 16 + 4 * q;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (c0 + (wc + j) * 16 >= a.K) continue;
            v4f* d = reinterpret_cast<v4f*>(dst + 16 * j);
            *d = *d - sums.acc[i][j];
        }
    }
}

// codes[n, kb] = code of column 2 kb | code of column 2 kb + 1 << 4, fetched from their visiting positions: the row goes through LDS,
// a thread packs eight columns (byte reads from memory: 30 us for [6144, 4096], now 10)
__global__ __launch_bounds__(256) void gptq_pack_kernel(GptqArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t qrow[];  // K codes
    const int n = blockIdx.x;
    const uint4* src = reinterpret_cast<const uint4*>(a.q + (int64_t)n * a.K);
    for (int i = threadIdx.x; i < a.K / 16; i += 256) reinterpret_cast<uint4*>(qrow)[i] = src[i];
    __syncthreads();
    uint32_t* dst = reinterpret_cast<uint32_t*>(a.codes + (int64_t)n * (a.K / 2));
    for (int i = threadIdx.x; i < a.K / 8; i += 256) {
        uint32_t packed = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int4 at = reinterpret_cast<const int4*>(a.iperm)[2 * i + h];
            packed |= ((qrow[at.x] & 15u) | (qrow[at.y] & 15u) << 4 | (qrow[at.z] & 15u) << 8 | (qrow[at.w] & 15u) << 12) << (16 * h);
        }
        dst[i] = packed;
    }
}

constexpr size_t kPairsPerIndex = kOuter * 4 + kOuter / kB * 4;   // bytes of a row's (column's) pairs and exponents
inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// working weights, codes and the inverse order, beside the update's operands
inline size_t weights_bytes(int64_t N, int64_t K) { return align256((size_t)N * K * 4) + align256((size_t)N * K) + align256((size_t)K * 4); }

}  // namespace

size_t gptq_workspace_bytes(int64_t N, int64_t K)
{
    // the pairs and exponents of an outer block's errors and of its rows of U
    return weights_bytes(N, K) + ((size_t)(N + 15) / 16 * 16 + (size_t)K) * kPairsPerIndex;
}

size_t gptq_workspace_least(int64_t N, int64_t K) { return weights_bytes(N, K) + align256((size_t)N * kOuter * 4); }   // the errors alone

hipError_t launch_gptq_sweep(const void* w, int64_t N, int64_t K, int b, int fmt, const float* U, const int* perm,
                             const void* scales, const float* s_T, const float* table, float factor, void* codes, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    GptqArgs a{};
    a.w = static_cast<const uint16_t*>(w);
    a.U = U;
    a.perm = perm;
    char* ws = static_cast<char*>(workspace);
    a.wp = reinterpret_cast<float*>(ws);
    ws += align256((size_t)N * K * 4);
    a.q = reinterpret_cast<uint8_t*>(ws);
    ws += align256((size_t)N * K);
    a.iperm = reinterpret_cast<int*>(ws);
    ws += align256((size_t)K * 4);
    a.Np = (int)((N + 15) / 16 * 16);
    // Less room than fp4_workspace_bytes asks for: the update prepares its operands on the spot, with the same results (a sweep of [4096, 4096] 607 -> 783 us, of [1024, 4096] 445 -> 573).
    const bool packed = workspace_bytes >= gptq_workspace_bytes(N, K);
    if (packed) {
        a.e_pairs = ws;
        ws += (size_t)a.Np * kOuter * 4;
        a.u_pairs = ws;
        ws += (size_t)K * kOuter * 4;
        a.e_scales = reinterpret_cast<int*>(ws);
        ws += (size_t)a.Np * (kOuter / kB) * 4;
        a.u_scales = reinterpret_cast<float*>(ws);
    } else {
        a.err = reinterpret_cast<float*>(ws);
    }
    a.scales = static_cast<const uint8_t*>(scales);
    a.s_T = s_T;
    a.table = table;
    a.codes = static_cast<uint8_t*>(codes);
    a.N = (int)N;
    a.K = (int)K;
    a.b = b;
    a.G = fmt == 0 ? 32 : 16;
    const double c = 1.0 / sqrt((double)b);
    a.c_hi = (float)c;
    a.c_lo = (float)(c - (double)a.c_hi);
    a.factor = factor;
    if (K % kB != 0 || N <= 0 || K > 24576) return hipErrorInvalidValue;  // (a row is staged in LDS)

    const size_t row_lds = (size_t)K * 4;
    static LdsAttrOnce raised;
    if (row_lds > 48 * 1024) {
        const hipError_t le = raised.ensure(reinterpret_cast<const void*>(gptq_rotate_gather_kernel), 24576 * 4);
        if (le != hipSuccess) return le;
    }
    hipLaunchKernelGGL(gptq_rotate_gather_kernel, dim3((unsigned)N), dim3(256), row_lds, st, a);
    const unsigned row128 = (unsigned)((N + 127) / 128), row16 = (unsigned)((N + 15) / 16);
    static LdsAttrOnce update_once, unpacked_once;
    if (K > kOuter) {
        const hipError_t le = packed ? update_once.ensure(reinterpret_cast<const void*>(gptq_update_kernel<true>), kUpdateLds)
                                     : unpacked_once.ensure(reinterpret_cast<const void*>(gptq_update_kernel<false>), kUpdateLdsUnpacked);
        if (le != hipSuccess) return le;
    }
    for (int o = 0; o < (int)K; o += kOuter) {
        const int oe = std::min(o + kOuter, (int)K);
        // the outer block itself: every workgroup takes 16 rows through the block's columns, four waves sweeping 64 of them at a
        // time, four pushing their errors onto the rest of the outer block, while others prepare the block's rows of U ...
        const unsigned pack = packed ? (unsigned)((K - oe) / 16) : 0u;
        if (fmt == 0) hipLaunchKernelGGL(gptq_outer_kernel<0>, dim3(row16 + pack), dim3(512), 0, st, a, o, oe, (int)row16);
        else hipLaunchKernelGGL(gptq_outer_kernel<1>, dim3(row16 + pack), dim3(512), 0, st, a, o, oe, (int)row16);
        // ... everything behind the outer block sees all of its errors in one pass
        if (oe == (int)K) break;
        const dim3 tiles(row128 * (unsigned)((K - oe + 127) / 128));
        if (packed) hipLaunchKernelGGL(gptq_update_kernel<true>, tiles, dim3(256), kUpdateLds, st, a, oe);
        else hipLaunchKernelGGL(gptq_update_kernel<false>, tiles, dim3(256), kUpdateLdsUnpacked, st, a, oe);
    }
    hipLaunchKernelGGL(gptq_pack_kernel, dim3((unsigned)N), dim3(256), (size_t)K, st, a);
    return hipGetLastError();
}

}  // namespace fp4mr
