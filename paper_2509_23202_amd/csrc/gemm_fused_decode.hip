// One launch for a handful of tokens (M <= 4; the weight-only form below M <= 16), MXFP4:  out = Q(X H_b) Q(W H_b)^T  with the activations rotated and
// quantized inside the GEMM (arXiv 2509.23202, Section 4.2 items 1 and 2 in one kernel; the appendix on inference regimes
// notes that at small batch the separate kernels give little: here the activation side costs no launch of its own).
//
// Same decomposition as the few-token weight-streaming kernel: a workgroup owns one 16-column block of the output
// (one row-block of W in GEMM layout), its 8 waves split K, W fragments go straight from global memory to registers.
// The activation fragments are not loaded but made: a wave's share of K is walked in chunks of four fragments
// (512 K-elements = 16 vectors of 32), and for every token the 16 vectors of the chunk are one rotation MFMA group
// (vectors consecutive along K in one row, so Hadamard blocks of 64 / 128 finish with butterfly levels across lanes),
// quantized by the same group quantizer as the stand-alone kernels, and scattered through LDS into the lane order of
// the GEMM's B operand.  A token's 512 activations are 1 KB of bf16: less L2 traffic than the 4 x 1 KB of 16-row padded
// code fragments the unfused path reads.  The codes are the stand-alone quantizer's codes, the K split and the order
// of additions are the weight-streaming kernel's: the result is bit-identical to the two-launch path.
#include "device_util.hpp"
#include "internal.hpp"
#include "layout.hpp"
#include "rq_core.hpp"

#include <algorithm>

namespace fp4mr {
namespace {

constexpr int kFusedWaves = 8;
constexpr int kLdsBytes = 160 * 1024;   // of a compute unit

struct FusedArgs {
    const uint16_t* x;       // [M, K] bf16
    const uint8_t* w_codes;  // GEMM layout
    const uint8_t* w_scales;
    void* out;
    int M, N, K, b;
    float c_hi, c_lo;        // 1/sqrt(b) split in two floats
    float alpha;             // factor on the result (4/3 when the weights' scales carry the tensor-level 4/3), else 1
};

// MP = token rows kept in the staging area: rows of the activation fragments beyond them are zero by construction and never
// touch LDS, which keeps the workgroup small enough for four of them per compute unit.
template <bool OUT_F32>
__global__ __launch_bounds__(kFusedWaves * 64) void gemm_fused_decode_kernel(FusedArgs a)
{
    constexpr int MP = 4;   // (the entry point takes M <= 4)
    constexpr int U = 4;    // fragments per chunk = 16 vectors of 32
    constexpr int TOK = 4;  // tokens whose loads are in flight together
    using GQ = GroupQuant<32, 8, 16, true>;

    // staging: entry (vector v of the chunk, token m) at v * MP + m: four code dwords and one scale dword (byte in bits 7:0)
    __shared__ __attribute__((aligned(16))) uint32_t st_codes[kFusedWaves][16 * MP * 4];
    __shared__ __attribute__((aligned(16))) uint32_t st_scales[kFusedWaves][16 * MP];
    __shared__ float partial[kFusedWaves][256];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane & 15, q = lane >> 4;
    const int rb = blockIdx.x;
    const int KC = a.K >> 7, KS = (a.K + 511) >> 9;
    const int per = (KC + kFusedWaves - 1) / kFusedWaves;
    const int k_begin = min(wave * per, KC), k_end = min(k_begin + per, KC);

    v8bf hop[2][1];
    build_hadamard_operand<32>(hop, g, q, a.b < 32 ? a.b : 32);
    const int kron = a.b > 32 ? (a.b == 64 ? 1 : 2) : 0;

    // rows of the staged fragments that belong to no token stay zero for the whole kernel
    uint32_t* const sc_codes = st_codes[wave];
    uint32_t* const sc_scales = st_scales[wave];
    for (int i = lane; i < 16 * MP * 4; i += 64) sc_codes[i] = 0u;
    for (int i = lane; i < 16 * MP; i += 64) sc_scales[i] = 0u;

    const v4i* wfrag = reinterpret_cast<const v4i*>(a.w_codes + (int64_t)rb * KC * 1024) + lane;
    v4f acc = {0.f, 0.f, 0.f, 0.f};

    for (int kc0 = k_begin; kc0 < k_end; kc0 += U) {
        // activations of the chunk: vector g of the chunk starts at element (kc0 * 4 + g) * 32; it exists if its fragment
        // is inside this wave's share of K
        const bool v_ok = kc0 + (g >> 2) < k_end;
        const int64_t k_lane = (int64_t)kc0 * 128 + g * 32 + 8 * q;
        for (int m0 = 0; m0 < a.M; m0 += TOK) {
            v4i xin[TOK];
#pragma unroll
            for (int t = 0; t < TOK; ++t) {
                const v4i z = {0, 0, 0, 0};
                const int m = m0 + t;
                xin[t] = (m < a.M && v_ok) ? *reinterpret_cast<const v4i*>(a.x + (int64_t)m * a.K + k_lane) : z;
            }
#pragma unroll
            for (int t = 0; t < TOK; ++t) {
                const int m = m0 + t;
                if (m >= a.M) break;  // uniform
                v4f h[2];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    h[tt] = v4f{0.f, 0.f, 0.f, 0.f};
                    h[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hop[tt][0], __builtin_bit_cast(v8bf, xin[t]), h[tt], 0, 0, 0);
                }
                kronecker_levels<2>(h, g, kron);
                float y[8];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) y[4 * tt + v] = __fmaf_rn(h[tt][v], a.c_hi, h[tt][v] * a.c_lo);
                uint32_t out[1], sc[1];
                GQ::mx(y, out, sc);
                // lane (g, q) holds elements 8q .. 8q+7 of vector g = K-block g%4 of fragment g/4, row m
                const int pos = g * MP + m;
                sc_codes[pos * 4 + q] = out[0];
                if (q == 0) sc_scales[pos] = sc[0];
            }
        }
        // W fragments and scales of the chunk, asked for only now: holding them across the quantization above would cost the
        // registers that let eight waves per SIMD stay resident, and resident waves are what keeps HBM busy here
        // (the tail repeats the last fragment; its products are skipped below)
        v4i wf[U];
        uint32_t swv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kc = min(kc0 + u, k_end - 1);
            wf[u] = __builtin_nontemporal_load(wfrag + (int64_t)kc * 64);
            const uint32_t d = *(reinterpret_cast<const uint32_t*>(a.w_scales) + ((int64_t)rb * KS + (kc >> 2)) * 64 + lane);
            swv[u] = d >> (8 * (kc & 3));
        }
        // the chunk's activation fragments in B-operand order (same wave wrote them: LDS operations of a wave are in order)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kc0 + u < k_end) {
                // B-operand lane = K-block (lane / 16) of the fragment, row lane % 16
                const int row = lane & 15, pos = (u * 4 + (lane >> 4)) * MP + (row < MP ? row : 0);
                const v4i z = {0, 0, 0, 0};
                const v4i xf = row < MP ? *reinterpret_cast<const v4i*>(sc_codes + pos * 4) : z;
                const uint32_t sx = row < MP ? sc_scales[pos] : 0u;
                const v8i a8 = {wf[u][0], wf[u][1], wf[u][2], wf[u][3], 0, 0, 0, 0};
                const v8i b8 = {xf[0], xf[1], xf[2], xf[3], 0, 0, 0, 0};
                acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, b8, acc, 4, 4, 0, (int)swv[u], 0, (int)sx);
            }
        }
    }

    *reinterpret_cast<v4f*>(&partial[wave][lane * 4]) = acc;
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += kFusedWaves * 64) {
        const int l = e >> 2, v = e & 3;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kFusedWaves; ++w) s += partial[w][e];
        s *= a.alpha;
        const int m = l & 15;
        const int n = rb * 16 + (l >> 4) * 4 + v;
        if (m < a.M && n < a.N) {
            if constexpr (OUT_F32) static_cast<float*>(a.out)[(int64_t)m * a.N + n] = s;
            else static_cast<__bf16*>(a.out)[(int64_t)m * a.N + n] = (__bf16)s;
        }
    }
}


// ------------------------------------------------------------------------------------------------------
// Weight-only variant (W4A16) for a handful of tokens: out = bf16(X H_b) Q(W H_b)^T.  The paper's appendix on
// inference regimes recommends weight-only quantization where the layer is memory-bound: activation quantization
// buys no speed there and costs accuracy.  Same streaming of W, same rotation MFMA group per token and chunk; the
// rotated activations are rounded to bf16 instead of quantized, the E2M1 codes of W are decoded with their E8M0
// scale straight to bf16 (exact: two significant bits, bf16 has the exponent range of the scale) and the product runs
// on the bf16 MFMA, four K = 32 instructions per fragment.  The contraction index inside a fragment is permuted the
// same way for both operands (instruction j takes elements 32*kb + 8*j .. +8 of K-block kb), which a dot product
// does not see.
typedef __bf16 v2bf_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v8bf decode8_bf16(uint32_t codes, float scale)
{
    const v2bf_t p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 0);
    const v2bf_t p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 1);
    const v2bf_t p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 2);
    const v2bf_t p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, 3);
    const v8bf r = {p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
    return r;
}

template <bool OUT_F32, int MP>
__global__ __launch_bounds__(kFusedWaves * 64) void gemm_w4a16_decode_kernel(FusedArgs a)
{
    constexpr int U = 4;    // fragments per chunk = 16 vectors of 32
    constexpr int TOK = 4;  // tokens whose loads are in flight together

    // staging: rotated activations in bf16, entry (vector v of the chunk, token m, part q) = 8 values = 16 bytes
    __shared__ __attribute__((aligned(16))) uint32_t st_y[kFusedWaves][16 * MP * 16];
    __shared__ float partial[kFusedWaves][256];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane & 15, q = lane >> 4;
    const int rb = blockIdx.x;
    const int KC = a.K >> 7, KS = (a.K + 511) >> 9;
    const int per = (KC + kFusedWaves - 1) / kFusedWaves;
    const int k_begin = min(wave * per, KC), k_end = min(k_begin + per, KC);

    v8bf hop[2][1];
    build_hadamard_operand<32>(hop, g, q, a.b < 32 ? a.b : 32);
    const int kron = a.b > 32 ? (a.b == 64 ? 1 : 2) : 0;

    uint32_t* const sy = st_y[wave];
    for (int i = lane; i < 16 * MP * 16; i += 64) sy[i] = 0u;  // rows that belong to no token stay zero

    const v4i* wfrag = reinterpret_cast<const v4i*>(a.w_codes + (int64_t)rb * KC * 1024) + lane;
    v4f acc = {0.f, 0.f, 0.f, 0.f};

    for (int kc0 = k_begin; kc0 < k_end; kc0 += U) {
        const bool v_ok = kc0 + (g >> 2) < k_end;
        const int64_t k_lane = (int64_t)kc0 * 128 + g * 32 + 8 * q;
        for (int m0 = 0; m0 < a.M; m0 += TOK) {
            v4i xin[TOK];
#pragma unroll
            for (int t = 0; t < TOK; ++t) {
                const v4i z = {0, 0, 0, 0};
                const int m = m0 + t;
                xin[t] = (m < a.M && v_ok) ? *reinterpret_cast<const v4i*>(a.x + (int64_t)m * a.K + k_lane) : z;
            }
#pragma unroll
            for (int t = 0; t < TOK; ++t) {
                const int m = m0 + t;
                if (m >= a.M) break;  // uniform
                v4f h[2];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    h[tt] = v4f{0.f, 0.f, 0.f, 0.f};
                    h[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hop[tt][0], __builtin_bit_cast(v8bf, xin[t]), h[tt], 0, 0, 0);
                }
                kronecker_levels<2>(h, g, kron);
                v8bf yb;
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) yb[4 * tt + v] = (__bf16)__fmaf_rn(h[tt][v], a.c_hi, h[tt][v] * a.c_lo);
                // lane (g, q) holds elements 8q .. 8q+7 of vector g, token m
                *reinterpret_cast<v8bf*>(sy + ((g * MP + m) * 4 + q) * 4) = yb;
            }
        }
        // W fragments and scales of the chunk, asked for only now (registers: see the quantizing kernel above)
        v4i wf[U];
        uint32_t swv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kc = min(kc0 + u, k_end - 1);
            wf[u] = __builtin_nontemporal_load(wfrag + (int64_t)kc * 64);
            const uint32_t d = *(reinterpret_cast<const uint32_t*>(a.w_scales) + ((int64_t)rb * KS + (kc >> 2)) * 64 + lane);
            swv[u] = (d >> (8 * (kc & 3))) & 0xffu;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kc0 + u < k_end) {
                const float wscale = __uint_as_float(swv[u] << 23);  // E8M0 byte as the exponent field of a binary32
                const int row = lane & 15, kb = lane >> 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // lane (row n, kb) of W holds elements 32 kb .. +32 of its row: dword j = elements 32 kb + 8 j .. +8
                    const v8bf w8 = decode8_bf16((uint32_t)wf[u][j], wscale);
                    const v8bf z = {(__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f, (__bf16)0.f};
                    // lane (token row, kb) of X: the same elements 32 kb + 8 j .. +8 = part j of vector 4u + kb
                    const v8bf x8 = row < MP ? *reinterpret_cast<const v8bf*>(sy + (((u * 4 + kb) * MP + row) * 4 + j) * 4) : z;
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w8, x8, acc, 0, 0, 0);
                }
            }
        }
    }

    *reinterpret_cast<v4f*>(&partial[wave][lane * 4]) = acc;
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += kFusedWaves * 64) {
        const int l = e >> 2, v = e & 3;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kFusedWaves; ++w) s += partial[w][e];
        s *= a.alpha;
        const int m = l & 15;
        const int n = rb * 16 + (l >> 4) * 4 + v;
        if (m < a.M && n < a.N) {
            if constexpr (OUT_F32) static_cast<float*>(a.out)[(int64_t)m * a.N + n] = s;
            else static_cast<__bf16*>(a.out)[(int64_t)m * a.N + n] = (__bf16)s;
        }
    }
}

// ------------------------------------------------------------------------------------------------------
// The same product with PERSISTENT workgroups, one per compute unit, each walking the row-blocks of W with a stride of the
// grid.  The kernel above rotates the activations again in every workgroup (M = 4, N = 28672, K = 4096: 1792 times, 18.5 us),
// and its W loads wait for that; here they are rotated once per workgroup into LDS (M K bf16, in the order in which a
// fragment's MFMAs read them: [fragment][MFMA j][K-block][token], neighbouring lanes 16 bytes apart), under the first W
// loads, and from then on NBUF - 1 batches of four W fragments per wave are in flight while one is multiplied.  A batch that
// does not exist is requested with zero size, so that every request is unconditional (the compiler's waits count on it).
// Bound: start-up, then HBM.  A request of eight waves costs the compute unit's address path some 0.2 us, also one of zero size, and every copy of a
// step is code to fetch, cold in each launch: so a batch asks for its scales twice instead of four times, and NBUF is as small as the
// loads allow: 1 where a workgroup has a single batch (nothing else is requested), 2 else (3 where launch_few_stream says so).  Against three buffers
// everywhere, us, M = 4, weight-only: N = K = 1024 3.7 -> 3.1, 4096 5.1 -> 4.2, N = 6144, K = 4096 6.6 -> 5.6, N = 28672 13.4 -> 12.7, N = 4096,
// K = 14336 11.9 -> 10.7.  (Four or five buffers: 6 and 10 % slower than three.  A last step without a request: a third copy of the
// step, N = 6144 5.7 -> 6.0.)
// Same K split, same order of additions: bit-identical.
// QUANT: the quantizing product; a fragment in LDS is then 4 M entries [K-block][token] of sixteen code bytes and behind them
// 4 M dwords with the scale byte.
template <bool QUANT, bool OUT_F32, int NBUF>
__global__ __launch_bounds__(kFusedWaves * 64) void gemm_few_stream_kernel(FusedArgs a)
{
    using GQ = GroupQuant<32, 8, 16, true>;
    constexpr int U = 4, TOK = 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float (*const partial)[kFusedWaves][256] = reinterpret_cast<float (*)[kFusedWaves][256]>(smem);   // [2]: alternating

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane & 15, q = lane >> 4;
    const int KC = a.K >> 7, KS = (a.K + 511) >> 9, n_rb = (a.N + 15) >> 4, G = (int)gridDim.x;
    const int per = (KC + kFusedWaves - 1) / kFusedWaves;
    const int k_begin = min(wave * per, KC), k_end = min(k_begin + per, KC);
    const int nb = (per + U - 1) / U;   // batches per row-block, the same for every wave
    const int frag_bytes = a.M * (QUANT ? 80 : 256);
    char* const xs = smem + 2 * sizeof(partial[0]) + wave * per * frag_bytes;

    auto make_rsrc = [](const void* base, int64_t bytes) {
        const uint32_t n = bytes > 0xffffffffll ? 0xffffffffu : (uint32_t)bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)n, 0x00020000);
    };
    struct Batch {
        v4i wf[U];
        uint32_t sw[2];   // a dword holds the scale bytes of four fragments: of those up to a multiple of four, of those behind it
    };
    int rb_ahead = (int)blockIdx.x, batch_ahead = 0;   // the next batch to be requested
    auto request = [&](Batch& b) {
        const int kc0 = k_begin + batch_ahead * U;
        const bool valid = rb_ahead < n_rb && kc0 < k_end;
        const int rb = valid ? rb_ahead : 0;
        const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(a.w_codes + (int64_t)rb * KC * 1024, valid ? (int64_t)KC * 1024 : 0);
        const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(a.w_scales + (int64_t)rb * KS * 256, valid ? (int64_t)KS * 256 : 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kc = max(min(kc0 + u, k_end - 1), 0);   // (the tail repeats the last fragment; its products are skipped)
            b.wf[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_w, lane * 16, kc * 1024, 2));   // streamed once
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            b.sw[h] = __builtin_amdgcn_raw_buffer_load_b32(rs_s, lane * 4, (max(min(kc0 + h * (U - 1), k_end - 1), 0) >> 2) * 256, 0);
        if (++batch_ahead == nb) {
            batch_ahead = 0;
            rb_ahead += G;
        }
    };
    // the wave's share of the activations, rotated, into LDS: four tokens of sixteen 32-element vectors (a batch of fragments)
    // at a time, the next loads under the current rotation (tokens past M read the last one again and are not written).
    v8bf hop[2][1];
    build_hadamard_operand<32>(hop, g, q, a.b < 32 ? a.b : 32);
    const int kron = a.b > 32 ? (a.b == 64 ? 1 : 2) : 0;
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(a.x, (int64_t)a.M * a.K * 2);
    const int groups = (a.M + TOK - 1) / TOK;
    auto load_x = [&](v4i (&x)[TOK], int item) {
        const int c = item / groups, m0 = (item - c * groups) * TOK;
        const int k_lane = (k_begin + c * U) * 256 + g * 64 + q * 16;
#pragma unroll
        for (int t = 0; t < TOK; ++t) x[t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs_x, k_lane, min(m0 + t, a.M - 1) * a.K * 2, 0));
    };
    auto rotate = [&](v4i (&x)[TOK], int item) {
        const int c = item / groups, m0 = (item - c * groups) * TOK;
        const int f = c * U + (g >> 2);   // fragment of the wave's share; its K-block g % 4 is vector g
#pragma unroll 1
        for (int m = m0; m < min(m0 + TOK, a.M); ++m) {   // (not unrolled, the tokens move up instead: less code to fetch)
            v4f h[2];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                h[tt] = v4f{0.f, 0.f, 0.f, 0.f};
                h[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hop[tt][0], __builtin_bit_cast(v8bf, x[0]), h[tt], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t + 1 < TOK; ++t) x[t] = x[t + 1];
            kronecker_levels<2>(h, g, kron);
            float y[8];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int v = 0; v < 4; ++v) y[4 * tt + v] = __fmaf_rn(h[tt][v], a.c_hi, h[tt][v] * a.c_lo);
            if constexpr (QUANT) {
                uint32_t codes[1], sc[1];
                GQ::mx(y, codes, sc);
                char* const dst = xs + f * frag_bytes;
                const int pos = (g & 3) * a.M + m;
                if (k_begin + f < k_end) {
                    *reinterpret_cast<uint32_t*>(dst + pos * 16 + q * 4) = codes[0];
                    if (q == 0) *reinterpret_cast<uint32_t*>(dst + a.M * 64 + pos * 4) = sc[0];
                }
            } else {
                v8bf yb;
#pragma unroll
                for (int i = 0; i < 8; ++i) yb[i] = (__bf16)y[i];
                if (k_begin + f < k_end) *reinterpret_cast<v8bf*>(xs + f * frag_bytes + ((q * 4 + (g & 3)) * a.M + m) * 16) = yb;
            }
        }
    };
    const int items = (k_end - k_begin + U - 1) / U * groups;
    // (the first activations are asked for before W: loads return in order)
    v4i x0[TOK], x1[TOK];
    load_x(x0, 0);
    if (items > 1) load_x(x1, 1);
    Batch buf[NBUF];
    request(buf[0]);
    if constexpr (NBUF == 3) request(buf[1]);
    if (items > 0) rotate(x0, 0);
    for (int item = 1; item < items; item += 2) {
        if (item + 1 < items) load_x(x0, item + 1);
        rotate(x1, item);
        if (item + 1 < items) {
            if (item + 2 < items) load_x(x1, item + 2);
            rotate(x0, item + 1);
        }
    }

    // (columns of the product past M read the last token again and are not stored)
    const int x_pos = q * a.M + min(g, a.M - 1);
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    int rb = (int)blockIdx.x, batch = 0, it = 0;
    // one batch: request the one NBUF - 1 behind it, multiply this one, and behind a row-block's last batch add the eight waves' partial sums in
    // wave order and store; true = that was the last row-block
    auto step = [&](const Batch& cur, Batch& nxt) -> bool {
        if constexpr (NBUF > 1) request(nxt);
        const int kc0 = k_begin + batch * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kc = kc0 + u;
            if (kc < k_end) {
                const char* const xf = xs + (kc - k_begin) * frag_bytes;
                const uint32_t sw = ((kc0 & 3) + u < 4 ? cur.sw[0] : cur.sw[1]) >> (8 * (kc & 3));
                if constexpr (QUANT) {
                    const v4i x = *reinterpret_cast<const v4i*>(xf + x_pos * 16);
                    const uint32_t sx = *reinterpret_cast<const uint32_t*>(xf + a.M * 64 + x_pos * 4);
                    const v8i a8 = {cur.wf[u][0], cur.wf[u][1], cur.wf[u][2], cur.wf[u][3], 0, 0, 0, 0};
                    const v8i b8 = {x[0], x[1], x[2], x[3], 0, 0, 0, 0};
                    acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, b8, acc, 4, 4, 0, (int)sw, 0, (int)sx);
                    continue;
                }
                const float wscale = __uint_as_float((sw & 0xffu) << 23);   // E8M0 byte as a binary32's exponent
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v8bf w8 = decode8_bf16((uint32_t)cur.wf[u][j], wscale);
                    const v8bf x8 = *reinterpret_cast<const v8bf*>(xf + (x_pos + j * 4 * a.M) * 16);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w8, x8, acc, 0, 0, 0);
                }
            }
        }
        if (NBUF > 1 && ++batch < nb) return false;
        batch = 0;
        *reinterpret_cast<v4f*>(&partial[it][wave][lane * 4]) = acc;
        acc = v4f{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the LDS writes have landed
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int e = wave * 32 + (lane & 31), l = e >> 2;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < kFusedWaves; ++w) s += partial[it][w][e];
        s *= a.alpha;
        const int m = l & 15, n = rb * 16 + (l >> 4) * 4 + (e & 3);
        if (lane < 32 && m < a.M && n < a.N) {
            if constexpr (OUT_F32) static_cast<float*>(a.out)[(int64_t)m * a.N + n] = s;
            else static_cast<__bf16*>(a.out)[(int64_t)m * a.N + n] = (__bf16)s;
        }
        it ^= 1;
        rb += G;
        return NBUF == 1 || rb >= n_rb;
    };
    for (;;) {
        if (step(buf[0], buf[NBUF - 1])) break;
        if constexpr (NBUF > 1) { if (step(buf[1], buf[0])) break; }
        if constexpr (NBUF > 2) { if (step(buf[2], buf[1])) break; }
    }
}

// LDS of the persistent kernel: two sets of partial sums and the rotated activations
size_t few_stream_lds(int64_t M, int64_t K, bool quant)
{
    const int64_t per = ((K >> 7) + kFusedWaves - 1) / kFusedWaves;
    return 2 * kFusedWaves * 256 * sizeof(float) + (size_t)(kFusedWaves * per * M * (quant ? 80 : 256));
}

template <bool QUANT, bool OUT_F32, int NBUF>
hipError_t launch_few_stream_as(const FusedArgs& a, int grid, hipStream_t st)
{
    const size_t lds = few_stream_lds(a.M, a.K, QUANT);
    if (lds > 48 * 1024) {   // (what every kernel may have; asking for the device costs the smallest calls 0.1 us of their 4.5)
        static LdsAttrOnce raised;
        const hipError_t e = raised.ensure(reinterpret_cast<const void*>(gemm_few_stream_kernel<QUANT, OUT_F32, NBUF>), kLdsBytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((gemm_few_stream_kernel<QUANT, OUT_F32, NBUF>), dim3((unsigned)grid), dim3(kFusedWaves * 64), lds, st, a);
    return hipGetLastError();
}

template <bool QUANT, bool OUT_F32>
hipError_t launch_few_stream(const FusedArgs& a, hipStream_t st)
{
    const int n_rb = (a.N + 15) / 16, grid = std::min(n_rb, compute_units());
    if (n_rb == grid && a.K <= 4096) return launch_few_stream_as<QUANT, OUT_F32, 1>(a, grid, st);   // (a compute unit each, with one batch)
    if constexpr (QUANT) {
        // (two batches per row-block, both nearly full, and two row-blocks for nearly every workgroup, or more.  Medians over 12909 products of K =
        // 4224 to 8192, two buffers' time over three's: up to 1.75 row-blocks per workgroup on average 0.90 - 0.99 (N = 4400 to 4800, K about 6144, M = 1 /
        // 4: 6.8 / 8.4 us with three, 6.3 / 8.0 with two), from there to two 1.00 up to K = 7168, beyond that 1.01 - 1.02 (N = K = 8192, M = 4: 9.4 us with
        // two, 8.9 with three); more 0.95 - 1.00 up to K = 7168, beyond that 0.97 - 1.00 with one token and 1.01 - 1.03 with more)
        if (a.K > 7168 && a.K <= 8192 && 4 * n_rb > 7 * grid && (a.M > 1 || n_rb <= 2 * grid)) return launch_few_stream_as<QUANT, OUT_F32, 3>(a, grid, st);
    }
    return launch_few_stream_as<QUANT, OUT_F32, 2>(a, grid, st);
}

}  // namespace

hipError_t launch_fused_decode(const void* x, int64_t M, int64_t K, int b, const void* w_codes, const void* w_scales,
                               int64_t N, void* out, bool out_f32, bool weight_only, float alpha, hipStream_t st)
{
    FusedArgs a{};
    a.x = static_cast<const uint16_t*>(x);
    a.w_codes = static_cast<const uint8_t*>(w_codes);
    a.w_scales = static_cast<const uint8_t*>(w_scales);
    a.out = out;
    a.M = (int)M;
    a.N = (int)N;
    a.K = (int)K;
    a.b = b;
    const double c = 1.0 / sqrt((double)b);
    a.c_hi = (float)c;
    a.c_lo = (float)(c - (double)a.c_hi);
    a.alpha = alpha;
    const dim3 grid((unsigned)((N + 15) / 16)), block(kFusedWaves * 64);
    // Persistent workgroups wherever their LDS holds the activations (weight-only: M K <= 73728).  Cold weights, one-shot ->
    // persistent, us, M = 1 / 4 / 16: N = 6144, K = 4096 6.3 / 6.3 / 18.0 -> 5.7 / 5.7 / 9.0; N = 28672 16.2 / 18.2 / 60.5 ->
    // 13.2 / 12.7 / 16.0; N = 4096, K = 14336 10.9 / 13.9 -> 9.4 / 10.7.
    // The quantizing product, M = 1 / 4: N = K = 1024 3.1 / 3.9 -> 2.6 / 3.5, 4096 4.2 / 5.0 -> 3.8 / 3.9, N = 6144, K = 4096 5.4 / 5.9 -> 4.8 / 5.0,
    // N = 28672 13.0 / 16.2 -> 11.4 / 11.7, N = K = 8192 8.7 / 9.6 -> 8.1 / 8.9, N = 4096, K = 14336 9.3 / 12.2 -> 8.9 / 11.2.
    const bool fits = few_stream_lds(M, K, !weight_only) <= (size_t)kLdsBytes;
    if (weight_only && fits) return out_f32 ? launch_few_stream<false, true>(a, st) : launch_few_stream<false, false>(a, st);
    if (!weight_only && fits)
        return out_f32 ? launch_few_stream<true, true>(a, st) : launch_few_stream<true, false>(a, st);
    if (weight_only) {
        if (M <= 4) {
            if (out_f32) hipLaunchKernelGGL((gemm_w4a16_decode_kernel<true, 4>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((gemm_w4a16_decode_kernel<false, 4>), grid, block, 0, st, a);
        } else {
            if (out_f32) hipLaunchKernelGGL((gemm_w4a16_decode_kernel<true, 16>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((gemm_w4a16_decode_kernel<false, 16>), grid, block, 0, st, a);
        }
    } else {
        if (out_f32) hipLaunchKernelGGL(gemm_fused_decode_kernel<true>, grid, block, 0, st, a);
        else hipLaunchKernelGGL(gemm_fused_decode_kernel<false>, grid, block, 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace fp4mr
