// NVFP4 W4A4 GEMM for 33 tokens and more, both operands dequantized by every wave for itself (arXiv 2509.23202, Section 2 "The NVFP4
// Format", Section 4.1 "Ingredient 1").
//
//   out[m,n] = sT_a * sT_w * sum_k (sa[m,k/16] * a[m,k]) * (sw[n,k/16] * w[n,k])
//
// on the fp16 MFMA over exactly dequantized operands, as in gemm_nv16.hip.  That kernel converts X in a launch of its own and moves two
// bytes for every value of it; here both operands travel as codes (4.5 bits a value) into LDS, and a wave converts its rows of X and of W
// under its own MFMAs.  No pass in front, no fp16 copy, no second launch for partial sums: the waves of a workgroup split K among
// themselves and add their sums through LDS, in a fixed order, so that few tiles and a long K fill the chip as well.
//
// Bound: a SIMD issues an MFMA 16x16x32 in 8 clocks and a vector instruction in 4 through one port, whichever of its waves they come from (two
// waves, 32 MFMAs with 64 / 96 / 128 vector instructions each: 1077 / 1344 / 1622 clocks for both).  A 64 x 64 tile over 64 of K is 32 MFMAs and 140
// vector instructions: 128 of them convert two values each, or multiply them by their scale, 8 decode a scale.  816 clocks, where the matrix pipe alone would take 512; 128 tokens by 64
// columns: 1360 and 1024.  So tiles are as large as the grid lets them be, both scales come from one conversion each, and two waves share a SIMD.
// What it takes against the kernel for many tokens and the few-token kernels, each by its own rules, cold weights, us: N = K = 4096, M = 128 / 192 / 512 / 1024 11.9 / 20.5 / 32.3 / 42.9
// -> 9.5 / 11.2 / 21.2 / 36.7; N = 6144, K = 4096, M = 192 29.5 -> 16.4; N = 28672, K = 4096, M = 96 42.8 -> 29.3; N = K = 8192, M = 64 / 128 / 768 19.4 / 36.8 / 111 -> 14.8 / 20.6 / 92; N = 4096,
// K = 14336, M = 192 35.3 -> 27.8; N = 57344, K = 8192, M = 96 / 512 124 / 418 -> 98 / 377; N = 2048, K = 2048, M = 768 23.9 -> 10.7; N = 1280, K = 1024, M = 320 14.8 -> 5.2.
// (v_mfma_f32_32x32x16_f16, half the MFMAs and half the LDS reads: level, for it takes the port as long as two of the others.  X converted once per workgroup and
// shared as fp16 through LDS: fewer vector instructions, but a barrier per 32 of K; level with the kernel for many tokens on large layers, 2 to 4 times as long on small ones.  X
// read three blocks ahead instead of two, multiplications two conversions behind, copies and the wait for them behind a stage's first products: level or slower.)
#include "device_util.hpp"
#include "internal.hpp"
#include "layout.hpp"

#include <algorithm>
#include <type_traits>

namespace fp4mr {
namespace {

struct NvCodesArgs {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* w_codes;
    const uint8_t* w_scales;
    const float* a_ts;
    const float* w_ts;
    void* out;
    int M, N, K;
    int sets;      // of 16 TM tokens
};

__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ v4f mfma_f16(v8h a, v8h b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v2h scale_f16(uint32_t e4m3) { return __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(e4m3, 1.0f, false); }
// 16 bytes a lane, straight into LDS, lane l's at base + 16 l
__device__ __forceinline__ void copy16(__amdgpu_buffer_rsrc_t rs, char* base, uint32_t lane_at, int at)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)base, 16, lane_at, at, 0, 0);
}
__device__ __forceinline__ void copy16(const uint8_t* src, char* base)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (lds_void*)base, 16, 0, 0);
}

// A workgroup is KW groups of NWN waves.  A group takes its share of K; its waves have 16 TM tokens in common and 16 TN columns each.
//
// A stage is 64 of K of one group: codes of X and of its waves' W, then per wave the scales of X and of its W.
template <int TM, int TN, int NWN>
constexpr int codes_stage() { return (TM + NWN * TN) * 512 + NWN * (TM + TN) * 64; }
template <int TM, int TN, int NWN, int KW>
constexpr int codes_stages()
{
    const int room = (NWN * KW >= 8 ? 160 : 80) * 1024;
    return std::min(6, room / (codes_stage<TM, TN, NWN>() * KW));
}
// a 16 x 16 block of sums in LDS, its four groups of sixteen lanes 272 bytes apart
constexpr int kSumBlock = 4 * 272;

// The waves of a group copy its stages straight into LDS, X between them, W each its own; S stages are a ring.  With one wave to a group nobody waits for anybody
// until the end.  An MFMA operand's lane (r, q) holds of row r of a 16-row block the group of sixteen q of the stage's four -- one scale -- and two MFMAs (s = 0, 1) take eight elements each.
template <int TM, int TN, int NWN, int KW, bool OUT_F32>
__global__ __launch_bounds__(NWN * KW * 64, 2) void gemm_nv_codes_kernel(NvCodesArgs g)
{
    constexpr int NW = NWN * KW, S = codes_stages<TM, TN, NWN, KW>(), STAGE = codes_stage<TM, TN, NWN>();
    constexpr int XI = (TM + 1) / 2, XW = (XI + NWN - 1) / NWN, WI = (TN + 1) / 2, OPS = XW + WI + 1;   // copies of a wave per stage
    constexpr int W_AT = TM * 512, SC_AT = (TM + NWN * TN) * 512, SC = (TM + TN) * 64;
    static_assert(S >= 3, "a stage is read, one has landed, one is filled");
    static_assert(TN % 2 == 0, "W is copied in pairs of row-blocks");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), wn = wave % NWN, wk = wave / NWN;

    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of tiles, those of the same columns behind each other
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7;
    const int id = xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3);
    const int set = id % g.sets, tn = id / g.sets;
    const int KH = g.K >> 6, KC = g.K >> 7;
    const int a_rbs = (g.M + 15) >> 4, w_rbs = (g.N + 15) >> 4;
    const int a_rb0 = min(set * TM, a_rbs - 1), w_rb0 = min((tn * NWN + wn) * TN, w_rbs - 1);
    const int a_last = a_rbs - 1 - a_rb0, w_last = w_rbs - 1 - w_rb0;
    // the group's share of K: whole fragments of 128
    const int share = (KC + KW - 1) / KW * 2;
    const int k_begin = min(wk * share, KH), KT = min(share, KH - k_begin);

    auto make_rsrc = [](const uint8_t* base, int64_t bytes) {
        const uint32_t b = bytes > 0xffffffffll ? 0xffffffffu : (uint32_t)bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, (int)b, 0x00020000);
    };
    const int c_rb = KC * 1024, s_rb = KC * 128;   // bytes of a row-block
    const __amdgpu_buffer_rsrc_t rs_xc = make_rsrc(g.a_codes + (int64_t)a_rb0 * c_rb, (int64_t)(a_rbs - a_rb0) * c_rb);
    const __amdgpu_buffer_rsrc_t rs_wc = make_rsrc(g.w_codes + (int64_t)w_rb0 * c_rb, (int64_t)(w_rbs - w_rb0) * c_rb);
    // A copy takes half a fragment (64 of K) of two row-blocks.  Row-blocks that do not exist are the last one again.
    int x_pair[XW];
    uint32_t xc_off[XW], wc_off[WI];
#pragma unroll
    for (int i = 0; i < XW; ++i) {
        x_pair[i] = min(wn + i * NWN, XI - 1);
        xc_off[i] = (uint32_t)((lane & 31) * 16 + min(min(2 * x_pair[i] + (lane >> 5), TM - 1), a_last) * c_rb);
    }
#pragma unroll
    for (int i = 0; i < WI; ++i) wc_off[i] = (uint32_t)((lane & 31) * 16 + min(2 * i + (lane >> 5), w_last) * c_rb);
    const int srb = lane >> 2;   // scales: four lanes a row-block
    const uint8_t* const s_src = (srb < TM ? g.a_scales + (int64_t)(a_rb0 + min(srb, a_last)) * s_rb
                                           : g.w_scales + (int64_t)(w_rb0 + min(min(srb - TM, TN - 1), w_last)) * s_rb) + (lane & 3) * 16;

    char* const ring = smem + wk * (S * STAGE);
    auto issue = [&](int k) {
        const int kk = min(k_begin + min(k, KT - 1), KH - 1);
        char* base = ring + (k % S) * STAGE;
#pragma unroll
        for (int i = 0; i < XW; ++i) {
            if (TM % 2 == 0) copy16(rs_xc, base + x_pair[i] * 1024, xc_off[i], kk * 512);
            else if (lane < (x_pair[i] == XI - 1 ? 32 : 64)) copy16(rs_xc, base + x_pair[i] * 1024, xc_off[i], kk * 512);
        }
#pragma unroll
        for (int i = 0; i < WI; ++i) copy16(rs_wc, base + W_AT + (wn * TN + 2 * i) * 512, wc_off[i], kk * 512);
        if (lane < 4 * (TM + TN)) copy16(s_src + kk * 64, base + SC_AT + wn * SC);
    };

    const int code_off = ((q >> 1) * 16 + r) * 16 + (q & 1) * 8, scale_off = SC_AT + wn * SC + ((q >> 1) * 16 + r) * 2 + (q & 1);
    struct Raw {
        v2i codes;
        uint32_t scale;   // (the low byte)
    };
    struct Half {
        v2h h[8];
    };
    auto read_x = [&](const char* base, int f) {
        Raw x;
        x.codes = *reinterpret_cast<const v2i*>(base + f * 512 + code_off);
        x.scale = *reinterpret_cast<const uint8_t*>(base + f * 64 + scale_off);
        return x;
    };
    auto read_w = [&](const char* base, int f) {
        Raw x;
        x.codes = *reinterpret_cast<const v2i*>(base + W_AT + (wn * TN + f) * 512 + code_off);
        x.scale = *reinterpret_cast<const uint8_t*>(base + (TM + f) * 64 + scale_off);
        return x;
    };
    auto scale2 = [&](const Raw& x) {
        const v2h s = scale_f16(x.scale);
        return v2h{s[0], s[0]};
    };
    auto micro = [&](const Raw& x, v2h s2, Half& o, int u) {
        const uint32_t c = (uint32_t)x.codes[u >> 2];
        v2h p;
        switch (u & 3) {
            case 0: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 0); break;
            case 1: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 1); break;
            case 2: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 2); break;
            default: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 3); break;
        }
        o.h[u] = p * s2;
    };
    auto operand = [&](const Half& x, int s) {
        return v8h{x.h[4 * s][0], x.h[4 * s][1], x.h[4 * s + 1][0], x.h[4 * s + 1][1], x.h[4 * s + 2][0], x.h[4 * s + 2][1], x.h[4 * s + 3][0], x.h[4 * s + 3][1]};
    };

    const float ts = (*g.a_ts) * (*g.w_ts);
    v4f acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int s = 0; s < S - 1; ++s) issue(s);
    wait_vmcnt<(S - 2) * OPS>();
    if (NWN > 1) block_barrier();
    asm volatile("" ::: "memory");
    Raw wr[TN], xr[2];          // (xr[t & 1]: block t + 1 of X while block t is multiplied)
    Half w[TN], w2[TN], x;
#pragma unroll
    for (int i = 0; i < TN; ++i) wr[i] = read_w(ring, i);
    xr[1] = read_x(ring, 0);
    xr[0] = read_x(ring, 1);
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const v2h s2 = scale2(wr[i]);
#pragma unroll
        for (int u = 0; u < 8; ++u) micro(wr[i], s2, w[i], u);
    }
    {
        const v2h s2 = scale2(xr[1]);
#pragma unroll
        for (int u = 0; u < 8; ++u) micro(xr[1], s2, x, u);
    }
    // One stage.  w and x are W and the first block of X of stage k; wnext and x take the next one's.
    auto step = [&](int k, Half (&w)[TN], Half (&wnext)[TN], auto odd) {
        constexpr int O = decltype(odd)::value;   // (the ring of two X blocks is indexed by TM k + t)
        const char* const here = ring + (k % S) * STAGE;
        const char* const next = ring + ((k + 1) % S) * STAGE;
        // stage k + 1 has landed, everything of stage k - 1 has been read: its slot is refilled
        wait_vmcnt<(S - 3) * OPS>();
        if (NWN > 1) block_barrier();
        asm volatile("" ::: "memory");
        issue(k + S - 1);
        if (k >= KT) return;   // (a group with a shorter share)
#pragma unroll
        for (int i = 0; i < TN; ++i) wr[i] = read_w(next, i);
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            // while block t is multiplied: block t + 1 (or the next stage's first) and a share of the next W are converted
            const Raw cx = xr[(t + O) & 1];
            if (t + 2 < TM) xr[(t + 1 + O) & 1] = read_x(here, t + 2);
            else xr[(t + 1 + O) & 1] = read_x(next, t + 2 - TM);
            sched_fence();
            constexpr int NM = 2 * TN, W8 = TN * 8;
            const int w0 = t * W8 / TM, w1 = (t + 1) * W8 / TM, tot = 8 + w1 - w0;
            const v2h sx = scale2(cx);
            v2h sw{0, 0};
            Half xn;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int i = m % TN, s = m / TN;
                acc[i][t] = mfma_f16(operand(w[i], s), operand(x, s), acc[i][t]);
#pragma unroll
                for (int u = m * tot / NM; u < (m + 1) * tot / NM; ++u) {
                    // W behind X
                    if (u < 8) micro(cx, sx, xn, u);
                    else {
                        const int c = w0 + u - 8;
                        if (u == 8 || c % 8 == 0) sw = scale2(wr[c / 8]);
                        micro(wr[c / 8], sw, wnext[c / 8], c % 8);
                    }
                }
                sched_fence();
            }
            x = xn;
        }
    };
    for (int k = 0; k < share; k += 2) {
        step(k, w, w2, std::integral_constant<int, 0>{});
        step(k + 1, w2, w, std::integral_constant<int, TM & 1>{});
    }
    wait_vmcnt<0>();
    // sums of JP token blocks at a time through LDS
    constexpr int QUADS = NWN * TN * 4, JP = std::min(TM, S * STAGE * KW / (NW * TN * kSumBlock)), GROUP = NWN * JP * TN * kSumBlock;
    static_assert(JP >= 1, "a row of blocks of all waves' sums fits");
#pragma unroll
    for (int j0 = 0; j0 < TM; j0 += JP) {
        __syncthreads();
        char* const mine = smem + wk * GROUP + r * 16 + q * 272;
#pragma unroll
        for (int j = j0; j < j0 + JP && j < TM; ++j)
#pragma unroll
            for (int i = 0; i < TN; ++i) *reinterpret_cast<v4f*>(mine + ((j - j0) * (NWN * TN) + wn * TN + i) * kSumBlock) = acc[i][j];
        __syncthreads();
        const int rows = 16 * (JP < TM - j0 ? JP : TM - j0);
        for (int e = threadIdx.x; e < rows * QUADS; e += NW * 64) {
            const int c = e % QUADS, row = e / QUADS;
            const char* p = smem + ((row >> 4) * (NWN * TN) + (c >> 2)) * kSumBlock + (c & 3) * 272 + (row & 15) * 16;
            v4f s = *reinterpret_cast<const v4f*>(p);
#pragma unroll
            for (int v = 1; v < KW; ++v) s += *reinterpret_cast<const v4f*>(p + v * GROUP);
            s *= ts;
            const int m = (set * TM + j0) * 16 + row, col = tn * (NWN * TN * 16) + c * 4;
            if (m >= g.M || col >= g.N) continue;
            const int64_t at = (int64_t)m * g.N + col;
            if ((g.N & 3) == 0) {
                typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
                if constexpr (OUT_F32) *reinterpret_cast<v4f*>(static_cast<float*>(g.out) + at) = s;
                else *reinterpret_cast<v4bf*>(static_cast<__bf16*>(g.out) + at) = __builtin_convertvector(s, v4bf);
            } else {
                for (int v = 0; v < 4; ++v)
                    if (col + v < g.N) {
                        if constexpr (OUT_F32) static_cast<float*>(g.out)[at + v] = s[v];
                        else static_cast<__bf16*>(g.out)[at + v] = (__bf16)s[v];
                    }
            }
        }
    }
}

template <int TM, int TN, int NWN, int KW, bool OUT_F32>
hipError_t launch_codes(const NvCodesArgs& g, hipStream_t st)
{
    constexpr int lds = codes_stages<TM, TN, NWN, KW>() * codes_stage<TM, TN, NWN>() * KW;
    static LdsAttrOnce once;
    auto k = gemm_nv_codes_kernel<TM, TN, NWN, KW, OUT_F32>;
    const hipError_t e = once.ensure(reinterpret_cast<const void*>(k), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)(g.sets * ((g.N + 16 * TN * NWN - 1) / (16 * TN * NWN)))), dim3(NWN * KW * 64), lds, st, g);
    return hipGetLastError();
}

// What a launch of one of the tiles takes, microseconds: `once`, and tile_rounds_us of its workgroups, their steps (of 64) two thirds those of the
// longest share of K and one third the mean's.  Fitted to 25 000 launches of 5053 products on two cards (M = 33 ... 4096, N = 256 ... 57344, K = 256 ... 28672, half of them multiples of 256, whose
// launches are whole rounds more often than others), five of the tiles each: the median error is 2 %, one in ten is off by more than 5 to 8 %.
struct CodesTile {
    int tm, tn, nwn, kw;
    double once;
    TileRounds rounds;
};
constexpr CodesTile kCodesTiles[] = {
    {2, 2, 1, 8, 0.000, {1, 2.212, 0.472, 3.913, 0.457, 0.075}},
    {2, 4, 1, 8, 0.000, {1, 3.231, 0.658, 4.261, 0.625, 0.135}},
    {4, 4, 1, 8, 0.000, {1, 3.426, 1.020, 4.766, 0.827, 0.217}},
    {3, 4, 1, 4, 3.866, {2, 2.879, 0.783, 0.000, 0.469, 0.073, 1.288, 0.768, 0.128}},
    {4, 4, 1, 4, 4.086, {2, 3.070, 0.907, 0.000, 0.507, 0.131, 1.458, 0.875, 0.140}},
    {5, 4, 1, 4, 4.522, {2, 3.326, 1.097, 0.000, 0.589, 0.130, 1.663, 1.038, 0.166}},
    {6, 4, 1, 4, 4.925, {2, 3.672, 1.251, 0.000, 0.632, 0.179, 1.711, 1.193, 0.191}},
    {7, 4, 2, 2, 6.108, {2, 4.706, 1.440, 0.000, 0.742, 0.216, 2.543, 1.339, 0.206}},
    {8, 4, 2, 2, 6.761, {2, 4.906, 1.625, 0.000, 0.795, 0.225, 2.328, 1.496, 0.305}},
};

// the cheapest of them and its price
double codes_us(int64_t M, int64_t N, int64_t K, int cus, int* tile)
{
    double best = __builtin_inf();
    for (int i = 0; i < (int)(sizeof(kCodesTiles) / sizeof(kCodesTiles[0])); ++i) {
        const CodesTile& c = kCodesTiles[i];
        const double wgs = (double)((M + 16 * c.tm - 1) / (16 * c.tm)) * (double)((N + 16 * c.tn * c.nwn - 1) / (16 * c.tn * c.nwn));
        const double shares = (double)(K >> 7) / c.kw, steps = (4.0 * (double)(((K >> 7) + c.kw - 1) / c.kw) + 2.0 * shares) / 3.0;
        const double us = c.once + tile_rounds_us(c.rounds, wgs, steps, cus);
        if (us < best) {
            best = us;
            *tile = i;
        }
    }
    return best;
}

}  // namespace

// Which NVFP4 products this kernel takes: those of more than 32 tokens that it is estimated to do in 0.98 of what the kernel for many tokens takes, in 0.95 of what the few-token kernels do (where it is estimated at
// 0.92 to 0.95 of them it took 0.98 on average, at 0.95 to 0.97 0.995), or in 0.90 where there are more than 5e7 outputs, whose stores put the estimates off by 8 % (with 0.97 there 4 products more were
// slower, 20 % the worst).  Of 5053 products timed both ways (as above, M N K up to 4e11) it takes 3737; all of them together take 0.796 of the time that the others alone do (0.793 if every one went the faster
// way), and 16 are more than 3 % slower for it, 6 % the worst.  (With last rounds that are whole priced like those in front of them, 0.92 for all, and never beyond M N K = 1.5e11: 0.800 and 59, 15 % the worst.
// M = 1024, N = 8192, K = 8192 and 14336 118 and 205 us, with this kernel 126 and 221; M = 512, N = 16384, K = 8192 120 and 130; M = 192, N = 57344, K = 5120 107 and 118.)
// Up to 32 tokens there is nothing to gain: 194 products, 0.999 if every one went the faster way.  33 to 64 tokens where those kernels have no price (N > 12288, K > 8192, K <= 1024) stay with them.
int plan_nv_codes(int64_t M, int64_t N, int64_t K, double other, bool few)
{
    if (M <= 32 || other == 0.0) return -1;
    int tile = -1;
    return codes_us(M, N, K, compute_units(), &tile) < (M * N > 50000000 ? 0.90 : few ? 0.95 : 0.98) * other ? tile : -1;
}

hipError_t launch_gemm_nv_codes(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes, const void* w_scales, const float* w_ts,
                                int64_t M, int64_t N, int64_t K, void* out, bool out_f32, int tile, hipStream_t st)
{
    NvCodesArgs g{};
    g.a_codes = static_cast<const uint8_t*>(a_codes);
    g.a_scales = static_cast<const uint8_t*>(a_scales);
    g.w_codes = static_cast<const uint8_t*>(w_codes);
    g.w_scales = static_cast<const uint8_t*>(w_scales);
    g.a_ts = a_ts;
    g.w_ts = w_ts;
    g.out = out;
    g.M = (int)M;
    g.N = (int)N;
    g.K = (int)K;
    const CodesTile& c = kCodesTiles[tile];
    g.sets = (int)((M + 16 * c.tm - 1) / (16 * c.tm));
    switch (tile) {
        case 0: return out_f32 ? launch_codes<2, 2, 1, 8, true>(g, st) : launch_codes<2, 2, 1, 8, false>(g, st);
        case 1: return out_f32 ? launch_codes<2, 4, 1, 8, true>(g, st) : launch_codes<2, 4, 1, 8, false>(g, st);
        case 2: return out_f32 ? launch_codes<4, 4, 1, 8, true>(g, st) : launch_codes<4, 4, 1, 8, false>(g, st);
        case 3: return out_f32 ? launch_codes<3, 4, 1, 4, true>(g, st) : launch_codes<3, 4, 1, 4, false>(g, st);
        case 4: return out_f32 ? launch_codes<4, 4, 1, 4, true>(g, st) : launch_codes<4, 4, 1, 4, false>(g, st);
        case 5: return out_f32 ? launch_codes<5, 4, 1, 4, true>(g, st) : launch_codes<5, 4, 1, 4, false>(g, st);
        case 6: return out_f32 ? launch_codes<6, 4, 1, 4, true>(g, st) : launch_codes<6, 4, 1, 4, false>(g, st);
        case 7: return out_f32 ? launch_codes<7, 4, 2, 2, true>(g, st) : launch_codes<7, 4, 2, 2, false>(g, st);
        case 8: return out_f32 ? launch_codes<8, 4, 2, 2, true>(g, st) : launch_codes<8, 4, 2, 2, false>(g, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fp4mr
