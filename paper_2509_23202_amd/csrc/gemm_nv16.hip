// NVFP4 W4A4 GEMM for many tokens (arXiv 2509.23202, Section 2 "The NVFP4 Format", Section 4.1 "Ingredient 1":
// Xhat = s_T * s_G * Q(.), groups of 16 with E4M3 scales plus one fp32 tensor scale per operand).
//
//   out[m,n] = sT_a * sT_w * sum_k (sa[m,k/16] * a[m,k]) * (sw[n,k/16] * w[n,k])
//
// E4M3 scales on 16-element groups cannot go through CDNA4's block-scaled MFMA (one power-of-two scale per 32
// elements), so the product runs on the fp16 MFMA (v_mfma_f32_16x16x32_f16) over exactly dequantized operands: an E2M1
// value times an E4M3 value has at most 6 significant bits and lies in [2^-10, 2688].  What bounds such a kernel is the
// vector-ALU work of the dequantization, which grows with (tile rows + tile columns) while the MFMAs grow with their
// product.  Two things keep it below the MFMA time here:
//   * the activations are dequantized ONCE, by a pre-pass that writes them as fp16 in the MFMA's operand order into the
//     caller's workspace (2 bytes per element; every tile column of the product re-reads them from L2 instead of
//     re-converting them);
//   * only W is converted inside the product, and a wave's tile is 128 rows of X by 64 (or 32) rows of W: four (two)
//     half-fragment conversions per 64 (32) MFMAs.
// A last row of tiles with at most 64 tokens copies and multiplies four of the eight row-blocks: 0.62 of a tile's time
// (N = 28672, K = 4096, M = 192: 58 -> 48 us; N = 57344, K = 8192, M = 320 with the launch that suits it 282 -> 247 with one W
// again and again, 302 -> 265 on another card with three in turn).
// Block tile 128 x 256 (or 128 x 128 for a remainder of the tile grid, or 128 x 512), four (eight) waves side by side along
// N, K-step 64, three-stage LDS ring fed by direct-to-LDS loads, one barrier per K-step.  75 KB of LDS and 256 registers per
// wave: two workgroups share a compute unit (or one of eight waves fills it).
// What bounds it (timing builds of N = 57344, K = 8192, M = 2048): the MFMAs alone, on real operands, take 1054 us of 1350; the
// copies into LDS cost 200, the conversions of W 65, the reads of X 55, the barrier nothing measurable.
//
// Operand order of one K-step of 64 (16 rows): the MFMA takes 8 halves per lane and call (lane = row r + 16 q); lane (r, q)
// owns the 16 elements k = 16 q .. 16 q + 15 -- exactly one NVFP4 group, one E4M3 scale -- and two MFMAs (s = 0, 1) consume
// its elements 8 s .. 8 s + 7; X and W use the same assignment, which a dot product does not see.
//   X (fp16, workspace): [row-block][K-step][plane s][lane][16 bytes]
//   W (codes, GEMM layout): the K-step is half a fragment, 512 contiguous bytes; lane (r, q) reads 8 bytes.
#include "device_util.hpp"
#include "internal.hpp"
#include "layout.hpp"
#include "nv_dequant.hpp"

#include <algorithm>
#include <type_traits>

namespace fp4mr {
namespace {

struct Nv16Args {
    const uint8_t* x16;
    const uint8_t* w_codes;
    const uint8_t* w_scales;
    const float* a_ts;
    const float* w_ts;
    void* out;
    int64_t M, N, K;
    int tiles_m;
    int half_row;  // 1: the last row of tiles holds at most 64 tokens, its tiles come last
    int n_first;   // first output column of this launch (a multiple of 256)
    int n_cols;    // number of output columns this launch covers (to the end of N when the tile grid is ragged)
    // split-K launches: parts along K of a whole tile and of one of the last row's, K-steps of 64 in a part (even), where the partials of either begin
    int parts[2], steps[2];
    float* partial[2];
};

// ---------------------------------------------------------------------------------------------------------------
// Pre-pass: NVFP4 activations (GEMM layout) -> exact fp16 values code * s_G in the operand order above.  One wave per
// fragment (16 rows x 128 K): 1 KB of codes and 128 scale bytes in, two K-steps of 2 KB out.
__global__ __launch_bounds__(256) void nv_x16_kernel(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                                     uint8_t* __restrict__ x16, int64_t n_frags)
{
    const int lane = threadIdx.x & 63;
    const int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (f >= n_frags) return;
    const v4i c = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(codes + f * 1024) + lane);
    const uint32_t sc = *(reinterpret_cast<const uint16_t*>(scales + f * 128) + lane);
    const NvFrag16 v = nv_dequant_frag(c, sc);
    // lane (r, Q) holds k = 32 Q .. 32 Q + 31 of the fragment: K-step Q / 2, lanes q = 2 (Q % 2) + t of that step for its
    // elements 16 t .. 16 t + 15, plane s for elements 8 s .. 8 s + 7 of those
    const int r = lane & 15, Q = lane >> 4;
    uint8_t* dst = x16 + (f * 2 + (Q >> 1)) * 2048;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s)
            *reinterpret_cast<v8h*>(dst + s * 1024 + ((2 * (Q & 1) + t) * 16 + r) * 16) = v.s[2 * t + s];
}

// ---------------------------------------------------------------------------------------------------------------
// SPLITK: tiles in several parts along K.  The workgroup multiplies the K-steps of its part only and writes its fp32 partial tile, without the
// tensor scales, to its slice of the partials; nv16_reduce_kernel adds the slices in the parts' order, four neighbouring values a thread.
// (M = 320, layers of 8192 features with N = 10240, 8192, 57344 and K = 28672: 591 -> 553 us with parts that suit half tiles, half tiles' copies and that
// reduction, quantizers included.)
template <int NW, int TN, bool OUT_F32, int STAGES, bool SPLITK = false>
__global__ __launch_bounds__(NW * 64, 2) void gemm_nv16_kernel(Nv16Args g)
{
    static_assert(!SPLITK || OUT_F32, "split-K workgroups write fp32 partials");
    constexpr int BM = 128, WN = 16 * TN, BN = NW * WN;   // 64 or 32 columns per wave
    constexpr int TM = BM / 16;
    constexpr int FX = BM / 16, FW = BN / 16;
    constexpr int WS_SLOT = 256;           // scale bytes one full-wave copy writes: four row-blocks' worth per wave
    constexpr int X_BYTES = FX * 2048, WC_BYTES = FW * 512, WS_BYTES = NW * WS_SLOT;
    constexpr int STAGE_BYTES = X_BYTES + WC_BYTES + WS_BYTES;
    constexpr int WPW = FW / NW;                          // W half-fragments a wave copies per stage
    constexpr int WCI = WPW / 2;                          // W code instructions per wave and stage
    static_assert(FX % NW == 0 && FW % NW == 0, "the copies are dealt evenly to the waves");

    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // consecutive workgroups share a W column band; the tiles of a last row of at most 64 tokens, which are shorter, come behind all others
    const int whole = g.tiles_m - g.half_row, tiles_n = (g.n_cols + BN - 1) / BN, whole_tiles = tiles_n * whole;
    const int all_whole = whole_tiles * (SPLITK ? g.parts[0] : 1);
    const bool half = (int)blockIdx.x >= all_whole;
    int id = half ? (int)blockIdx.x - all_whole : (int)blockIdx.x, part = 0;
    if constexpr (SPLITK) {   // part by part
        const int n = half ? tiles_n : whole_tiles;
        part = id / n;
        id -= part * n;
    }
    const int tm = half ? whole : id % whole, tn = half ? id : id / whole;
    const int64_t n_tile0 = (int64_t)g.n_first + (int64_t)tn * BN;

    const int KH_all = (int)(g.K >> 6), KC = (int)(g.K >> 7);   // K-steps of 64 / fragments of 128 per row-block in memory
    const int kh0 = SPLITK ? part * g.steps[half] : 0;  // (even: a part starts on a fragment)
    const int KH = SPLITK ? min(g.steps[half], KH_all - kh0) : KH_all;
    const int a_rbs = (int)((g.M + 15) / 16), w_rbs = (int)((g.N + 15) / 16);
    const int a_rb0 = min(tm * FX, a_rbs - 1), w_rb0 = min((int)(n_tile0 / 16), w_rbs - 1);
    const int a_rb_last = a_rbs - 1 - a_rb0, w_rb_last = w_rbs - 1 - w_rb0;
    auto make_rsrc = [](const uint8_t* base, int64_t bytes) {
        const uint32_t n = bytes > 0xffffffffll ? 0xffffffffu : (uint32_t)bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, (int)n, 0x00020000);
    };
    const int64_t x0 = (int64_t)kh0 * 2048, c0 = (int64_t)(kh0 >> 1) * 1024, s0 = (int64_t)(kh0 >> 1) * 128;
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(g.x16 + (int64_t)a_rb0 * KH_all * 2048 + x0, (int64_t)(a_rbs - a_rb0) * KH_all * 2048 - x0);
    const __amdgpu_buffer_rsrc_t rs_wc = make_rsrc(g.w_codes + (int64_t)w_rb0 * KC * 1024 + c0, (int64_t)(w_rbs - w_rb0) * KC * 1024 - c0);
    const __amdgpu_buffer_rsrc_t rs_ws = make_rsrc(g.w_scales + (int64_t)w_rb0 * KC * 128 + s0, (int64_t)(w_rbs - w_rb0) * KC * 128 - s0);
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const int x_rb_bytes = KH_all * 2048, wc_rb_bytes = KC * 1024, ws_rb_bytes = KC * 128;

    // Row-blocks past the end of an operand (last tile) are clamped to its last row-block: the duplicates only feed
    // outputs that are never stored.  A stage's copies are issued in three pieces (X, W codes, W scales) at three points of
    // the K-step.  Every copy is a full-wave instruction (no lane predicate, hence no branch inside the K-step):
    //   X: 1 KB chunks, 16 bytes per lane;
    //   W codes: a K-step of a fragment is 512 contiguous bytes -- one instruction copies the halves of TWO row-blocks,
    //     lanes 0-31 from one and lanes 32-63 from the next, into adjacent LDS slots (direct-to-LDS loads place lane l's
    //     data at 16 l behind the base whatever address the lane reads from);
    //   W scales: 64 bytes per row-block and K-step -- one instruction copies those of FOUR row-blocks, 16 lanes each.
    static_assert(WPW % 2 == 0 && (WPW == 4 || WPW == 2), "W halves are copied in pairs, scales in fours (or twos)");
    const uint32_t wc_voff0 = (uint32_t)((lane & 31) * 16 + min(wave * WPW + (lane >> 5), w_rb_last) * wc_rb_bytes);
    const uint32_t wc_voff1 = (uint32_t)((lane & 31) * 16 + min(wave * WPW + 2 + (lane >> 5), w_rb_last) * wc_rb_bytes);   // (WCI = 2 only)
    // (a wave that owns two row-blocks only fills the rest of its 256-byte slot with the scales of the two behind them)
    const uint32_t ws_voff = (uint32_t)((lane & 15) * 4 + min(wave * WPW + (lane >> 4), w_rb_last) * ws_rb_bytes);
    auto issue_x = [&](auto rm, int kl, char* base) {
        constexpr int XPW = decltype(rm)::value * 2 / NW;   // 1 KB chunks a wave copies per stage
#pragma unroll
        for (int i = 0; i < XPW; ++i) {
            const int c = wave * XPW + i;                 // chunk = (row-block, plane)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (lds_void*)(base + c * 1024), 16, lane16,
                                                     min(c >> 1, a_rb_last) * x_rb_bytes + kl * 2048 + (c & 1) * 1024, 0, 0);
        }
    };
    auto issue_wc = [&](int kl, char* base) {
#pragma unroll
        for (int i = 0; i < WCI; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_wc, (lds_void*)(base + X_BYTES + (wave * WPW + 2 * i) * 512), 16, i == 0 ? wc_voff0 : wc_voff1,
                                                     (kl >> 1) * 1024 + (kl & 1) * 512, 0, 0);
    };
    auto issue_ws = [&](int kl, char* base) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ws, (lds_void*)(base + X_BYTES + WC_BYTES + wave * WS_SLOT), 4, ws_voff,
                                                 (kl >> 1) * 128 + (kl & 1) * 64, 0, 0);
    };
    // stage k goes to ring slot k % STAGES; past the last stage the copies repeat it into a slot nobody reads any more, so
    // that every K-step issues the same operations (no branch, uniform vmcnt bookkeeping)
    auto issue = [&](auto rm, int k) {
        const int kl = min(k, KH - 1);
        char* base = smem + (k % STAGES) * STAGE_BYTES;
        issue_x(rm, kl, base);
        issue_wc(kl, base);
        issue_ws(kl, base);
    };

    v4f acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // where lane (r, q) finds its 8 code bytes and its scale byte inside a W half-fragment
    const int r = lane & 15, q = lane >> 4;
    const int w_code_off = ((q >> 1) * 16 + r) * 16 + (q & 1) * 8;
    const int w_scale_off = ((q >> 1) * 16 + r) * 2 + (q & 1);

    // A W half-fragment in three states: raw (8 code bytes + the scale byte), its scale as packed halves, and the 16
    // dequantized halves.  The conversion is cut into eight micro-steps (one byte of codes = two values each: a convert and
    // a packed multiply) that the K-step places between the MFMAs of the column-tile before: a wave issues in order, so
    // vector-ALU work overlaps MFMA execution only where the two alternate in the instruction stream.
    struct WRaw {
        v2i codes;
        uint32_t scale;
    };
    struct WHalf {
        v2h h[8];   // h[4 s + b] = elements 8 s + 2 b, 8 s + 2 b + 1
    };
    auto read_w = [&](const char* base, int i) {
        const int f = wave * TN + i;
        WRaw w;
        w.codes = *reinterpret_cast<const v2i*>(base + X_BYTES + f * 512 + w_code_off);
        w.scale = *reinterpret_cast<const uint8_t*>(base + X_BYTES + WC_BYTES + wave * WS_SLOT + i * 64 + w_scale_off);
        return w;
    };
    auto scale2 = [&](const WRaw& w) {
        const _Float16 sh = (_Float16)e4m3_decode<true>(w.scale);
        return v2h{sh, sh};
    };
    auto micro = [&](const WRaw& w, v2h s2, WHalf& out, int u) {   // u = 0..7, a compile-time constant after unrolling
        const uint32_t c = (uint32_t)w.codes[u >> 2];
        v2h p;
        switch (u & 3) {
            case 0: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 0); break;
            case 1: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 1); break;
            case 2: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 2); break;
            default: p = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, 3); break;
        }
        out.h[u] = p * s2;
    };
    auto operand = [&](const WHalf& w, int s) {
        const v8h v = {w.h[4 * s][0], w.h[4 * s][1], w.h[4 * s + 1][0], w.h[4 * s + 1][1],
                       w.h[4 * s + 2][0], w.h[4 * s + 2][1], w.h[4 * s + 3][0], w.h[4 * s + 3][1]};
        return v;
    };

    // The K-step's operands are read one step ahead: behind the barrier that says stage kh + 1 has landed, the MFMAs of step
    // kh's LAST column-tile alternate with the reads of stage kh + 1 -- every X fragment is replaced right after its last use --
    // and with the conversion of its first W half-fragment, so that no MFMA waits for LDS at the head of a step.
    v8h xf[TM][2];
    WRaw wraw[TN];
    WHalf wcur, wnext;
    auto read_x = [&](const char* base, int j, int s) { xf[j][s] = *(reinterpret_cast<const v8h*>(base + (j * 2 + s) * 1024) + lane); };
    // RM: 16-row blocks that are copied and multiplied, eight or -- the tile holds at most 64 tokens -- the first four
    auto steps = [&](auto rm) {
        constexpr int RM = decltype(rm)::value;
        constexpr int OPS = RM * 2 / NW + WCI + 1;   // vector-memory operations per wave and stage
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s) issue(rm, s);
        wait_vmcnt<(STAGES - 2) * OPS>();
        block_barrier();
#pragma unroll
        for (int i = 0; i < TN; ++i) wraw[i] = read_w(smem, i);
#pragma unroll
        for (int t = 0; t < 2 * RM; ++t) read_x(smem, t % RM, t / RM);
        {
            const v2h s2 = scale2(wraw[0]);
#pragma unroll
            for (int u = 0; u < 8; ++u) micro(wraw[0], s2, wcur, u);
        }
        // lgkmcnt(0): nothing is pending where the loop is entered, so that the waits inside count its own reads only (with an
        // order of its own on the way in, the compiler waits for everything at the head of every step)
        __builtin_amdgcn_s_waitcnt(0xc07f);
        for (int kh = 0; kh < KH; ++kh) {
            const int kn = kh + STAGES - 1, kl = min(kn, KH - 1);
            char* const fill = smem + (kn % STAGES) * STAGE_BYTES;
            const char* const next = smem + ((kh + 1) % STAGES) * STAGE_BYTES;
            __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
            for (int i = 0; i < TN; ++i) {
                const bool last = i + 1 == TN;
                if (last) {
                    // stage kh + 1 has landed (this wave's copies: vmcnt; everybody's: barrier); the barrier also says that every
                    // wave holds stage kh in registers, so that its slot may be refilled
                    wait_vmcnt<(STAGES - 2) * OPS>();
                    block_barrier();
    #pragma unroll
                    for (int v = 0; v < TN; ++v) wraw[v] = read_w(next, v);
                    __builtin_amdgcn_sched_barrier(0);
                }
                v2h s2 = {0, 0};
                if (!last) s2 = scale2(wraw[i + 1]);
                if (last && RM == 4) s2 = scale2(wraw[0]);
                const v8h a0 = operand(wcur, 0), a1 = operand(wcur, 1);
    #pragma unroll
                for (int t = 0; t < 2 * RM; ++t) {
                    const int j = t % RM, s = t / RM;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(s == 0 ? a0 : a1, xf[j][s], acc[i][j], 0, 0, 0);
                    if (!last) {
                        if (t < 8) micro(wraw[i + 1], s2, wnext, t);
                    } else {
                        read_x(next, j, s);
                        if (t == 2 * RM - 9) s2 = scale2(wraw[0]);
                        if (t >= 2 * RM - 8) micro(wraw[0], s2, wnext, t - (2 * RM - 8));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the refill of the slot everybody left at the barrier of the step before, in pieces behind the first column-tiles
                if (i == 0) issue_x(rm, kl, fill);
                if (i == (TN == 2 ? 0 : 1)) issue_wc(kl, fill);
                if (i == (TN == 2 ? 0 : 2)) issue_ws(kl, fill);
                __builtin_amdgcn_sched_barrier(0);
                wcur = wnext;
            }
        }
    };
    if (half) steps(std::integral_constant<int, 4>{});
    else steps(std::integral_constant<int, TM>{});
    wait_vmcnt<0>();   // (the repeated copies of the last steps: nothing may be in flight into LDS when the workgroup ends)

    // A lane owns out[m][n .. n+3] with m = m0 + 16 j + lane % 16, n = n0 + 16 i + 4 (lane / 16).
    const float ts = SPLITK ? 1.0f : (*g.a_ts) * (*g.w_ts);
    const int64_t n_lim = (int64_t)g.n_first + g.n_cols;
    const int64_t n_end = n_lim < g.N ? n_lim : g.N;
    const int64_t m_base = (int64_t)tm * BM + (lane & 15);
    // a part's slice: the rows of the whole tiles, or those of the last row of tiles
    const int64_t rows0 = (int64_t)whole * BM, slice_rows = half ? g.M - rows0 : min(rows0, g.M);
    float* const slice = SPLITK ? g.partial[half] + (part * slice_rows - (half ? rows0 : 0)) * g.N : nullptr;
    const int64_t n_base = n_tile0 + wave * WN + (lane >> 4) * 4;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int64_t m = m_base + 16 * j;
        if (m >= g.M) continue;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int64_t n = n_base + 16 * i;
            if (n >= n_end) continue;
            v4f v = acc[i][j];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= ts;
            if constexpr (OUT_F32) {
                float* o = (SPLITK ? slice : static_cast<float*>(g.out)) + m * g.N + n;
                if (n + 3 < n_end && (g.N & 3) == 0) {
                    *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
                    for (int e = 0; e < 4; ++e)
                        if (n + e < n_end) o[e] = v[e];
                }
            } else {
                __bf16* o = static_cast<__bf16*>(g.out) + m * g.N + n;
                typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
                if (n + 3 < n_end && (g.N & 3) == 0) {
                    const v4bf p = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                    __builtin_nontemporal_store(p, reinterpret_cast<v4bf*>(o));
                } else {
                    for (int e = 0; e < 4; ++e)
                        if (n + e < n_end) o[e] = (__bf16)v[e];
                }
            }
        }
    }
}

// out[i] = s_T(A) s_T(W) (partial[0][i] + partial[1][i] + ...), the parts added in their order, as bf16 or fp32: the rows of the whole
// tiles, then those of the last row of tiles, either with slices of its own.  VEC neighbouring elements per thread.
struct Nv16Sums {
    const float* partial[2];
    int parts[2];
    int64_t count[2];   // elements
    const float *a_ts, *w_ts;
    void* out;
};
template <bool OUT_F32, int VEC>
__global__ __launch_bounds__(256) void nv16_reduce_kernel(Nv16Sums a)
{
    typedef float vf __attribute__((ext_vector_type(VEC)));
    typedef __bf16 vb __attribute__((ext_vector_type(VEC)));
    const int64_t at = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VEC;
    const bool last = at >= a.count[0];
    const int64_t count = a.count[last], i = last ? at - a.count[0] : at;
    if (i >= count) return;
    const float* p = a.partial[last] + i;
    const int parts = a.parts[last];
    vf s = *reinterpret_cast<const vf*>(p);
    for (int k = 1; k < parts; k += 4) {
        vf v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const vf*>(p + min(k + u, parts - 1) * count);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k + u < parts) s += v[u];
    }
    s *= (*a.a_ts) * (*a.w_ts);
    if constexpr (OUT_F32) *reinterpret_cast<vf*>(static_cast<float*>(a.out) + at) = s;
    else *reinterpret_cast<vb*>(static_cast<__bf16*>(a.out) + at) = __builtin_convertvector(s, vb);
}

// Split-K plan (see the MXFP4 kernels' plan: few tiles and a long K leave the launch bound by the latency of a handful of
// compute units' loads; here M = 128, N = 8192, K = 28672 is 32 tiles and 411 us, slower than a bf16 GEMM).  128 x 256
// (or 128 x 128) tiles, two workgroups per compute unit, at least 8 K-steps of 64 per part, at most sixteen parts.  A K-step takes about
// 0.93 us in a workgroup that has its compute unit to itself and half as much again when two share one; a 128 x 128 tile's
// takes 0.58 us.  The number of parts minimises the estimate (microseconds)
//     10 + K-steps per part x step time + (split only) 3 + splits x M x N x 8 bytes of partials at 8 TB/s
// (the partials are written and read back within microseconds: most of them never leave the last-level cache)
// and the product is split only for an estimated gain of at least 10 % over the unsplit launch (which uses the narrow
// tiles when the wide ones are at most a round and a quarter: see launch_gemm_nv16).
bool nv16_narrow_tiles(int64_t tiles_w, int cus)
{
    return 4 * tiles_w <= 5 * (int64_t)cus;
}

// bytes of the partials (0: not split)
size_t partial_bytes(const Nv16Parts& p, int64_t M, int64_t N)
{
    const int64_t last = p.half_row ? (M - 1) % 128 + 1 : 0;
    return p.parts[0] > 1 ? (size_t)(p.parts[0] * (M - last) + p.parts[1] * last) * (size_t)N * 4 : 0;
}

// `most`: bytes that as many parts for all tiles may take, `room`: that parts of different numbers may
Nv16Parts search_split_k_nv16(int64_t M, int64_t N, int64_t K, int cus, size_t most, size_t room)
{
    Nv16Parts plan;
    const int64_t tiles_m = (M + 127) / 128;
    const int64_t tiles_w = tiles_m * ((N + 255) / 256), tiles_n = tiles_m * ((N + 127) / 128);
    const int64_t slots = 2 * (int64_t)cus;
    const int kh = (int)(K >> 6);
    // every part is as slow as the slowest compute unit's, and that one runs two workgroups as soon as there are more
    // workgroups than compute units
    auto shared = [&](int64_t wgs) { return wgs <= cus ? 1.0 : 1.47; };
    double unsplit = 10.0 + kh * 0.93 * shared(tiles_w);
    if (nv16_narrow_tiles(tiles_w, cus)) unsplit = 10.0 + kh * 0.58 * shared(tiles_n);
    double best = 0.9 * unsplit;
    // parts of at least eight K-steps (whole multiples of eight), up to sixteen of them, of wide or of narrow tiles, on at most
    // two workgroups per compute unit
    for (int nar = 0; nar < 2; ++nar) {
        const int64_t tiles = nar ? tiles_n : tiles_w;
        const double step = nar ? 0.58 : 0.93;
        const int64_t s_max = std::min<int64_t>(std::min<int64_t>(slots / tiles, kh / 8), 16);
        for (int64_t s = 2; s <= s_max; ++s) {
            const int st = (int)(((kh + s - 1) / s + 7) / 8 * 8);
            const int64_t n = (kh + st - 1) / st;
            if (n < 2 || (double)n * (double)M * (double)N * 4.0 > (double)most) continue;
            const double t = 10.0 + st * step * shared(n * tiles) + 3.0 + (double)n * (double)M * (double)N * 8.0 / 8.0e6;
            if (t < best) {
                best = t;
                plan.parts[0] = plan.parts[1] = (int)n;
                plan.steps[0] = plan.steps[1] = st;
                plan.narrow = nar != 0;
            }
        }
    }
    if (plan.parts[0] == 1) return plan;
    // Split launches gain from K = 4096 on with half tiles last (M = 320: N = 8192, K = 28672 148 -> 142 us, N = 6144, K = 4096 37 -> 33); below, as often lose.
    // But where the whole tiles' parts are a round of compute units or less and all are more, no unit should have two whole ones (N = 18432, K = 3840, three
    // parts, M = 129 / 161: 51.9 / 53.2 us in turn, halves last 43.8 / 46.5).
    const int64_t row_wgs = (plan.narrow ? (N + 127) / 128 : (N + 255) / 256) * plan.parts[0], all = tiles_m * row_wgs;
    plan.half_row = (M - 1) % 128 < 64 && (K >= 4096 || (all > cus && all - row_wgs <= cus));
    const int64_t cols = (N + 511) / 512, rows = tiles_m - 1;
    plan.rows512 = !plan.narrow && K >= 6656 && tiles_w * plan.parts[0] > cus && tiles_m * cols * plan.parts[0] <= cus;   // (see wide())
    if (!plan.rows512 || !plan.half_row || rows == 0) return plan;
    // One workgroup per compute unit, and a part of a half tile takes 0.62 of a whole one's time: with as many parts for either as
    // suit each other, parts are shorter.  Microseconds: steps of the longer part times 1.38, and the partials as above.  M = 320, K = 8192,
    // N = 8192 and K = 28672, N = 8192: six and four parts instead of four, five of both, 60.9 -> 55.2 us, 143.9 -> 131.2.
    best = 0.0;
    for (int64_t s = 2; s <= std::min<int64_t>(16, kh / 8) && (rows * s + 1) * cols <= cus; ++s) {
        auto even = [&](int64_t n) { return (int)((kh + 2 * n - 1) / (2 * n) * 2); };
        const int st = even(s);
        int64_t h = std::min<int64_t>(cus / cols - rows * s, s);
        while (h > 1 && 0.62 * even(h - 1) <= st) --h;
        const int sh = even(h), n = (kh + st - 1) / st, nh = (kh + sh - 1) / sh;
        const int64_t partials = ((int64_t)n * rows * 128 + (int64_t)nh * (M - rows * 128)) * N;
        const double t = 1.38 * std::max<double>(st, 0.62 * sh) + (double)partials * 8.0 / 8.0e6;
        if ((size_t)partials * 4 > room || (best > 0.0 && t >= best)) continue;
        best = t;
        plan.parts[0] = n;
        plan.parts[1] = nh;
        plan.steps[0] = st;
        plan.steps[1] = sh;
    }
    return plan;
}

// the plan with all the room it likes, and only where its partials do not fit `room` that of the parts which do
Nv16Parts plan_split_k_nv16(int64_t M, int64_t N, int64_t K, int cus, size_t room)
{
    const Nv16Parts plan = search_split_k_nv16(M, N, K, cus, SIZE_MAX, room);
    return partial_bytes(plan, M, N) <= room ? plan : search_split_k_nv16(M, N, K, cus, room, room);
}

template <int NW, int TN, int STAGES, bool OUT_F32, bool SPLITK>
hipError_t launch_kernel(const Nv16Args& g, unsigned workgroups, hipStream_t st)
{
    constexpr size_t lds = STAGES * (size_t)(8 * 2048 + NW * TN * 512 + NW * 256);
    static LdsAttrOnce raised;
    auto k = gemm_nv16_kernel<NW, TN, OUT_F32, STAGES, SPLITK>;
    const hipError_t e = raised.ensure(reinterpret_cast<const void*>(k), (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(workgroups), dim3(NW * 64), lds, st, g);
    return hipGetLastError();
}

// (g.parts[0] == 0: tiles are not split)
template <int NW, int TN, int STAGES>
hipError_t launch_tiles(const Nv16Args& g, bool out_f32, hipStream_t st)
{
    constexpr int BN = NW * TN * 16;
    const int tiles_n = (g.n_cols + BN - 1) / BN;
    if (g.parts[0]) {
        const int n = tiles_n * ((g.tiles_m - g.half_row) * g.parts[0] + g.half_row * g.parts[1]);
        return launch_kernel<NW, TN, STAGES, true, true>(g, (unsigned)n, st);
    }
    const unsigned n = (unsigned)(g.tiles_m * tiles_n);
    return out_f32 ? launch_kernel<NW, TN, STAGES, true, false>(g, n, st) : launch_kernel<NW, TN, STAGES, false, false>(g, n, st);
}

hipError_t launch_width(int width, const Nv16Args& g, bool out_f32, hipStream_t st)
{
    return width == 512 ? launch_tiles<8, 4, 3>(g, out_f32, st) : width == 128 ? launch_tiles<4, 2, 3>(g, out_f32, st) : launch_tiles<4, 4, 3>(g, out_f32, st);
}

Nv16Launch of_width(int width, int64_t first, int64_t cols, int64_t tiles_m, bool half_row, int64_t cus)
{
    Nv16Launch l{width, (int)first, (int)cols, 0};
    if (half_row) {
        // Half tiles go last where that evens out the launch's end or gives every compute unit one whole tile at most.  Else the launch takes
        // the time of whole tiles, and all of them in turn leave an XCD its rows of X (K = 2048, N = 12288, M = 960: 58 us, halves last 61.5).
        const int64_t tiles_n = (cols + width - 1) / width, all = tiles_m * tiles_n;
        l.half_row = all > 2 * cus || (all > cus && all - tiles_n <= cus) ? 1 : 0;
    }
    return l;
}

// Tile columns of 256 (or wider).  Two workgroups of 128 x 256 share a compute unit, and one's epilogue runs under the other's
// products; but each copies the same rows of X into LDS for itself.  Where a single round of the chip has more such
// workgroups than compute units and no more than one of twice the width, eight waves share a 128 x 512 tile instead (34 KB
// copied per K-step, not 50; there is no second round for an epilogue to run under): N = 8192, M = 2048: K = 28672 669 ->
// 641 us, K = 8192 205 -> 201.  Over several rounds the pairs stay ahead (N = 57344, K = 8192: 1324 against 1342 us), and below
// K = 6656, where a tile is short for its start-up and epilogue, which the pair overlaps: on 23 shapes from there to K = 15000
// 512 columns took 0.95 - 1.02 of the pairs' time (M = 419, N = 24064, K = 8576: 180 -> 171 us), on 47 below it 0.98 - 1.11
// (M = 451, N = 25992, K = 1536: 54 against 60).
// Three stages either way: a fourth for the 512 columns measured 1 % slower.
Nv16Launch wide(int64_t first, int64_t cols, int64_t tiles_m, bool half_row, int64_t K, int64_t cus)
{
    // (a compute unit that gets one whole tile and one of half the rows is done sooner as a pair: M = 192, N = 57344, K = 8192 163 -> 153 us)
    const bool pairs = half_row && (tiles_m - 1) * ((cols + 255) / 256) <= cus;
    const bool rows512 = !pairs && K >= 6656 && tiles_m * ((cols + 255) / 256) > cus && tiles_m * ((cols + 511) / 512) <= cus;
    return of_width(rows512 ? 512 : 256, first, cols, tiles_m, half_row, cus);
}

// Estimated time of a launch, microseconds per K-step: `whole` tiles and behind them `half` ones (of at most 64 tokens), wide or narrow.
// A tile's step takes `alone` on a compute unit of its own, `shared` beside another, 0.62 of that with half the rows.
double nv16_tiles_cost(int64_t whole, int64_t half, bool narrow, int64_t cus)
{
    const double alone = narrow ? 0.58 : 0.93, shared = 1.47 * alone, part = 0.62;
    const int64_t slots = 2 * cus, left = whole % slots;
    const double t = (double)(whole / slots) * shared;
    auto last = [&](int64_t n, double f) { return n == 0 ? 0.0 : f * (n <= cus ? alone : shared); };
    if (left == 0) return t + (double)(half / slots) * part * shared + last(half % slots, part);
    if (left + half <= cus) return t + alone;
    if (left <= cus && left + half <= slots) return t + 0.5 * (alone + shared);
    // halves run on the slots that whole tiles leave, and behind all of them what does not fit there
    return t + shared + ((double)half * part > (double)(slots - left) ? part * alone : 0.0);
}

// The product in one piece along K: one launch or two.  Two workgroups per compute unit: a round of the chip is 2 * CUs tiles.  The tile columns that
// fill whole rounds run as 128 x 256 tiles; what is left over runs as 128 x 128 tiles in a second launch when that fits it
// into fewer rounds-worth of time (N = 10240 at M = 4096: 1280 wide tiles are two and a half rounds; 1024 of them
// plus 512 narrow ones are two and a half rounds' worth of work in two and a half rounds' time).
int plan_whole(int64_t M, int64_t N, int64_t K, int cus, Nv16Launch (&l)[2])
{
    const int64_t tiles_m = (M + 127) / 128;
    const bool half_row = (M - 1) % 128 < 64;
    const int64_t slots = 2 * (int64_t)cus;
    const int64_t cols_w = (N + 255) / 256;                         // wide tile columns
    const int64_t tiles_w = cols_w * tiles_m;
    const int64_t full_cols = tiles_w / slots * slots / tiles_m;    // wide tile columns inside whole rounds
    const int64_t rest_cols = N - full_cols * 256;                  // output columns left over
    if (full_cols > 0 && full_cols < cols_w) {
        const int64_t narrow = (rest_cols + 127) / 128 * tiles_m;
        // time in units of a wide tile: ceil-rounds of wide tiles, against whole rounds + narrow tiles at half a unit each
        double t_wide = (double)((tiles_w + slots - 1) / slots);
        double t_split = (double)(full_cols * tiles_m / slots) + 0.5 * (double)((narrow + slots - 1) / slots);
        if (half_row) {
            const int64_t whole = tiles_m - 1, cols_n = (rest_cols + 127) / 128, all_n = (N + 127) / 128;
            t_wide = std::min(nv16_tiles_cost(whole * cols_w, cols_w, false, cus), nv16_tiles_cost(whole * all_n, all_n, true, cus));
            t_split = nv16_tiles_cost(whole * full_cols, full_cols, false, cus) + nv16_tiles_cost(whole * cols_n, cols_n, true, cus) + 10.0 / (double)(K >> 6);
        }
        if (t_split < t_wide) {
            l[0] = wide(0, full_cols * 256, tiles_m, half_row, K, cus);
            l[1] = of_width(128, full_cols * 256, rest_cols, tiles_m, half_row, cus);
            return 2;
        }
    }
    // With a last row of half tiles, which are handed out last and even out the end of the launch, one launch is the better one unless the
    // narrow tiles of the second fill what the wide ones leave (K, N, M: whole rounds first -> one launch, us: 8192, 57344, 320
    // 259 -> 247; 8192, 57344, 560 430 -> 416; 4096, 28672, 1080 224 -> 207; 28672, 8192, 1080 narrow 494, wide 466).
    // Less than a round and a quarter of wide tiles (one per compute unit and a few doubled up, or compute units left
    // idle): 128 x 128 tiles spread the same work twice as finely (N = 10240, K = 8192 at M = 512: 136 -> 119 us;
    // N = 8192, K = 28672 at M = 512 without the split-K workspace: 412 -> 280 us).
    const int64_t cols_n = (N + 127) / 128, whole = tiles_m - 1;
    const bool narrow = half_row ? nv16_tiles_cost(whole * cols_n, cols_n, true, cus) < nv16_tiles_cost(whole * cols_w, cols_w, false, cus) : nv16_narrow_tiles(tiles_w, cus);
    l[0] = narrow ? of_width(128, 0, N, tiles_m, half_row, cus) : wide(0, N, tiles_m, half_row, K, cus);
    return 1;
}

// the product in parts, and their sums
hipError_t launch_parts(Nv16Args g, const Nv16Parts& plan, bool out_f32, float* partial, hipStream_t st)
{
    g.n_first = 0;
    g.n_cols = (int)g.N;
    g.half_row = plan.half_row ? 1 : 0;
    const int64_t rows0 = std::min<int64_t>((int64_t)(g.tiles_m - g.half_row) * 128, g.M);
    Nv16Sums r{};
    r.a_ts = g.a_ts;
    r.w_ts = g.w_ts;
    r.out = g.out;
    for (int h = 0; h < 2; ++h) {
        g.steps[h] = plan.steps[h];
        r.parts[h] = g.parts[h] = plan.parts[h];
        r.partial[h] = g.partial[h] = partial;
        r.count[h] = (h ? g.M - rows0 : rows0) * g.N;
        partial += r.parts[h] * r.count[h];
    }
    const hipError_t e = launch_width(plan.width(), g, out_f32, st);
    if (e != hipSuccess) return e;
    const bool vec = g.N % 4 == 0;
    const dim3 grid((unsigned)((g.M * g.N / (vec ? 4 : 1) + 255) / 256));
    if (out_f32) {
        if (vec) hipLaunchKernelGGL((nv16_reduce_kernel<true, 4>), grid, dim3(256), 0, st, r);
        else hipLaunchKernelGGL((nv16_reduce_kernel<true, 1>), grid, dim3(256), 0, st, r);
    } else {
        if (vec) hipLaunchKernelGGL((nv16_reduce_kernel<false, 4>), grid, dim3(256), 0, st, r);
        else hipLaunchKernelGGL((nv16_reduce_kernel<false, 1>), grid, dim3(256), 0, st, r);
    }
    return hipGetLastError();
}

}  // namespace

size_t nv16_workspace_bytes(int64_t M, int64_t K)
{
    return (size_t)(round_up(M, 16) * K * 2);
}

// Price of the whole call: the fp16 copy of X, the launches of the plan, the sum of the parts, the output.  A half tile counts as 0.7 of a whole one; where a unit has one whole tile at most and some a half
// one besides, the launch takes a way of 0.3 from whole tiles alone to as many whole ones; parts count half as the longest of them and half as their mean.  Fitted to 3902 products on two cards (M = 33 ... 4096, N = 256 ... 57344, K = 256 ... 28672, half of them
// multiples of 256), where they run in parts with room for them and without: median error 3 %, one in ten off by more than 10 %.
static double nv16_us(int64_t M, int64_t N, int64_t K, int cus, const Nv16Plan& plan)
{
    constexpr TileRounds narrow = {2, 5.7906, 0.6708, 0.0000, 0.4982, 0.0202, 1.9628, 0.6652, 0.1387}, wide = {2, 10.5536, 1.2001, 2.3438, 0.3651, 0.5578, 6.5882, 1.0898, 0.2570},
                         rows512 = {1, 4.023, 1.3912, 4.023, 0.8982, 0.4930};   // (one round at most)
    const int64_t tiles_m = (M + 127) / 128;
    double us = 6.579 + 0.3803e-6 * (double)M * (double)K + 0.8693e-6 * (double)M * (double)N;
    auto add = [&](int width, int64_t cols, int64_t half_row, int64_t parts, int64_t half_parts, double steps) {
        const TileRounds& c = width == 512 ? rows512 : width == 256 ? wide : narrow;
        const double tiles_n = (double)((cols + width - 1) / width), whole = tiles_n * (double)((tiles_m - half_row) * parts), half = tiles_n * (double)(half_row * half_parts);
        if (c.per_cu == 2 && whole <= cus && whole + half > cus && whole + half <= 2 * cus)
            us += 0.7 * tile_rounds_us(c, cus, steps, cus) + 0.3 * tile_rounds_us(c, whole + half, steps, cus);
        else
            us += tile_rounds_us(c, whole + 0.7 * half, steps, cus);
    };
    const Nv16Parts& p = plan.split;
    if (p.parts[0] > 1) {
        us += 6.429 + 0.1332e-6 * (double)plan.partial_bytes;
        add(p.width(), N, p.half_row, p.parts[0], p.parts[1], 0.5 * (p.steps[0] + (double)(K >> 6) / p.parts[0]));
        return us;
    }
    for (int i = 0; i < plan.launches; ++i) add(plan.launch[i].width, plan.launch[i].n_cols, plan.launch[i].half_row, 1, 1, (double)(K >> 6));
    return plan.launches > 1 ? us + 7.763 : us;
}

Nv16Plan plan_nv16(int64_t M, int64_t N, int64_t K, size_t partial_room)
{
    const int cus = compute_units();
    Nv16Plan p;
    // few tiles, long K: every tile's K range shared by several workgroups, partial results added by a second kernel
    if (partial_room) p.split = plan_split_k_nv16(M, N, K, cus, partial_room);
    p.partial_bytes = partial_bytes(p.split, M, N);
    if (!p.partial_bytes) p.launches = plan_whole(M, N, K, cus, p.launch);
    p.us = nv16_us(M, N, K, cus, p);
    return p;
}

hipError_t launch_gemm_nv16(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes,
                            const void* w_scales, const float* w_ts, int64_t M, int64_t N, int64_t K, void* out,
                            bool out_f32, const Nv16Plan& plan, void* workspace, void* partial, hipStream_t st)
{
    // 1. activations -> fp16 in operand order (workspace)
    const int64_t n_frags = round_up(M, 16) / 16 * (K / 128);
    hipLaunchKernelGGL(nv_x16_kernel, dim3((unsigned)((n_frags + 3) / 4)), dim3(256), 0, st, static_cast<const uint8_t*>(a_codes),
                       static_cast<const uint8_t*>(a_scales), static_cast<uint8_t*>(workspace), n_frags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    // 2. the product
    Nv16Args g{};
    g.x16 = static_cast<const uint8_t*>(workspace);
    g.w_codes = static_cast<const uint8_t*>(w_codes);
    g.w_scales = static_cast<const uint8_t*>(w_scales);
    g.a_ts = a_ts;
    g.w_ts = w_ts;
    g.out = out;
    g.M = M;
    g.N = N;
    g.K = K;
    g.tiles_m = (int)((M + 127) / 128);
    if (plan.partial_bytes) return launch_parts(g, plan.split, out_f32, static_cast<float*>(partial), st);
    for (int i = 0; i < plan.launches; ++i) {
        g.n_first = plan.launch[i].n_first;
        g.n_cols = plan.launch[i].n_cols;
        g.half_row = plan.launch[i].half_row;
        if ((e = launch_width(plan.launch[i].width, g, out_f32, st)) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fp4mr
