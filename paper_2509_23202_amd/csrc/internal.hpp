// Host-side launchers behind the C ABI (one per kernel family).  All pointers are device pointers that the
// C-ABI layer has already validated.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace fp4mr {

// Process-wide tuning / cross-check switches behind fp4_set_option (plain ints: set them before concurrent use).
struct Options {
    int gemm_variant = 0;  // 0 = tile shape by the cost model, else a forced tile configuration of the GEMM kernels
    int gemm_grid = 0;     // > 0: cap on the number of persistent workgroups (a small grid walks many tiles each)
    int sw_codec = 0;      // != 0: element and scale codecs in integer arithmetic instead of the converting instructions
};
Options& options();

// Raises a kernel's dynamic-LDS limit the first time the kernel is launched on a device (one object per kernel).
struct LdsAttrOnce {
    std::atomic<uint64_t> done{0};  // bit d: set on device d
    hipError_t ensure(const void* kernel, int lds_bytes)
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 63;  // (unknown device: set it every time)
        const uint64_t bit = 1ull << dev;
        if (dev != 63 && (done.load(std::memory_order_relaxed) & bit)) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
        return e;
    }
};

// compute units of the current device (cached per device)
int compute_units();

// largest valid forced tile configuration per format (fp4_gemm rejects anything else before it launches)
constexpr int kMaxGemmVariantMx = 18;
constexpr int kMaxGemmVariantNv = 4;
// NVFP4: chosen as by itself, but without the kernel that dequantizes both operands in its waves
constexpr int kVariantNvNoCodes = 4;

// policy: group scales by 0 abs-max, 1 squared-error search, 2 rounded exponent with the 4/3 factor (MXFP4 only).
// rot: null for the normalised Hadamard of size b, else a bf16 [b, b] row-major matrix (y = x . rot per block)
hipError_t launch_rotate_quantize(const void* x, int64_t rows, int64_t K, int b, const void* rot, int fmt, bool in_f32,
                                  int layout_gemm, bool static_scale, int policy, void* codes, void* scales,
                                  float* tensor_scale, void* workspace, bool hw_codec, hipStream_t st);

// canonical -> GEMM layout copy of one quantized operand (codes and scales)
hipError_t launch_repack_to_gemm(const void* codes, const void* scales, int64_t rows, int64_t K, int fmt,
                                 void* codes_gemm, void* scales_gemm, hipStream_t st);

// variant: a tile configuration of the MXFP4 GEMM, or 0 for the few-token kernels; splits > 1: parts of `steps` K-steps each
struct MxPlan {
    int variant, splits, steps;
};

// both operands in GEMM layout; alpha multiplies the result (1, or powers of 4/3 for operands quantized with the
// rounded-exponent rule whose scale bytes leave that tensor-level factor out)
hipError_t launch_gemm_mxfp4(const void* a_codes, const void* a_scales, const void* w_codes, const void* w_scales,
                             int64_t M, int64_t N, int64_t K, void* out, bool out_f32, const MxPlan& plan, float alpha, void* partial,
                             hipStream_t st);
// how an MXFP4 product runs best with `room` bytes for partials
MxPlan plan_mx(int64_t M, int64_t N, int64_t K, size_t room);
// what the few-token kernels take for it, in microseconds; 0: they take it, whatever that is; infinity: they do not take it
double gemm_stream_us(int64_t M, int64_t N, int64_t K);
// fp32 partials of a split-K run (few tiles, long K: every tile's K range shared by several workgroups); 0 = not split
size_t gemm_mx_split_k_bytes(int64_t M, int64_t N, int64_t K);

// variants 1..3: the tile kernels that dequantize both operands
hipError_t launch_gemm_nvfp4(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes,
                             const void* w_scales, const float* w_ts, int64_t M, int64_t N, int64_t K, void* out,
                             bool out_f32, int variant, hipStream_t st);

// A many-token NVFP4 product in parts along K (1: not in parts): numbers and K-steps of 64 of the parts of whole tiles, and of those of a last row of at most 64 tokens.
struct Nv16Parts {
    int parts[2] = {1, 1}, steps[2] = {0, 0};
    bool narrow = false, rows512 = false;       // tiles of 128 columns; of 512
    bool half_row = false;
    int width() const { return rows512 ? 512 : narrow ? 128 : 256; }
};
// one launch of it in one piece: columns n_first .. n_first + n_cols - 1 in tiles of `width`, the last row's half tiles behind all others or not
struct Nv16Launch {
    int width, n_first, n_cols, half_row;
};
struct Nv16Plan {
    Nv16Parts split;
    size_t partial_bytes = 0;   // 0: not in parts, but in these launches
    int launches = 0;
    Nv16Launch launch[2] = {};
    double us = 0.0;            // what it is estimated to take
};

// NVFP4 product for many tokens: the activations are dequantized once to fp16 into `workspace`
// (nv16_workspace_bytes(M, K) bytes, 256-byte aligned), then multiplied against W dequantized on the fly.  plan: with that room for fp32 partials (with little, in
// fewer parts or not split).
size_t nv16_workspace_bytes(int64_t M, int64_t K);
Nv16Plan plan_nv16(int64_t M, int64_t N, int64_t K, size_t partial_room);
hipError_t launch_gemm_nv16(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes,
                            const void* w_scales, const float* w_ts, int64_t M, int64_t N, int64_t K, void* out,
                            bool out_f32, const Nv16Plan& plan, void* workspace, void* partial, hipStream_t st);

// What the workgroups of a launch take, microseconds, `steps` of K each: `per_cu` to a compute unit in rounds, each (fixed + steps x step), and a last round, whole or
// not: on units of their own (alone + steps x (alone_step + alone_busy x the share of the units)), or some of them two to a unit.
struct TileRounds {
    int per_cu;
    double fixed, step, alone, alone_step, alone_busy, pair, pair_step, pair_busy;
};
inline double tile_rounds_us(const TileRounds& c, double workgroups, double steps, int cus)
{
    const double slots = (double)cus * c.per_cu;
    double full = (double)(int64_t)(workgroups / slots), rest = workgroups - full * slots;
    if (rest <= 0.0 && full > 0.0) {   // (a last round that is whole is no faster for it: priced as one of many, 512 workgroups were 15 % too cheap)
        full -= 1.0;
        rest = slots;
    }
    const double t = full * (c.fixed + steps * c.step);
    if (rest <= cus) return t + c.alone + steps * (c.alone_step + c.alone_busy * rest / cus);
    return t + c.pair + steps * (c.pair_step + c.pair_busy * (rest - cus) / cus);
}

// NVFP4 product of 33 tokens and more, both operands dequantized inside it, in one launch without a workspace.  plan: the tile that suits it, or -1 where what
// takes `other` microseconds otherwise, on the few-token kernels or the one for many tokens, is the better choice.
int plan_nv_codes(int64_t M, int64_t N, int64_t K, double other, bool few);
hipError_t launch_gemm_nv_codes(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes, const void* w_scales, const float* w_ts,
                                int64_t M, int64_t N, int64_t K, void* out, bool out_f32, int tile, hipStream_t st);

// few-token weight-streaming GEMM, both formats, operands in GEMM layout: every shape up to 64 tokens, and above that those that
// gemm_nv_streams accepts (NVFP4) and gemm_stream_us prices (MXFP4)
bool gemm_nv_streams(int64_t M, int64_t N, int64_t K);
// what they take for an NVFP4 product of more than 16 tokens, in microseconds, where a set of workgroups per 16 tokens does it (gemm_nv_streams); 0: they take
// it, whatever that is
double gemm_nv_stream_us(int64_t M, int64_t N, int64_t K);
hipError_t launch_gemm_skinny(const void* a_codes, const void* a_scales, const float* a_ts, const void* w_codes,
                              const void* w_scales, const float* w_ts, int64_t M, int64_t N, int64_t K, int fmt, void* out,
                              bool out_f32, float alpha, hipStream_t st);

// M <= 16, MXFP4: rotation + quantization of the activations inside the weight-streaming GEMM (W in GEMM layout);
// weight_only: the rotated activations stay bf16 (W4A16)
hipError_t launch_fused_decode(const void* x, int64_t M, int64_t K, int b, const void* w_codes, const void* w_scales,
                               int64_t N, void* out, bool out_f32, bool weight_only, float alpha, hipStream_t st);

// MR-GPTQ sweep over fixed scales (canonical layout) with the factor U of the damped inverse Hessian in visiting order;
// workspace of gptq_workspace_bytes(N, K) bytes, or of gptq_workspace_least at least, with the same codes later; K % 64 == 0, K <= 24576
size_t gptq_workspace_bytes(int64_t N, int64_t K);
size_t gptq_workspace_least(int64_t N, int64_t K);
hipError_t launch_gptq_sweep(const void* w, int64_t N, int64_t K, int b, int fmt, const float* U, const int* perm,
                             const void* scales, const float* s_T, const float* table, float factor, void* codes, void* workspace,
                             size_t workspace_bytes, hipStream_t st);

// Hessian [K,K] fp32 -> static activation order and the upper-triangular U with U^T U = (H[perm][:,perm] + damp mean(diag) I)^-1
size_t gptq_prepare_workspace_bytes(int64_t K);
hipError_t launch_gptq_prepare(const float* H, int64_t K, float damp, bool use_order, int* perm, float* U, void* workspace,
                               hipStream_t st);

// H (+)= (x H_b)^T (x H_b); workspace of 4 T K bytes: the rotated rows, or without rotation the partial sums of the last tiles
hipError_t launch_gptq_hessian(const void* x, int64_t T, int64_t K, int b, float* H, bool accumulate, void* workspace, hipStream_t st);

// measurement aids (fp4_probe): which = 0 scaled-FP4 MFMA issue loop, 1 fp16 MFMA issue loop (buf: one 24-byte record per
// compute unit), 2 streaming copy of the first half of buf to the second, 3 streaming read of the first half
// mode: 0 MXFP4, 1 MXFP4 with the tensor-level 4/3, 2 NVFP4, 3 scale byte fitted to the tensor's range (table at tensor_scale + 2)
hipError_t launch_dequantize(const void* codes, const void* scales, const float* tensor_scale, int64_t rows, int64_t K, int mode,
                             bool gemm_layout, void* out, bool out_f32, hipStream_t st);

hipError_t launch_probe(int which, void* buf, size_t bytes, int iters, hipStream_t st);

}  // namespace fp4mr
