// Hessian of a layer from calibration rows (arXiv 2509.23202, Section 4 "Standard GPTQ": the second-order information of
// ||X What - X W||^2 is X^T X; Section 4.1 "Ingredient 3": of the ROTATED inputs X H_b).
//
// The rotation is linear and the same for every row, so it is taken out of the sum:
//     (X H_b)^T (X H_b) = H_b^T (X^T X) H_b ,
// and X^T X is a product of bf16 values: its terms are exact in fp32, so the bf16 MFMA (16x the fp32 MFMA's rate) forms
// them without loss, with the fp32 accumulation the rotated product had.  The rotation then costs two butterflies on a
// finished 128 x 128 tile -- K^2 values instead of T K, none of them through memory -- and no rotated copy of X exists.
// The matrix is symmetric: only tiles on and below the diagonal are computed, each is stored twice.
//
// Bound: LDS bandwidth (a 64 x 64 wave tile reads 16 KB per 32 MFMAs), then the L2.  Tile 128 x 128 over 64 rows of X at a
// time, four waves, two workgroups per compute unit (64.5 KB of LDS) so that one's staging runs under the other's MFMAs.
// 8192 rows at K = 4096 (137 GFLOP in one triangle): 206 us; 4.12 ms before, when the rows were rotated into an fp32 copy
// (0.6 ms at b = 128) and multiplied, both triangles, on the fp32 MFMA (3.5 ms).  Against 64 bits: 3.9e-7 (1.4e-6 before).
// X is staged as it lies in memory, rows along the contraction; the MFMA operands want the contraction along a lane's
// registers, which the transposing LDS read (ds_read_b64_tr_b16) provides: no transposed copy in memory, no packing.
#include "device_util.hpp"
#include "internal.hpp"

#include <algorithm>

namespace fp4mr {
namespace {

constexpr int kT = 128;        // tile side
constexpr int kRows = 64;      // rows of X per stage
constexpr int kPitch = kT + 1; // of the fp32 tile in LDS: rows and columns both walk all banks
constexpr int kSuper = 8;      // tiles are visited in super-tiles of 8 x 8 (their operands are shared through one L2)

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));

struct HessArgs {
    const uint16_t* x;  // [T, K] bf16
    float* H;           // [K, K]
    float* part;        // partial tiles of the split tail
    int64_t T;
    int K, b, accumulate;
    int nt;             // tiles per side
    int full;           // tiles 0 .. full - 1 take all of T in one workgroup ...
    int parts;          // ... each of the others is shared by this many
    int chunk;          // rows of X per part (multiple of kRows)
    float inv_b;
};

// p-th tile of the lower triangle (row >= col), counted super-row by super-row
__device__ __forceinline__ void tile_of(int p, int nt, int& row, int& col)
{
    const int bs = kSuper;
    int R = 0, base = 0;
    for (;; ++R) {  // (at most nt / 8 scalar trips)
        const int h = min(bs, nt - R * bs);
        const int n = R * bs * h + h * (h + 1) / 2;
        if (p < base + n) break;
        base += n;
    }
    const int h = min(bs, nt - R * bs);
    int i = p - base;
    if (i < R * bs * h) {
        row = R * bs + i % h;
        col = i / h;
    } else {
        i -= R * bs * h;
        int r = 0;
        while (i > r) i -= ++r;  // row r of the small triangle holds r + 1 tiles
        row = R * bs + r;
        col = R * bs + i;
    }
}

// 32-byte chunk (16 columns) `ib` of staged row t lies at chunk (ib ^ swz(t)): the four rows that a lane group of a
// transposing read takes, and those of its neighbour group eight rows on, fall into different banks
__device__ __forceinline__ int swz(int t) { return (t & 7) ^ ((t >> 1) & 4); }

__device__ __forceinline__ void butterfly(float (&v)[64], int b, bool upper)
{
#pragma unroll
    for (int s = 1; s < 64; s *= 2) {
        if (s < b) {
#pragma unroll
            for (int e = 0; e < 64; ++e) {
                if (e & s) continue;
                const float lo = v[e], hi = v[e + s];
                v[e] = lo + hi;
                v[e + s] = lo - hi;
            }
        }
    }
    if (b == 128) {
#pragma unroll
        for (int e = 0; e < 64; ++e) {
            const float other = __shfl_xor(v[e], 1);
            v[e] = upper ? other - v[e] : v[e] + other;
        }
    }
}

// the finished sums of tile (ti, tj), in the MFMA's output order, rotated from both sides and stored with their mirror image
__device__ __forceinline__ void finish_tile(const HessArgs& a, int ti, int tj, const v4f (&acc)[4][4], float* S)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;
    __syncthreads();  // the staging buffers under S have been read
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) S[(wr + i * 16 + 4 * q + v) * kPitch + wc + j * 16 + l16] = acc[i][j][v];
    __syncthreads();
    if (a.b > 1) {
        float v[64];
        const int line = tid >> 1, half = tid & 1;
        float* p = S + line * kPitch + half * 64;
#pragma unroll
        for (int e = 0; e < 64; ++e) v[e] = p[e];
        butterfly(v, a.b, half);
#pragma unroll
        for (int e = 0; e < 64; ++e) p[e] = v[e];
        __syncthreads();
        p = S + half * 64 * kPitch + line;
#pragma unroll
        for (int e = 0; e < 64; ++e) v[e] = p[e * kPitch];
        butterfly(v, a.b, half);
#pragma unroll
        for (int e = 0; e < 64; ++e) p[e * kPitch] = v[e] * a.inv_b;  // (1/sqrt(b) from each side: a power of two, exact)
        __syncthreads();
    }
    const int r0 = ti * kT, c0 = tj * kT;
    const int c = tid & (kT - 1), r1 = tid >> 7;  // a wave stores 64 consecutive floats
    const bool diag = ti == tj;
    for (int side = 0; side < (diag ? 1 : 2); ++side) {
        const int row0 = side ? c0 : r0, col0 = side ? r0 : c0;
        if (col0 + c >= a.K) continue;
#pragma unroll 4
        for (int r = r1; r < kT; r += 2) {
            if (row0 + r >= a.K) break;
            // (on the diagonal both halves take the lower one's values: the two butterflies do not round symmetrically)
            const bool swap = side || (diag && c > r);
            const float s = swap ? S[c * kPitch + r] : S[r * kPitch + c];
            float* p = a.H + (int64_t)(row0 + r) * a.K + col0 + c;
            *p = a.accumulate ? *p + s : s;
        }
    }
}

template <bool WHOLE>  // WHOLE: K % 8 == 0, every 16-byte piece of a row is inside it or outside
__global__ __launch_bounds__(256, 2) void hessian_kernel(HessArgs a)
{
    __shared__ __attribute__((aligned(16))) float S[kT * kPitch];  // two stages of two [64][128] bf16 operands, then the fp32 tile
    static_assert(sizeof(S) >= 2 * 2 * kRows * kT * 2, "stages fit");
    char* const lds = reinterpret_cast<char*>(S);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of the full tiles
    int p = blockIdx.x, part = -1;
    if (p < a.full) {
        const int per = a.full >> 3, more = a.full & 7, xcd = p & 7;
        p = xcd * per + min(xcd, more) + (p >> 3);
    } else {
        part = (p - a.full) % a.parts;
        p = a.full + (p - a.full) / a.parts;
    }
    int ti, tj;
    tile_of(p, a.nt, ti, tj);
    const int64_t t_begin = part < 0 ? 0 : (int64_t)part * a.chunk;
    const int64_t t_end = part < 0 ? a.T : min(a.T, t_begin + a.chunk);
    const bool diag = ti == tj;
    const int r0 = ti * kT, c0 = tj * kT;

    // staging: thread -> 16-byte piece tid % 16 of rows tid / 16 + 16 i of either operand
    const int piece = tid & 15, trow = tid >> 4;
    uint4 ra[4], rb[4];
    auto load = [&](int64_t t, int col) -> uint4 {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (t >= t_end) return v;
        const uint16_t* src = a.x + t * a.K + col;
        if constexpr (WHOLE) {
            if (col < a.K) v = *reinterpret_cast<const uint4*>(src);
        } else {
            uint16_t e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) e[k] = (col + k < a.K) ? src[k] : (uint16_t)0;
            v = make_uint4(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16, e[6] | (uint32_t)e[7] << 16);
        }
        return v;
    };
    auto fetch = [&](int64_t t0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ra[i] = load(t0 + trow + 16 * i, r0 + piece * 8);
        if (!diag) {
#pragma unroll
            for (int i = 0; i < 4; ++i) rb[i] = load(t0 + trow + 16 * i, c0 + piece * 8);
        }
    };
    auto stash = [&](int buf) {
        char* base = lds + buf * (2 * kRows * kT * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = trow + 16 * i;
            char* d = base + t * (kT * 2) + (((piece >> 1) ^ swz(t)) << 5) + ((piece & 1) << 4);
            *reinterpret_cast<uint4*>(d) = ra[i];
            if (!diag) *reinterpret_cast<uint4*>(d + kRows * kT * 2) = rb[i];
        }
    };

    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // a lane's share of a transposing read: row 8 (lane / 16) + (lane % 16) / 4 (+ 4), 8 bytes at column 4 (lane % 4); the lane
    // receives column lane % 16 of four rows
    const int lrow = 8 * (lane >> 4) + ((lane & 15) >> 2), lcol = (lane & 3) * 8;
    const int wa = (wave >> 1) * 4, wb = (wave & 1) * 4;  // this wave's first 16-column chunk of either operand
    const int boff = diag ? 0 : kRows * kT * 2;
    auto frag = [&](const char* base, int kb, int ib) -> v8bf {
        v4s h[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int t = kb * 32 + lrow + 4 * u;
            const char* s = base + t * (kT * 2) + ((ib ^ swz(t)) << 5) + lcol;
            h[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)s);
        }
        const v8s r = __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(v8bf, r);
    };

    fetch(t_begin);
    stash(0);
    fetch(t_begin + kRows);
    __syncthreads();
    int buf = 0;
    for (int64_t t = t_begin; t < t_end; t += kRows) {
        const char* base = lds + buf * (2 * kRows * kT * 2);
#pragma unroll
        for (int kb = 0; kb < kRows / 32; ++kb) {
            v8bf fa[4], fb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) fa[i] = frag(base, kb, wa + i);
#pragma unroll
            for (int j = 0; j < 4; ++j) fb[j] = frag(base + boff, kb, wb + j);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (t + kRows < t_end) {
            stash(buf ^ 1);
            fetch(t + 2 * kRows);
        }
        __syncthreads();
        buf ^= 1;
    }
    if (part < 0) {
        finish_tile(a, ti, tj, acc, S);
    } else {
        float* d = a.part + (int64_t)(blockIdx.x - a.full) * (kT * kT) + tid;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) d[((i * 4 + j) * 4 + v) * 256] = acc[i][j][v];
    }
}

// the split tiles: their parts added in order, then finished like the others
__global__ __launch_bounds__(256, 2) void hessian_tail_kernel(HessArgs a)
{
    __shared__ __attribute__((aligned(16))) float S[kT * kPitch];
    int ti, tj;
    tile_of(a.full + blockIdx.x, a.nt, ti, tj);
    v4f acc[4][4];
    for (int s = 0; s < a.parts; ++s) {
        const float* d = a.part + (int64_t)(blockIdx.x * a.parts + s) * (kT * kT) + threadIdx.x;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float x = d[((i * 4 + j) * 4 + v) * 256];
                    acc[i][j][v] = s ? acc[i][j][v] + x : x;
                }
    }
    finish_tile(a, ti, tj, acc, S);
}

}  // namespace

hipError_t launch_gptq_hessian(const void* x, int64_t T, int64_t K, int b, float* H, bool accumulate, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    if (T <= 0 || K <= 0 || K > 24576) return hipErrorInvalidValue;
    HessArgs a{};
    a.x = static_cast<const uint16_t*>(x);
    a.H = H;
    a.part = static_cast<float*>(workspace);
    a.T = T;
    a.K = (int)K;
    a.b = b;
    a.accumulate = accumulate ? 1 : 0;
    a.inv_b = 1.0f / (float)b;
    a.nt = (int)((K + kT - 1) / kT);
    const int tiles = a.nt * (a.nt + 1) / 2, slots = 2 * compute_units();
    // Two workgroups per compute unit work at a time.  The tiles beyond whole rounds of those would run on a mostly idle
    // chip for a whole tile's time (K = 4096: 528 tiles for 512 slots), so T is cut into parts for them, of at least 512
    // rows (less does not repay the second launch), as many as fit the round and the caller's workspace.
    const int rem = tiles % slots;
    int parts = rem ? std::min({slots / rem, 8, (int)std::min<int64_t>(T / 512, 8)}) : 1;
    if (rem) parts = std::min(parts, (int)std::min<int64_t>(8, (int64_t)(workspace_bytes / ((size_t)rem * kT * kT * 4))));
    a.full = tiles;
    a.parts = 1;
    a.chunk = 0;
    int tail = 0;
    if (parts > 1) {
        a.chunk = (int)(((T + parts - 1) / parts + kRows - 1) / kRows * kRows);
        a.parts = (int)((T + a.chunk - 1) / a.chunk);
        a.full = tiles - rem;
        tail = rem;
    }
    const dim3 grid((unsigned)(a.full + tail * a.parts));
    if (K % 8 == 0) hipLaunchKernelGGL(hessian_kernel<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(hessian_kernel<false>, grid, dim3(256), 0, st, a);
    if (tail) hipLaunchKernelGGL(hessian_tail_kernel, dim3((unsigned)tail), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace fp4mr
