// Hessian of a layer from calibration rows (arXiv 2509.23202, Section 4 "Standard GPTQ": the second-order information of
// ||X What - X W||^2 is X^T X; Section 4.1 "Ingredient 3": of the ROTATED inputs X H_b).
//
// The rows are rotated FIRST and every rotated value is kept to 24 bits (few rows) or 23, so that an entry's error is relative to
// sqrt(h_ii h_jj) of its own two channels.  (Rotating the finished X^T X is faster, but where channels of a block have
// something in common most rotated channels are small differences of large sums: with an offset of 100 under unit noise
// the entries were off by 1 % of that scale, and diagonal entries could come out negative.)
//   many rows  hessian_pack_kernel   X -> the rotated rows as two fp16 parts, scaled by column, in the workspace as the MFMA takes them
//              hessian_tile_kernel   X'^T X' on the fp16 MFMA, a tile to a workgroup: the three products above 2^-23 of the whole
//              hessian_pair_kernel   the same, two tiles to a workgroup, from 2048 or 4096 rows on where they fill the chip (the rule stands at the launch)
//              hessian_part_kernel   the same for the tiles beyond whole rounds of the chip
//   few rows   hessian_rotate_kernel X -> the rotated rows in fp32, in the workspace, eight rows of a column side by side
//              hessian_split_kernel  X'^T X' on the bf16 MFMA, both factors split into three bf16 parts: the six products above
//                                    2^-24 of the whole
// 8192 rows at K = 4096: 0.39 - 0.42 ms (0.86 with six bf16 products, 4.15 on the fp32 MFMA over both triangles).  Largest error over
// sqrt(h_ii h_jj), T = 8192, b = 128, K = 1024 / 4096, bf16 -> fp16: normal rows with loud channels 9.3e-7 / 1.0e-6 -> 2.0e-7 / 5.6e-7, offset
// 30 9.5e-7 / 8.9e-7 -> 1.2e-7 / 4.6e-7, offset 100 6.2e-7 / 7.6e-7 -> 1.0e-7 / 3.6e-7, a channel of every 64th row 3000 times as large
// 9.2e-7 / 1.0e-6 -> 3.0e-7 / 5.2e-7 (for adding up four sums of 32 rows before they meet the large one).  Of one row alone, with nothing to
// add up, 1.1e-7 -> 3.3e-7.
// Without rotation (b == 1) the values are bf16 and their products exact in fp32: hessian_kernel, straight from X.
// The matrix is symmetric: only tiles on and below the diagonal are computed, each is stored twice.
#include "device_util.hpp"
#include "internal.hpp"
#include "pair16.hpp"

#include <algorithm>
#include <type_traits>

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
    float* xr;          // b > 1, few rows: the rotated rows, packed (packed_at)
    char* planes;       // b > 1, many rows: the stages of 32 rotated rows (see there), one behind the other ...
    uint8_t* exps;      // ... and the exponents of their columns, [group of stages][K]
    int stages;         // of them (the rows behind are rotated by every workgroup for itself)
    float* part;        // b == 1: partial tiles of the split tail
    int64_t T;
    int K, b, accumulate;
    int nt;             // tiles per side
    int full;           // tiles (pairs: b > 1, many rows) 0 .. full - 1 take all of T in one workgroup ...
    bool pairs;
    int parts;          // ... each of the others is shared by this many
    int chunk;          // rows of X per part (multiple of kRows)
    float in_scale, out_scale;  // powers of two: in_scale^2 * out_scale = 1 / b (few rows)
    int row_step;       // b > 1, many rows: kPairRow, and the exponent of b
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

// the finished sums of tile (ti, tj), in the MFMA's output order, stored with their mirror image
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
    const int r0 = ti * kT, c0 = tj * kT;
    const int c = tid & (kT - 1), r1 = tid >> 7;  // a wave stores 64 consecutive floats
    const bool diag = ti == tj;
    for (int side = 0; side < (diag ? 1 : 2); ++side) {
        const int row0 = side ? c0 : r0, col0 = side ? r0 : c0;
        if (col0 + c >= a.K) continue;
#pragma unroll 4
        for (int r = r1; r < kT; r += 2) {
            if (row0 + r >= a.K) break;
            const bool swap = side || (diag && c > r);  // (on the diagonal both halves take the lower one's values)
            const float s = swap ? S[c * kPitch + r] : S[r * kPitch + c];
            float* p = a.H + (int64_t)(row0 + r) * a.K + col0 + c;
            *p = a.accumulate ? *p + s : s;
        }
    }
}

// ---------------------------------------------------------------- b == 1: bf16 values, exact products
// Bound: LDS bandwidth (a 64 x 64 wave tile reads 16 KB per 32 MFMAs), then the L2.  Tile 128 x 128 over 64 rows of X at a
// time, four waves, two workgroups per compute unit (64.5 KB of LDS) so that one's staging runs under the other's MFMAs.
// X is staged as it lies in memory, rows along the contraction; the MFMA operands want the contraction along a lane's
// registers, which the transposing LDS read (ds_read_b64_tr_b16) provides: no transposed copy in memory, no packing.
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

// ---------------------------------------------------------------- b > 1, few rows

// Where element (t, column) of the rotated rows lies: eight rows of a column side by side (what a lane of the bf16 MFMA takes
// of the contraction), columns behind each other; a last group of fewer rows is packed, so that T K floats hold it all.
__device__ __forceinline__ int64_t packed_at(const HessArgs& a, int64_t group, int col, int rows) { return group * 8 * a.K + (int64_t)col * rows; }

// Sixteen neighbouring columns of row t per thread, rotated in registers -- butterflies, the levels above sixteen across lanes, fp32
// sums of up to 128 bf16 values.  Columns go with the lanes; rows and columns that do not exist are zero.
__device__ __forceinline__ void rotate_row(const HessArgs& a, int64_t t, int c, float (&v)[16])
{
    const int levels = a.b == 16 ? 0 : (a.b == 32 ? 1 : a.b == 64 ? 2 : 3);
    uint4 lo = make_uint4(0u, 0u, 0u, 0u), hi = lo;
    if (t < a.T && c < a.K) {  // (K is a multiple of b: lanes that exchange values are in or out of the row together)
        const uint4* src = reinterpret_cast<const uint4*>(a.x + t * a.K + c);
        lo = src[0];
        hi = src[1];
    }
    const uint32_t raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[2 * i] = __uint_as_float(raw[i] << 16);
        v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
    }
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
}

// Eight rows by 512 columns per workgroup.  A thread rotates sixteen neighbouring columns of a row in registers -- butterflies, the
// levels above sixteen across lanes, fp32 sums of up to 128 bf16 values -- and the power of two nearest below sqrt(b) is
// divided out, exactly; what is left of 1 / b (a half at b = 32 and 128) is multiplied onto the finished sums.
constexpr int kRotCols = 512;
__global__ __launch_bounds__(256) void hessian_rotate_kernel(HessArgs a)
{
    __shared__ __attribute__((aligned(16))) float S[kRotCols * 8 + kRotCols / 16 * 8];  // [column][row]; eight floats more every sixteen columns (banks)
    const int tid = threadIdx.x, r = tid >> 5, piece = tid & 31;
    const int c0 = blockIdx.y * kRotCols, cols = min(kRotCols, a.K - c0);
    const int64_t group = blockIdx.x;
    const int rows = (int)min((int64_t)8, a.T - group * 8);
    float v[16];
    rotate_row(a, r < rows ? group * 8 + r : a.T, piece * 16 < cols ? c0 + piece * 16 : a.K, v);
#pragma unroll
    for (int i = 0; i < 16; ++i) S[(piece * 16 + i) * 8 + piece * 8 + r] = v[i] * a.in_scale;
    __syncthreads();
    float* const dst = a.xr + packed_at(a, group, c0, rows);
    if (rows == 8) {
        for (int i = tid; i < cols * 2; i += 256)
            reinterpret_cast<float4*>(dst)[i] = *reinterpret_cast<const float4*>(&S[i * 4 + (i >> 5) * 8]);
    } else {
        for (int i = tid; i < cols * rows; i += 256) {
            const int c = i / rows;
            dst[i] = S[c * 8 + (c >> 4) * 8 + i - c * rows];
        }
    }
}

// 16 x 16 sums in the MFMA's output order -- a lane holds columns col .. col + 3 of a row -- stored with their mirror image; of a
// block on the diagonal the lower half counts (K is a multiple of 16)
__device__ __forceinline__ void store_block(const HessArgs& a, int row, int col, bool cut, v4f s)
{
    if (row >= a.K || col >= a.K) return;
    float* const own = a.H + (int64_t)row * a.K + col;
    float* const mirror = a.H + (int64_t)col * a.K + row;
    if (!cut) {
        v4f* const d = reinterpret_cast<v4f*>(own);
        *d = a.accumulate ? *d + s : s;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (cut && col + v <= row) own[v] = a.accumulate ? own[v] + s[v] : s[v];
        float* const m = mirror + (int64_t)v * a.K;
        if (!cut || col + v < row) *m = a.accumulate ? *m + s[v] : s[v];
    }
}

// A tile of 2 W x 2 W, a W x W quarter per wave, 32 rows of X' at a time: split and written to LDS in the MFMA's operand order
// (lane (r, q) of a 16-wide block: column r, rows 8 q .. 8 q + 7), the next 32 rows fetched meanwhile.  The products of 32 rows
// are summed from zero, the largest apart from the five others (the MFMA cuts off what an addition leaves over, the vector
// adder rounds), and added to the accumulator once.  The column operand is the MFMA's A, so that a lane
// owns four neighbouring columns of a row of H.
// Bound at W = 64: a wave issues 96 MFMAs (1536 cycles) and 370 vector instructions (1480, half of them the split) per stage, and
// two workgroups per compute unit overlap the two in part: 512 tiles over 1099 rows 127 us, 0.87 PFLOP/s.
template <int W>
__global__ __launch_bounds__(256, 2) void hessian_split_kernel(HessArgs a)
{
    constexpr int NT = W / 16, BL = 2 * NT, PER = BL / 2;   // 16-wide blocks per wave side, per operand, and staged per wave
    constexpr int AHEAD = W == 64 ? 1 : 4;                  // stages on their way (a small tile's is shorter than a load takes)
    constexpr int BUFS = W == 64 ? 1 : 2;                   // stages in LDS
    constexpr int SUB = 64 / W;
    __shared__ v8bf St[BUFS][3][2 * BL][64];                 // [part][block of 16 rows, then columns, of the tile][lane]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of the tiles
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7;
    const int p = xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3);
    int ti, tj;
    tile_of((SUB > 1 ? a.full : 0) + p / (SUB * SUB), a.nt, ti, tj);
    if constexpr (SUB > 1) {   // a part of one of the tiles that are left
        ti = SUB * ti + p / SUB % SUB;
        tj = SUB * tj + p % SUB;
        if (tj > ti || ti * 2 * W >= a.K) return;
    }
    const bool diag = ti == tj;
    const int r0 = ti * 2 * W, c0 = tj * 2 * W;
    const int wr = (wave >> 1) * NT, wc = (wave & 1) * NT;   // first block of rows / columns of the wave's quarter
    const bool idle = diag && wr < wc;                       // (above the diagonal)

    // This wave stages the blocks wave, wave + 4, ... of the 2 BL.  Every request is unconditional (the compiler's waits count on
    // it): what does not exist is requested with zero size and reads as zero.  (Columns past the end: the last one again,
    // it only feeds outputs that are not stored.  A diagonal tile takes its rows for both.)
    float ahead[AHEAD][PER][8];
    const int64_t stages = a.T / 32;
    int col[PER];
#pragma unroll
    for (int h = 0; h < PER; ++h) {
        const int block = wave + 4 * h;
        col[h] = min((block < BL ? r0 + block * 16 : c0 + (block - BL) * 16) + l16, a.K - 1);
    }
    auto fetch = [&](int64_t s, float (&v)[PER][8]) {
        const bool valid = s < stages;
        float* const base = a.xr + (valid ? s : 0) * 32 * a.K;
#pragma unroll
        for (int h = 0; h < PER; ++h) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, valid && !(diag && wave + 4 * h >= BL) ? 128 * a.K : 0, 0x00020000);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const v4f x = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs, (q * a.K + col[h]) * 32, half * 16, 0));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[h][half * 4 + i] = x[i];
            }
        }
    };
    // the last T % 32 rows, the rest of the stage zero
    auto fetch_rest = [&](float (&v)[PER][8]) {
        const int64_t last = (a.T - 1) / 8, group = stages * 4 + q, g = min(group, last);
        const int rows = (int)min((int64_t)8, a.T - g * 8);
#pragma unroll
        for (int h = 0; h < PER; ++h) {
            const float* src = a.xr + packed_at(a, g, col[h], rows);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = src[min(i, rows - 1)];
                v[h][i] = group == g && i < rows ? x : 0.0f;
            }
        }
    };
    v4f acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int wcol = diag ? wc : BL + wc;
    auto put = [&](const float (&v)[PER][8], int buf) {
#pragma unroll
        for (int h = 0; h < PER; ++h) {
            const Split3 x = split3(v[h]);
#pragma unroll
            for (int k = 0; k < 3; ++k) St[buf][k][wave + 4 * h][lane] = x.part[k];
        }
    };
    auto multiply = [&](int buf) {
        v8bf u[3][NT];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < NT; ++j) u[k][j] = St[buf][k][wcol + j][lane];
        v8bf next[3];   // row operands, one block ahead
#pragma unroll
        for (int k = 0; k < 3; ++k) next[k] = St[buf][k][wr][lane];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            v8bf e[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) e[k] = next[k];
            if (i + 1 < NT) {
#pragma unroll
                for (int k = 0; k < 3; ++k) next[k] = St[buf][k][wr + i + 1][lane];
            }
            __builtin_amdgcn_sched_barrier(0);
            // (part of the column, part of the row): 2^-16, 2^-8 of the product, then 1
            constexpr int order[6][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
            v4f low[NT], high[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) low[j] = high[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 6; ++s)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    v4f& d = s < 5 ? low[j] : high[j];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[order[s][0]][j], e[order[s][1]], d, 0, 0, 0);
                }
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] += high[j] + low[j];
        }
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) fetch(d, ahead[d]);
    if constexpr (BUFS == 1) {
        for (int64_t s = 0; s < stages; ++s) {
            __syncthreads();
            put(ahead[0], 0);
            __syncthreads();
            fetch(s + 1, ahead[0]);
            multiply(0);
        }
    } else {
        // the next stage is split under the products of this one; one barrier each: a stage overwrites what was read before the last
        put(ahead[0], 0);
        fetch(AHEAD, ahead[0]);
        for (int64_t s = 0; s < stages; s += AHEAD) {   // (up to AHEAD - 1 stages of zeros behind the last)
#pragma unroll
            for (int d = 0; d < AHEAD; ++d) {
                __syncthreads();
                put(ahead[(d + 1) % AHEAD], (d + 1) % 2);
                fetch(s + d + 1 + AHEAD, ahead[(d + 1) % AHEAD]);
                multiply(d % 2);
            }
        }
    }
    if (a.T % 32) {
        fetch_rest(ahead[0]);
        __syncthreads();
        put(ahead[0], 0);
        __syncthreads();
        multiply(0);
    }
    if (idle) return;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (!diag || wr + i >= wc + j)
                store_block(a, r0 + (wr + i) * 16 + l16, c0 + (wc + j) * 16 + 4 * q, diag && wr + i == wc + j, acc[i][j] * a.out_scale);
}

// ---------------------------------------------------------------- b > 1, many rows

// The rotated rows X' are kept as scaled pairs of halves (pair16.hpp), an exponent for every column and GROUP of four stages: what is
// left out of a value is relative to the largest value of its own channel, however loud the channels beside it are.
constexpr int kGroup = 4;           // stages that share their exponents

// The exponents, a byte each, of 128 columns from the largest values of every thread's sixteen.  The eight lanes of a wave that share
// columns halve them among themselves step by step, then the four waves meet in LDS.
__device__ __forceinline__ void column_exponents(const float (&top)[16], float (*red)[kT], uint8_t* exps)
{
    const int tid = threadIdx.x & 255, piece = tid & 7;
    float m8[8], m4[4], m2[2];
    const bool b3 = tid & 8, b4 = tid & 16, b5 = tid & 32;
#pragma unroll
    for (int i = 0; i < 8; ++i) m8[i] = fmaxf(b3 ? top[i + 8] : top[i], __shfl_xor(b3 ? top[i] : top[i + 8], 8));
#pragma unroll
    for (int i = 0; i < 4; ++i) m4[i] = fmaxf(b4 ? m8[i + 4] : m8[i], __shfl_xor(b4 ? m8[i] : m8[i + 4], 16));
#pragma unroll
    for (int i = 0; i < 2; ++i) m2[i] = fmaxf(b5 ? m4[i + 2] : m4[i], __shfl_xor(b5 ? m4[i] : m4[i + 2], 32));
    *reinterpret_cast<float2*>(&red[tid >> 6][piece * 16 + (b3 ? 8 : 0) + (b4 ? 4 : 0) + (b5 ? 2 : 0)]) = make_float2(m2[0], m2[1]);
    __syncthreads();
    if (tid < kT) exps[tid] = (uint8_t)pair_exponent(fmaxf(fmaxf(red[0][tid], red[1][tid]), fmaxf(red[2][tid], red[3][tid])));
    __syncthreads();
}

// the factors of a thread's sixteen columns
__device__ __forceinline__ void column_ups(const uint8_t* exps, float (&up)[16])
{
    const uint4 w = *reinterpret_cast<const uint4*>(exps + (threadIdx.x & 7) * 16);
    const uint32_t e[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 16; ++i) up[i] = pair_up(e[i >> 2] >> 8 * (i & 3) & 255u);
}

// pair_column of four exponents (14 at least: none borrows)
__device__ __forceinline__ v4f four_column_factors(uint32_t exps)
{
    const uint32_t w = exps - 0x01010101u;
    return v4f{__uint_as_float((w & 255u) << 23), __uint_as_float((w >> 8 & 255u) << 23), __uint_as_float((w >> 16 & 255u) << 23), __uint_as_float((w >> 24) << 23)};
}

// what a lane needs of the exponents of 128 rows and 128 columns at `exps`: of row l16 of a block, of columns 4 q .. 4 q + 3 of a block
__device__ __forceinline__ int row_exponent(const uint8_t* exps, int block) { return exps[block * 16 + (threadIdx.x & 15)]; }
__device__ __forceinline__ v4f col_factors(const uint8_t* exps, int block)
{
    return four_column_factors(*reinterpret_cast<const uint32_t*>(exps + block * 16 + 4 * (threadIdx.x >> 4 & 3)));
}

// a thread's sixteen values into the stage at dst, its blocks `pitch` bytes apart
__device__ __forceinline__ void put_row(const float (&v)[16], const float (&up)[16], char* dst, int pitch)
{
    const int r = threadIdx.x >> 3 & 31, piece = threadIdx.x & 7;
    _Float16* out = reinterpret_cast<_Float16*>(dst + piece * pitch) + (r >> 3) * 128 + (r & 7);
#pragma unroll
    for (int i = 0; i < 16; ++i) pair_split(v[i], up[i], out[i * 8], out[i * 8 + 512]);
}

// the stages that the workspace holds; a workgroup writes a group of them, 128 columns wide.  Bound: HBM, 2 bytes a value read
// and 4 written.
__global__ __launch_bounds__(256) void hessian_pack_kernel(HessArgs a)
{
    constexpr int kPad = kPairBytes + 16;   // (a row's eight pieces write to different banks)
    __shared__ __attribute__((aligned(16))) char S[8 * kPad];
    __shared__ __attribute__((aligned(16))) float red[4][kT];
    __shared__ __attribute__((aligned(16))) uint8_t exps[kT];
    const int tid = threadIdx.x, c0 = blockIdx.y * kT, blocks = min(kT, a.K - c0) / 16;
    const int s0 = blockIdx.x * kGroup, count = min(kGroup, a.stages - s0);
    float v[kGroup][16], top[16] = {}, up[16];
#pragma unroll
    for (int g = 0; g < kGroup; ++g) {
        rotate_row(a, g < count ? (int64_t)(s0 + g) * 32 + (tid >> 3) : a.T, c0 + (tid & 7) * 16, v[g]);
#pragma unroll
        for (int i = 0; i < 16; ++i) top[i] = fabs_max(top[i], v[g][i]);
    }
    column_exponents(top, red, exps);
    column_ups(exps, up);
    if (tid < blocks * 16) a.exps[(int64_t)blockIdx.x * a.K + c0 + tid] = exps[tid];
#pragma unroll
    for (int g = 0; g < kGroup; ++g) {
        if (g >= count) break;
        put_row(v[g], up, S, kPad);
        __syncthreads();
        uint4* const dst = reinterpret_cast<uint4*>(a.planes + (int64_t)(s0 + g) * 128 * a.K + c0 * 128);
        for (int i = tid; i < blocks * (kPairBytes / 16); i += 256)
            dst[i] = *reinterpret_cast<const uint4*>(S + (i >> 7) * kPad + (i & 127) * 16);
        __syncthreads();
    }
}

// the stage that begins with row t, of the 128 columns from c0, in LDS: for rows that the workspace has no room for
__device__ __forceinline__ void build_stage(const HessArgs& a, int64_t t, int c0, char* dst, uint8_t* exps, float (*red)[kT])
{
    float v[16], top[16], up[16];
    rotate_row(a, t + (threadIdx.x >> 3 & 31), c0 + (threadIdx.x & 7) * 16, v);
#pragma unroll
    for (int i = 0; i < 16; ++i) top[i] = fabsf(v[i]);
    column_exponents(top, red, exps);
    column_ups(exps, up);
    put_row(v, up, dst, kPairBytes);
}

// A tile of 128 x 128, a 64 x 64 quarter per wave, a stage at a time, copied into LDS as it lies in the workspace, the next one
// meanwhile.  Two workgroups per compute unit, so that one's barrier and LDS reads run under the
// other's MFMAs.  Bound at K = 4096, 512 tiles over 8192 rows, some 390 us (375 with an exponent for sixteen columns, of
// which without the copies into LDS 305): at the 1.6 PFLOP/s of a large bf16 product 257.  (Operands of the next stage read into registers ahead of its barrier: 3 % slower.)
constexpr int kTile = 4, kTileStage = 16 * kPairBytes, kTileLds = 2 * (kTileStage + 1024);   // 16-wide blocks per wave side; stages and their exponents
__global__ __launch_bounds__(256, 2) void hessian_tile_kernel(HessArgs a)
{
    constexpr int NT = kTile, STAGE = kTileStage;
    // two stages; per stage and wave the exponents of 128 rows and of 128 columns
    extern __shared__ __attribute__((aligned(1024))) char St[];
    uint8_t* const Sc = reinterpret_cast<uint8_t*>(St + 2 * STAGE);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of the tiles
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7;
    int ti, tj;
    tile_of(xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3), a.nt, ti, tj);
    const bool diag = ti == tj;
    const int r0 = ti * kT, c0 = tj * kT;
    const int wr = (wave >> 1) * NT, wc = (wave & 1) * NT;   // first block of rows / columns of the wave's quarter

    // Blocks past the end are the last one again: they only feed outputs that are not stored.  Past the last stage the copies
    // repeat it into a slot that nobody reads any more.
    const int kb = a.K / 16, stages = a.stages;
    const uint32_t exps_at = (uint32_t)min((lane < 32 ? r0 : c0) + 4 * (lane & 31), a.K - 4);
    auto issue = [&](int s) {
        const int from = min(s, stages - 1), slot = s & 1;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(a.planes + (int64_t)from * 128 * a.K, 0, 128 * a.K, 0x00020000);
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(a.exps + (int64_t)(from / kGroup) * a.K, 0, a.K, 0x00020000);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = wave * 8 + i;                      // 1 KB: half a block
            const int block = (c < 16 ? r0 : c0) / 16 + (c & 15) / 2;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(St + slot * STAGE + c * 1024), 16, lane * 16, min(block, kb - 1) * kPairBytes + (c & 1) * 1024, 0, 0);
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, (lds_void*)(Sc + (slot * 4 + wave) * 256), 4, exps_at, 0, 0, 0);
    };
    PairSums<NT> sums;
    sums.clear();
    auto scale_sums = [&](const uint8_t* exps) {
        sums.scale([&](int i) { return row_exponent(exps, wr + i) - a.row_step; }, [&](int j) { return col_factors(exps + kT, wc + j); });
    };
    if (stages > 0) {
        issue(0);
        for (int s = 0; s < stages; ++s) {
            wait_vmcnt<0>();
            wait_lgkmcnt0();
            block_barrier();   // stage s has landed, stage s - 1 has been read
            issue(s + 1);
            const char* base = St + (s & 1) * STAGE;
            if (s % kGroup == 0) sums.multiply<true>(base + wr * kPairBytes, base + (8 + wc) * kPairBytes);
            else sums.multiply<false>(base + wr * kPairBytes, base + (8 + wc) * kPairBytes);
            if ((s + 1) % kGroup == 0 || s + 1 == stages) {
                scale_sums(Sc + ((s & 1) * 4 + wave) * 256);
            }
        }
        wait_vmcnt<0>();
    }
    float(*const red)[kT] = reinterpret_cast<float(*)[kT]>(St + STAGE);
    for (int64_t row = (int64_t)stages * 32; row < a.T; row += 32) {
        __syncthreads();
        build_stage(a, row, r0, St, Sc, red);
        build_stage(a, row, c0, St + 8 * kPairBytes, Sc + kT, red);
        __syncthreads();
        sums.multiply<true>(St + wr * kPairBytes, St + (8 + wc) * kPairBytes);
        scale_sums(Sc);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (!diag || wr + i >= wc + j)
                store_block(a, r0 + (wr + i) * 16 + l16, c0 + (wc + j) * 16 + 4 * q, diag && wr + i == wc + j, sums.acc[i][j]);
}

// Row and column of the p-th pair of tiles (2 row, col) and (2 row + 1, col), col <= 2 row.  Four rows of pairs, then the next four, column by column:
// what runs on an XCD at a time shares its operands through one L2.
__device__ __forceinline__ void pair_of(int p, int rows, int& row, int& col)
{
    int R = 0;
    while (16 * (R + 1) * (R + 1) <= p) ++R;   // (at most rows / 4 scalar trips: 4 R rows hold (4 R)^2 pairs)
    p -= 16 * R * R;
    int h = min(4, rows - 4 * R);
    row = 4 * R;
    col = 8 * R + 1;
    if (p < h * col) {
        col = p / h;
        row += p % h;
        return;
    }
    p -= h * col;
    for (;;) {   // two columns each that one row less reaches
        --h;
        ++row;
        if (p < 2 * h) break;
        p -= 2 * h;
        col += 2;
    }
    col += p / h;
    row += p % h;
}

// Two tiles of 128 x 128, one below the other, a stage at a time, copied into LDS as it lies in the workspace: four waves multiply the upper
// one, in quarters of 64 x 64, four the lower one, in turn (pair_alternate).  48 KB are copied for what takes the tiles by themselves 64, and the
// matrix cores work 1540 of some 2250 cycles a stage, there 1540 of 2900.  Bound: the phases of a group's first stage (its exponents and steps are
// 150 vector instructions, which share a SIMD's issue with the other wave's MFMAs: 1400 cycles, the others 900) and the clock, 1.85 GHz
// under this load.  The products 8192 rows, K = 4096: 390 -> 310 us.
constexpr int kPairStage = 24 * kPairBytes;   // 16-wide blocks per wave side; a stage: 16 blocks of rows, 8 of columns
constexpr int kPairLds = 3 * kPairStage + 4 * 8 * 256;   // three stages, the exponents of four
__global__ __launch_bounds__(512, 2) void hessian_pair_kernel(HessArgs a)
{
    constexpr int NT = kTile, STAGE = kPairStage;
    extern __shared__ __attribute__((aligned(1024))) char St[];
    uint8_t* const Sc = reinterpret_cast<uint8_t*>(St + 3 * STAGE);   // [stage % 4][wave]: of its four's 128 rows, of 128 columns
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), four = wave >> 2;
    // workgroups are handed to the XCDs in turn: XCD x takes a contiguous run of the pairs
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7;
    int ti, tj;
    pair_of(xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3), a.nt / 2, ti, tj);
    const bool diag = 2 * ti + four == tj;
    const int r0 = ti * 2 * kT, c0 = tj * kT;
    const int wr = (wave >> 1 & 1) * NT, wc = (wave & 1) * NT;   // first block of rows / columns of the wave's quarter

    // Blocks past the end are the last one again: they only feed outputs that are not stored.  Stages past the end are zero.
    const int kb = a.K / 16, stages = a.stages;
    const uint32_t exps_at = (uint32_t)min((lane < 32 ? r0 + four * kT : c0) + 4 * (lane & 31), a.K - 4);
    auto exps_of = [&](int n) { return Sc + ((n & 3) * 8 + wave) * 256; };
    auto issue = [&](int n, auto between) {
        const int from = min(n, stages - 1);
        const uint32_t at = n < stages ? (uint32_t)lane * 16u : 0xfffff000u;
        char* const slot = St + n % 3 * STAGE;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(a.planes + (int64_t)from * 128 * a.K, 0, 128 * a.K, 0x00020000);
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(a.exps + (int64_t)(from / kGroup) * a.K, 0, a.K, 0x00020000);
        each<6>([&](auto i) {
            const int c = wave * 6 + i;   // 1 KB: half a block
            const int block = c < 32 ? r0 / 16 + c / 2 : c0 / 16 + c / 2 - 16;
            copy_to_lds(rs, slot + c * 1024, at, min(block, kb - 1) * kPairBytes + (c & 1) * 1024);
            between(i);
        });
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, (lds_void*)exps_of(n), 4, exps_at, 0, 0, 0);
    };
    PairChain<NT> sums;
    sums.clear();
    PairOperands<NT> held;
    // a group's exponents: of a lane's four rows, of its sixteen columns
    uint32_t row_exps[NT], col_exps[NT];
    auto read_exps = [&](const uint8_t* from) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            row_exps[i] = from[(wr + i) * 16 + l16];
            col_exps[i] = *reinterpret_cast<const uint32_t*>(from + kT + (wc + i) * 16 + 4 * q);
        }
    };
    auto row = [&](int i) { return (int)row_exps[i] - a.row_step; };
    auto col = [&](int j) { return four_column_factors(col_exps[j]); };
    if (stages > 0) {
        const int groups = (stages + kGroup - 1) / kGroup;
        pair_alternate<7, kGroup>(four, groups, issue,
            [&](auto part) { sums.template begin<part.value>(row, col); },
            [&](int n, auto i) {
                if (i.value == 0) read_exps(exps_of(max(n - 1, 0)));
                const char* base = St + n % 3 * STAGE;
                held.fetch(base + (four * 8 + wr) * kPairBytes, base + (16 + wc) * kPairBytes);
            },
            [&](auto i) { sums.template multiply<i.value == 0, (i.value > 1)>(held); });
        read_exps(exps_of(groups * kGroup - 1));
        sums.end(row, col);
    }
    // rows that the workspace has no room for, 32 at a time: either four its rows, and both the columns
    float(*const red)[kT] = reinterpret_cast<float(*)[kT]>(St + STAGE + four * 4 * kT * 4);
    uint8_t* const ex = Sc + four * 2 * kT;
    for (int64_t row0 = (int64_t)stages * 32; row0 < a.T; row0 += 32) {
        __syncthreads();
        build_stage(a, row0, r0 + four * kT, St + four * 8 * kPairBytes, ex, red);
        build_stage(a, row0, c0, St + 16 * kPairBytes, ex + kT, red);
        __syncthreads();
        held.fetch(St + (four * 8 + wr) * kPairBytes, St + (16 + wc) * kPairBytes);
        read_exps(ex);
        sums.restart();
        each<sums.kBegin>([&](auto part) { sums.template begin<part.value>(row, col); });
        sums.template multiply<true, false>(held);
        sums.end(row, col);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (!diag || wr + i >= wc + j)
                store_block(a, r0 + four * kT + (wr + i) * 16 + l16, c0 + (wc + j) * 16 + 4 * q, diag && wr + i == wc + j, sums.acc[i][j]);
}

// The p-th of the tiles that are left: those from `full` on or, of pairs, every other one of the diagonal, the last row if it has no partner,
// and the pairs from `full` on.
__device__ __forceinline__ void left_tile(const HessArgs& a, int p, int& ti, int& tj)
{
    if (!a.pairs) {
        tile_of(a.full + p, a.nt, ti, tj);
        return;
    }
    const int rows = a.nt / 2;
    if (p < rows) {
        ti = tj = 2 * p + 1;
        return;
    }
    p -= rows;
    if (a.nt & 1) {
        if (p < a.nt) {
            ti = a.nt - 1;
            tj = p;
            return;
        }
        p -= a.nt;
    }
    pair_of(a.full + p / 2, rows, ti, tj);
    ti = 2 * ti + (p & 1);
}

// A tile of 16 NT x 16 NT, for what is left beyond whole rounds of the tiles above: each of the four waves takes a quarter of the
// groups for itself, straight from memory to registers, no barrier; then their sums are added.  32 x 32: a group ahead.  64 x 64, half the
// bytes per product: a register is refilled behind its last use, and two workgroups per compute unit cover for each other.
template <int NT>
__global__ __launch_bounds__(256, 2) void hessian_part_kernel(HessArgs a)
{
    constexpr int SIDE = 16 * NT, SUB = kT / SIDE;
    __shared__ __attribute__((aligned(16))) char St[16 * kPairBytes];   // the stages rotated on the spot, then the waves' sums
    __shared__ __attribute__((aligned(16))) uint8_t Sc[2 * kT], Ex[4][2 * kT];   // exponents of rows and columns: of a stage rotated on the spot; a wave's group
    __shared__ __attribute__((aligned(16))) float red[4][kT];
    static_assert(sizeof(St) >= 4 * 2 * NT * 64 * sizeof(v4f), "two rows of blocks of the sums fit");
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int n = (int)gridDim.x, per = n >> 3, more = n & 7, xcd = blockIdx.x & 7;
    const int p = xcd * per + min(xcd, more) + ((int)blockIdx.x >> 3);
    int ti, tj;
    left_tile(a, p / (SUB * SUB), ti, tj);
    ti = SUB * ti + p / SUB % SUB;
    tj = SUB * tj + p % SUB;
    if (tj > ti || ti * SIDE >= a.K) return;
    const int r0 = ti * SIDE, c0 = tj * SIDE, kb = a.K / 16;
    const int groups = (a.stages + kGroup - 1) / kGroup, share = (groups + 3) / 4;
    const int g_begin = wave * share, g_end = min(groups, g_begin + share);
    const uint32_t exps_at = (uint32_t)min((lane < 32 ? r0 : c0) + 4 * (lane & 31), a.K - 4);

    PairSums<NT> sums;
    sums.clear();
    constexpr int AHEAD = NT == 2 ? kGroup : 1;
    v8h rows[AHEAD][2][NT], cols[AHEAD][2][NT];   // (blocks past the end: the last one again, for outputs that are not stored)
    auto fetch = [&](int s, int k, int block) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(a.planes + (int64_t)min(s, a.stages - 1) * 128 * a.K, 0, 128 * a.K, 0x00020000);
        return __builtin_bit_cast(v8h, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, min(block, kb - 1) * kPairBytes + k * 1024, 0));
    };
    auto fetch_row = [&](int s, int d, int k, int i) { rows[d][k][i] = fetch(s, k, r0 / 16 + i); };
    auto fetch_col = [&](int s, int d, int k, int j) { cols[d][k][j] = fetch(s, k, c0 / 16 + j); };
    // one stage, the first of its group or not, from registers d; next >= 0: that stage takes their place
    constexpr std::true_type first;
    constexpr std::false_type later;
    auto multiply = [&](auto first, int d, int next) {
        constexpr bool FIRST = decltype(first)::value;
        v4f sum[2][NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    v4f& x = sum[i & 1][j];
                    x = __builtin_amdgcn_mfma_f32_16x16x32_f16(cols[d][kPairParts[s][0]][j], rows[d][kPairParts[s][1]][i], s ? x : v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    if (i && s == 0) sums.template add<FIRST>(i - 1, j, sum[(i - 1) & 1][j]);
                    if (i + 1 == NT && s != 1 && next >= 0) fetch_col(next, d, kPairParts[s][0], j);
                }
            if (next >= 0) {
#pragma unroll
                for (int k = 0; k < 2; ++k) fetch_row(next, d, k, i);
            }
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) sums.template add<FIRST>(NT - 1, j, sum[(NT - 1) & 1][j]);
    };
    if (g_begin < g_end) {
#pragma unroll
        for (int d = 0; d < AHEAD; ++d)
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    fetch_row(g_begin * kGroup + d, d, k, i);
                    fetch_col(g_begin * kGroup + d, d, k, i);
                }
        for (int g = g_begin; g < g_end; ++g) {
            // (into LDS: in registers from here to the group's end, or fetched there, they cost more)
            wait_lgkmcnt0();
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(a.exps + (int64_t)g * a.K, 0, a.K, 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)Ex[wave], 4, exps_at, 0, 0, 0);
            if constexpr (AHEAD == kGroup) {
#pragma unroll
                for (int d = 0; d < kGroup; ++d) {
                    if (d == 0) multiply(first, d, -1);
                    else if (g * kGroup + d < a.stages) multiply(later, d, -1);
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int i = 0; i < NT; ++i) {
                            fetch_row((g + 1) * kGroup + d, d, k, i);
                            fetch_col((g + 1) * kGroup + d, d, k, i);
                        }
                }
            } else {
                const int end = min(kGroup, a.stages - g * kGroup);
#pragma unroll
                for (int i = 0; i < NT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) sums.t[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
                for (int d = 0; d < end; ++d) multiply(later, 0, g * kGroup + d + 1);
            }
            // the exponents have landed: at least this many fetches were issued behind them, and none is moved over these lines
            asm volatile("" ::: "memory");
            wait_vmcnt<AHEAD * 4 * NT>();
            asm volatile("" ::: "memory");
            sums.scale([&](int i) { return row_exponent(Ex[wave], i) - a.row_step; }, [&](int j) { return col_factors(Ex[wave] + kT, j); });
        }
    }
    for (int64_t row = (int64_t)a.stages * 32; row < a.T; row += 32) {
        __syncthreads();
        build_stage(a, row, r0 & ~(kT - 1), St, Sc, red);
        build_stage(a, row, c0 & ~(kT - 1), St + 8 * kPairBytes, Sc + kT, red);
        __syncthreads();
        if (wave != (int)((row - (int64_t)a.stages * 32) / 32 & 3)) continue;
        const int br = (r0 & (kT - 1)) / 16, bc = (c0 & (kT - 1)) / 16;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                rows[0][k][i] = *(reinterpret_cast<const v8h*>(St + (br + i) * kPairBytes + k * 1024) + lane);
                cols[0][k][i] = *(reinterpret_cast<const v8h*>(St + (8 + bc + i) * kPairBytes + k * 1024) + lane);
            }
        multiply(first, 0, -1);
        sums.scale([&](int i) { return row_exponent(Sc, br + i) - a.row_step; }, [&](int j) { return col_factors(Sc + kT, bc + j); });
    }
    v4f* const all = reinterpret_cast<v4f*>(St);   // [wave][two rows of blocks][lane]
#pragma unroll
    for (int half = 0; half < NT; half += 2) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) all[(wave * 2 * NT + i * NT + j) * 64 + lane] = sums.acc[half + i][j];
        __syncthreads();
        for (int block = wave; block < 2 * NT; block += 4) {
            const int i = half + block / NT, j = block % NT;
            v4f s = all[block * 64 + lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) s += all[(w * 2 * NT + block) * 64 + lane];
            if (ti != tj || i >= j) store_block(a, r0 + i * 16 + l16, c0 + j * 16 + 4 * q, ti == tj && i == j, s);
        }
    }
}

}  // namespace

hipError_t launch_gptq_hessian(const void* x, int64_t T, int64_t K, int b, float* H, bool accumulate, void* workspace, hipStream_t st)
{
    if (T <= 0 || K <= 0 || K > 24576) return hipErrorInvalidValue;
    HessArgs a{};
    a.x = static_cast<const uint16_t*>(x);
    a.H = H;
    a.xr = a.part = static_cast<float*>(workspace);   // 4 T K bytes either way
    a.T = T;
    a.K = (int)K;
    a.b = b;
    a.accumulate = accumulate ? 1 : 0;
    a.nt = (int)((K + kT - 1) / kT);
    // two workgroups per compute unit work at a time; the tiles beyond whole rounds of those would run on a mostly idle chip for a
    // whole tile's time (K = 4096: 528 tiles for 512 slots)
    const int tiles = a.nt * (a.nt + 1) / 2, slots = 2 * compute_units(), rem = tiles % slots;
    // Pairs of halves on the fp16 MFMA from 1408 rows, or from 1100 if there are tiles enough: fewer products, but one launch more and
    // 32 rows or more rotated on the spot.  The other way against this one, us: T = 1200, K = 1024 / 1280 / 1664 37 / 44 / 62 against
    // 37 / 39 / 44; T = 1408 and 1500, K = 512 25 and 28 against 21, K = 1024 39 and 43 against 38.  Not below, where it would still be the
    // faster one (T = 768 / 1024, K = 4096 112 / 135 against 87 / 98): of rows very different in size its error is the larger one there (rms over
    // sqrt(h_ii h_jj), b = 16, rows of 2^-20 .. 2^20: T = 768 2.7e-8 against 3.0e-8, 1024 2.8e-8 against 2.9e-8, 1100 3.0e-8 against 2.8e-8), as
    // those of few sums of 32 rows are.
    if (b > 1 && (T >= 1408 || (T >= 1100 && tiles > 50))) {
        // (a stage takes 128 K bytes, a group of four K for their exponents; what the 4 T K bytes do not hold is rotated on the spot)
        a.stages = (int)((T * 16 - 3) / 513);
        a.planes = static_cast<char*>(workspace);
        a.exps = reinterpret_cast<uint8_t*>(a.planes + (int64_t)a.stages * 128 * K);
        a.row_step = kPairRow + (b == 16 ? 4 : b == 32 ? 5 : b == 64 ? 6 : 7);
        hipLaunchKernelGGL(hessian_pack_kernel, dim3((unsigned)((a.stages + kGroup - 1) / kGroup), (unsigned)a.nt), dim3(256), 0, st, a);
        // The tiles beyond whole rounds, up to one per compute unit, in parts of 64 x 64, or of 32 x 32 if those leave most of the chip
        // idle.  8192 rows, left whole / in 64 / in 32, us: K = 512 (10 left) 257 / 103 / 46, 768 (21) 257 / 102 / 70, 1024 (36) 255 / 99 / 100,
        // 1664 (91) 264 / 135 / 183, 2048 (136) 264 / 213 / 234, 2560 (210) 271 / 261 / 360, 3072 (300) 350 / 350 / 515, 4096 (16) 624 / 517 / 468
        //
        // Pairs of tiles, one to a compute unit, where they fill it: from 2048 rows if nearly all units have one in every round, from 4096 if three
        // of four have.  Tiles / pairs, us: 1408 rows, K = 4096 104 / 104, 5120 (400 pairs for 256 units) 156 / 168, 8192 (1024) 328 / 331; 2048
        // rows, 4096 132 / 129, 5120 209 / 211, 8192 449 / 435; 4096 rows, 2944 (121) 176 / 203, 3584 (196) 190 / 188, 4096 228 / 210, 5120
        // 378 / 366, 8192 828 / 762; 8192 rows, 2944 326 / 357, 3584 356 / 335, 4096 424 / 386, 5120 719 / 664, 8192 1643 / 1481.
        const int units = slots / 2, rows = a.nt / 2, all = rows * rows, over = all % units;
        const int pairs = all > units && over <= units / 2 ? all - over : all, rounds = (pairs + units - 1) / units;
        a.pairs = (T >= 4096 && 4 * (int64_t)pairs >= 3 * (int64_t)rounds * units) || (T >= 2048 && 20 * (int64_t)pairs >= 19 * (int64_t)rounds * units);
        a.full = a.pairs ? pairs : rem > slots / 2 ? tiles : tiles - rem;
        const int small = tiles - (a.pairs ? 2 : 1) * a.full;
        static LdsAttrOnce pair_once, tile_once;
        if (a.pairs) {
            const hipError_t e = pair_once.ensure(reinterpret_cast<const void*>(hessian_pair_kernel), kPairLds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(hessian_pair_kernel, dim3((unsigned)a.full), dim3(512), kPairLds, st, a);
        } else if (a.full) {
            const hipError_t e = tile_once.ensure(reinterpret_cast<const void*>(hessian_tile_kernel), kTileLds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(hessian_tile_kernel, dim3((unsigned)a.full), dim3(256), kTileLds, st, a);
        }
        if (small > slots / 16) hipLaunchKernelGGL(hessian_part_kernel<4>, dim3((unsigned)(4 * small)), dim3(256), 0, st, a);
        else if (small) hipLaunchKernelGGL(hessian_part_kernel<2>, dim3((unsigned)(16 * small)), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    if (b > 1) {
        a.in_scale = b >= 64 ? 0.125f : 0.25f;
        a.out_scale = 1.0f / ((float)b * a.in_scale * a.in_scale);
        hipLaunchKernelGGL(hessian_rotate_kernel, dim3((unsigned)((T + 7) / 8), (unsigned)((K + kRotCols - 1) / kRotCols)), dim3(256), 0, st, a);
        // in parts of 64 x 64, or of 32 x 32 where they are so few that those have compute units to themselves.  1000 rows, the tiles
        // left whole / in 64 / in 32, us: K = 512 (10 left) 80 / 37 / 21, 1024 (36) 88 / 40 / 32, 1408 (66) 92 / 52 / 42, 1664 (91) 92 / 54 / 50,
        // 2048 (136) 90 / 63 / 65, 2944 (276) 117 / 97 / 111, 3328 (351) 118 / 111 / 134, 3712 (435) 119 / 130 / 165, 4096 (16) 179 / 155 / 139;
        // 256 rows: 1664 36 / 22 / 19, 2048 37 / 26 / 24, 3328 52 / 45 / 47
        const int parts = rem > slots * 5 / 8 ? 0 : rem > slots / 6 ? 32 : 16, small = parts ? rem : 0;
        a.full = tiles - small;
        if (a.full) hipLaunchKernelGGL(hessian_split_kernel<64>, dim3((unsigned)a.full), dim3(256), 0, st, a);
        if (small && parts == 16) hipLaunchKernelGGL(hessian_split_kernel<16>, dim3((unsigned)(16 * small)), dim3(256), 0, st, a);
        else if (small) hipLaunchKernelGGL(hessian_split_kernel<32>, dim3((unsigned)(4 * small)), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    // So T is cut into parts for them, of at least 512 rows (less does not repay the second launch), as many as fit the round
    // and the workspace that every caller has (not the one at hand: the last bits do not depend on its size).
    int parts = rem ? std::min({slots / rem, 8, (int)std::min<int64_t>(T / 512, 8)}) : 1;
    if (rem) parts = std::min(parts, (int)std::min<int64_t>(8, T * K / (int64_t)(rem * kT * kT)));
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
