// From a layer's Hessian to what the MR-GPTQ sweep consumes (arXiv 2509.23202, Section 4 "Standard GPTQ" and Section
// 4.1 "Ingredient 2"; Section 5 "Algorithms": dampening 1e-2): the static activation order (columns by descending
// Hessian diagonal), the dampened, re-ordered Hessian A = H[perm][:,perm] + lambda mean(diag H) I, and the upper
// triangular U with U^T U = A^-1 whose row j drives the update after column j.
//
// U is obtained without forming A^-1: factor A = R R^T with R UPPER triangular; then A^-1 = R^-T R^-1 and U = R^-1.
// With J the index reversal, J A J = L L^T is an ordinary (lower) Cholesky factorization, R = J L J and U = J L^-1 J.
//
// L^-1 comes out of the factorization itself: the row operations that turn J A J into L^T turn the identity beside it into
// L^-1 (Gauss elimination of [A | I]).  Block column k of A is finished when that of I begins to fill, so ONE square
// matrix M holds both: after step k its block columns 0 .. k are those of the right-hand side, the others those of A.
// Step k of K / 128, with D = the inverse of the diagonal block's Cholesky factor:
//   panel    L_ik = M_ik D^T  (i > k, into a scratch panel),  M_kj <- D M_kj  (j < k),  M_kk <- D, and the next diagonal block
//   update   M_ij <- M_ij - L_ik X_j  for all i > k, j <= i, where X_j = M_kj (j <= k; M_ik counts as zero) or L_jk^T (j > k)
// and the first workgroup of the update factors the next diagonal block and inverts the factor while the others work, so the
// only serial chain of the method -- K columns, one behind the other -- runs beside the products instead of between them.
// Two launches per 128 columns.  The diagonal block is treated by the same elimination, 16 columns at a time.  All in fp32: the
// panel and the diagonal blocks on the fp32 MFMA (v_mfma_f32_16x16x4_f32), the update as six products of the three bf16 parts that
// the panel leaves its results in.
//
// Bound by that chain: [4096, 4096] takes 0.98 ms, per 128 columns 7.5 us of panel and 18 - 24 us of update, of which the
// diagonal block is 2 us of loads, 16 of elimination and 2 of stores.  (1.45 ms with one MFMA per column of a diagonal tile, with
// the diagonal block's product in the workgroup that factors it, and with fp32 products in the update, whose two rounds of
// workgroups were longer than the chain; error against 64 bits, K = 512 .. 4096: 0.82 - 0.99 of what it was.  6.3 ms with
// 64-column blocks, one wave per diagonal block between the products and an inversion by recursive doubling behind.)
#include "device_util.hpp"
#include "internal.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace fp4mr {
namespace {

constexpr int NB = 128;        // block size of the elimination
constexpr int SB = 16;         // columns per step inside a diagonal block
constexpr int NS = NB / SB;    // such steps
constexpr int PW = 32;         // columns per workgroup of the panel kernel

struct PrepArgs {
    float* M;        // [Kp, Kp], lower block triangle used
    char* P;         // the panel, L_jk^T of the blocks j > k and X_j of the blocks j < k, as operands (operand_at); the block k is left out
    float* DT;       // the 36 tiles of D, lane (l16, q) of a tile with row l16, columns 4 q .. 4 q + 3
    int Kp;          // K rounded up to whole blocks; the padding is the identity
    int nt;          // Kp / NB
    int k;
};

// ---------------------------------------------------------------- ordering and gather

// the diagonal as a contiguous array; perm = identity (a diagonal with NaNs does not rank into a permutation below: every
// entry is at least valid)
__global__ __launch_bounds__(256) void diag_kernel(const float* H, int K, float* diag, int* perm)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= K) return;
    diag[i] = H[(int64_t)i * K + i];
    perm[i] = i;
}

// rank of column i in the order "descending diagonal, ties by ascending index", counted by one wave; perm[rank] = i.
// The last workgroup sums the diagonal (in double, in a fixed order) for its mean instead.
__global__ __launch_bounds__(256) void order_kernel(const float* diag, int K, int use_order, int* perm, float* mean)
{
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double part[256];
        double s = 0.0;
        for (int i = threadIdx.x; i < K; i += 256) s += (double)diag[i];
        part[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) *mean = (float)(part[0] / (double)K);
        return;
    }
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= K || !use_order) return;
    const float di = diag[i];
    int rank = 0;
    for (int j = lane; j < K; j += 64) {
        const float dj = diag[j];
        rank += (dj > di) || (dj == di && j < i);
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) rank += __shfl_xor(rank, s);
    if (lane == 0) perm[min(rank, K - 1)] = i;
}

// M[i][j] = H[perm[K-1-i]][perm[K-1-j]] + (i == j) damp * mean up to the end of row i's diagonal block.  One workgroup per row:
// the row of H goes through LDS, so that memory is read and written in order.
__global__ __launch_bounds__(256) void gather_kernel(const float* H, const int* perm, const float* mean, float damp, int K, int Kp, float* M)
{
    extern __shared__ float row[];
    const int i = blockIdx.x;
    const int end = (i / NB + 1) * NB;
    if (i < K) {
        const float* src = H + (int64_t)min(max(perm[K - 1 - i], 0), K - 1) * K;
        for (int j = threadIdx.x; j < K; j += 256) row[j] = src[j];
        __syncthreads();
        const float add = damp * (*mean);
        for (int j = threadIdx.x; j < end; j += 256) {
            float v = 0.0f;
            if (j < K) v = row[min(max(perm[K - 1 - j], 0), K - 1)];
            if (i == j) v += add;
            M[(int64_t)i * Kp + j] = v;
        }
    } else {
        for (int j = threadIdx.x; j < end; j += 256) M[(int64_t)i * Kp + j] = (i == j) ? 1.0f : 0.0f;
    }
}

// U[i][j] = V[K-1-i][K-1-j] on and above the diagonal, 0 below
__global__ __launch_bounds__(256) void reverse_kernel(const float* V, int K, int Kp, float* U)
{
    const int i = blockIdx.x;
    for (int j = threadIdx.x; j < K; j += 256)
        U[(int64_t)i * K + j] = (j >= i) ? V[(int64_t)(K - 1 - i) * Kp + (K - 1 - j)] : 0.0f;
}

// ---------------------------------------------------------------- tiles

// 16 x 16 tiles in LDS as an MFMA leaves them -- lane (l16, q) holds rows 4 q .. 4 q + 3 of column l16, one 16-byte access -- with
// four floats more behind every sixteen lanes, so that the other way round (four columns of a row per lane) is free of bank
// conflicts as well.  The contraction of a product of two such tiles goes along 4 q + v, MFMA v taking the four rows 4 q + v of
// either: operands need no other order.  The lower block triangle of a diagonal block is kept row by row.
constexpr int TF = 4 * 68;                       // floats per tile
constexpr int TILES = NS * (NS + 1) / 2;
__device__ __forceinline__ int tile_index(int i, int j) { return i * (i + 1) / 2 + j; }
// row of tile t (three bits each)
__device__ __forceinline__ int tile_row(int t)
{
    constexpr uint64_t low = 0x5b6db2491b6d2448ull, high = 0x1ffffffb6db6ull;
    return (int)((t < 21 ? low >> (3 * t) : high >> (3 * (t - 21))) & 7);
}
static_assert(NS == 8, "tile_row");

// a lane's share of a tile
__device__ __forceinline__ int lane_at() { return (threadIdx.x & 63) * 4 + ((threadIdx.x >> 4) & 3) * 4; }
__device__ __forceinline__ v4f get_tile(const float* tile) { return *reinterpret_cast<const v4f*>(tile + lane_at()); }
__device__ __forceinline__ void put_tile(float* tile, v4f v) { *reinterpret_cast<v4f*>(tile + lane_at()) = v; }
// where element (row, col) lies
__device__ __forceinline__ int tile_at(int row, int col) { return (row >> 2) * 68 + col * 4 + (row & 3); }

// a^T b over the rows of two tiles
__device__ __forceinline__ v4f product(v4f a, v4f b)
{
    v4f e = v4f{0.f, 0.f, 0.f, 0.f}, o = e;   // (two chains)
    e = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], e, 0, 0, 0);
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], o, 0, 0, 0);
    e = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], e, 0, 0, 0);
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], o, 0, 0, 0);
    return e + o;
}

// ---------------------------------------------------------------- operands of the update

// Rows of 128 columns on the contraction side, sixteen columns to a block, as the bf16 MFMA takes them: a quarter w of the
// contraction is strips w and 7 - w, of which lane (l16, q) holds rows 4 q .. 4 q + 3 of column l16 -- what an fp32 MFMA leaves there.
// Three parts of eight bits each, one behind the other, 1 KB a part.
__device__ __forceinline__ int64_t operand_at(int w, int blocks, int block) { return ((int64_t)w * blocks + block) * 3072; }
// of the panel of step k: how many sixteens, and where those of NB-block j != k begin
__device__ __forceinline__ int panel_blocks(const PrepArgs& a) { return (a.nt - 1) * NS; }
__device__ __forceinline__ int panel_block(const PrepArgs& a, int j) { return (j < a.k ? j : j - 1) * NS; }
__device__ __forceinline__ void put_operand(char* p, v4f low, v4f high)
{
    const float x[8] = {low[0], low[1], low[2], low[3], high[0], high[1], high[2], high[3]};
    const Split3 s = split3(x);
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<v8bf*>(p + k * 1024 + (threadIdx.x & 63) * 16) = s.part[k];
}

// ---------------------------------------------------------------- panel

// A workgroup takes 32 columns of either half: rows k of M to the left of the diagonal block (B = M_kj as it lies), or rows of
// M below it (B = M_ik^T, transposed on its way into LDS); out = D B, 128 x 32.  D is lower triangular: of its strips of sixteen
// rows wave w takes w and 7 - w, nine sixteenths of the contraction between them, straight from memory (tiles, the other way
// round).  36 more workgroups take two strips of block row k + 1 for their 32 columns and, of its products L L^T, the tile that
// the two meet in: the next diagonal block is finished when the update begins to factor it (where one workgroup
// would spend 6 us on that product).
// Bound: latency -- loads some 2 us, 72 MFMAs a wave one, the launch.
__global__ __launch_bounds__(256) void panel_kernel(PrepArgs a)
{
    __shared__ __attribute__((aligned(16))) float Bs[NS][2][TF];    // [sixteen of the contraction][sixteen columns]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int k0 = a.k * NB, regular = (a.nt - 1) * (NB / PW);
    const bool extra = (int)blockIdx.x >= regular;
    const int blk = blockIdx.x / (NB / PW), sub = (blockIdx.x % (NB / PW)) * PW;
    const bool left = !extra && blk < a.k;
    // first column of M_kj, or first row of M_ik; of the second sixteen
    int c0[2];
    c0[0] = (left ? blk : blk + 1) * NB + sub;
    c0[1] = c0[0] + SB;
    const int te = (int)blockIdx.x - regular;
    if (extra) {
        const int i = tile_row(te), j = te - tile_index(i, 0);
        c0[0] = k0 + NB + SB * i;
        c0[1] = k0 + NB + SB * j;
    }
    const int low = wave, high = NS - 1 - wave;
    v4f dl[NS / 2], dh[NS];   // (tiles that the strip does not have: its last one, not used)
#pragma unroll
    for (int t = 0; t < NS; ++t) dh[t] = *reinterpret_cast<const v4f*>(a.DT + tile_index(high, min(t, high)) * 256 + lane * 4);
#pragma unroll
    for (int t = 0; t < NS / 2; ++t) dl[t] = *reinterpret_cast<const v4f*>(a.DT + tile_index(low, min(t, low)) * 256 + lane * 4);
    v4f m[4];
    if (left) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int idx = it * 256 + tid;  // 8 float4 per row of 32
            m[it] = *reinterpret_cast<const v4f*>(a.M + (int64_t)(k0 + idx / 8) * a.Kp + c0[0] + (idx % 8) * 4);
        }
    } else {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int idx = it * 256 + tid;  // 32 float4 per row of 128
            m[it] = *reinterpret_cast<const v4f*>(a.M + (int64_t)(c0[it >> 1] + (idx / 32) % SB) * a.Kp + k0 + (idx % 32) * 4);
        }
    }
    float* const Mt = a.M + (int64_t)(c0[0] + 4 * q) * a.Kp + c0[1] + l16;   // (extra) the tile that is updated
    v4f old = v4f{0.f, 0.f, 0.f, 0.f};
    if (extra && wave == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) old[v] = Mt[(int64_t)v * a.Kp];
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int idx = it * 256 + tid;
        if (left) {
            const int row = idx / 8, col = (idx % 8) * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) Bs[row / SB][col / SB][tile_at(row % SB, col % SB + e)] = m[it][e];
        } else {
            const int col = idx / 32, row = (idx % 32) * 4;
            *reinterpret_cast<v4f*>(&Bs[row / SB][col / SB][tile_at(row % SB, col % SB)]) = m[it];
        }
    }
    __syncthreads();
    v4f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        if (t > high) break;
        const v4f y[2] = {get_tile(Bs[t][0]), get_tile(Bs[t][1])};
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(dh[t][v], y[j][v], acc[1][j], 0, 0, 0);
        if (t < NS / 2 && t <= low) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(dl[t & 3][v], y[j][v], acc[0][j], 0, 0, 0);
        }
    }
    if (extra) {
        // rows of L^T on both sides: this wave's two strips, then the four waves' sums in order
        const v4f part = product(acc[0][0], acc[0][1]) + product(acc[1][0], acc[1][1]);
        __syncthreads();
        put_tile(Bs[wave][0], part);
        __syncthreads();
        if (wave == 0) {
            const v4f s = (get_tile(Bs[0][0]) + get_tile(Bs[1][0])) + (get_tile(Bs[2][0]) + get_tile(Bs[3][0]));
#pragma unroll
            for (int v = 0; v < 4; ++v) Mt[(int64_t)v * a.Kp] = old[v] - s[v];
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        put_operand(a.P + operand_at(wave, panel_blocks(a), blk * NS + sub / SB + j), acc[0][j], acc[1][j]);
        if (left) {   // (rows k of the inverse are finished)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) a.M[(int64_t)(k0 + (i ? high : low) * SB + 4 * q + v) * a.Kp + c0[j] + l16] = acc[i][j][v];
        }
    }
}

// ---------------------------------------------------------------- diagonal block

struct DiagLds {
    float S[TILES * TF];
    float D[TF];             // of the present step, the other way round: lane (l16, q) holds D[l16][4 q .. 4 q + 3]
    float X[2][NS][TF];      // per step p: blocks j <= p hold X_j = D S_pj (j == p: D), the others L_jp^T
};

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// 1 / sqrt(d) to an ulp (one Newton step).  SUBNORMAL: for pivots that are subnormal, which v_rsq_f32 takes for zero: they are
// moved up by 2^48 on the way.
template <bool SUBNORMAL>
__device__ __forceinline__ float inverse_root(float d)
{
    const float y = SUBNORMAL && d < 0x1p-126f ? __builtin_amdgcn_rsqf(d * 0x1p48f) * 0x1p24f : __builtin_amdgcn_rsqf(d);
    return fmaf(0.5f * y, fmaf(-d * y, y, 1.0f), y);
}

// register k of the result holds, in its group g of sixteen lanes, what m[g] held in group k
template <int K>
__device__ __forceinline__ float transposed(const float (&m)[4])
{
    auto swap16 = [](float a, float b) {   // the odd groups of a for the even ones of b
        return __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)[K & 1];
    };
    const auto r = __builtin_amdgcn_permlane32_swap(swap16(m[0], m[1]), swap16(m[2], m[3]), false, false);   // the upper half of one for the lower of the other
    return __uint_as_float(r[K >> 1]);
}

// x (a finished 16 x 16 diagonal block, as an MFMA leaves it: column l16, rows 4 q + v) -> its Cholesky factor's inverse; one wave,
// four columns at a time.  The 4 x 4 block on the diagonal is factored by every lane for itself, from ten values that
// v_readlane spreads.  Column 4 J + v is row 4 J + v as well (the block is symmetric), so the lanes of group J hold
// four columns of X with the row along the lanes, and four rows of the inverse in the making: both are solved
// for there.  Transposed between the lane groups they are the operands of one MFMA each that takes four columns off the rest.
// The chain -- pivot, root, column, next pivot -- is ordinary fp32 arithmetic inside four columns; an MFMA, whose result is some 50
// cycles away, comes once in four (one per column: 3700 cycles a tile, now 2100 to 2500, the more when another workgroup shares the compute unit).
template <bool SUBNORMAL, int J>
__device__ __forceinline__ void factor_four(v4f& x, v4f& w)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    auto a = [&](int i, int j) { return lane_value(x[i], 20 * J + j); };
    const float a00 = a(0, 0), a10 = a(1, 0), a11 = a(1, 1), a20 = a(2, 0), a21 = a(2, 1), a22 = a(2, 2), a30 = a(3, 0), a31 = a(3, 1), a32 = a(3, 2), a33 = a(3, 3);
    const float y0 = inverse_root<SUBNORMAL>(a00);
    const float l10 = a10 * y0, l20 = a20 * y0, l30 = a30 * y0;
    const float y1 = inverse_root<SUBNORMAL>(fmaf(-l10, l10, a11));
    const float l21 = fmaf(-l20, l10, a21) * y1, l31 = fmaf(-l30, l10, a31) * y1;
    const float y2 = inverse_root<SUBNORMAL>(fmaf(-l21, l21, fmaf(-l20, l20, a22)));
    const float l32 = fmaf(-l31, l21, fmaf(-l30, l20, a32)) * y2;
    const float y3 = inverse_root<SUBNORMAL>(fmaf(-l32, l32, fmaf(-l31, l31, fmaf(-l30, l30, a33))));
    auto solve = [&](const v4f& v, float (&r)[4]) {
        r[0] = v[0] * y0;
        r[1] = fmaf(-r[0], l10, v[1]) * y1;
        r[2] = fmaf(-r[1], l21, fmaf(-r[0], l20, v[2])) * y2;
        r[3] = fmaf(-r[2], l32, fmaf(-r[1], l31, fmaf(-r[0], l30, v[3]))) * y3;
    };
    float r[4];
    solve(w, r);
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = q == J ? r[v] : w[v];
    if constexpr (J < 3) {
        float c[4];
        solve(x, c);
        float l = transposed<J>(c);
        l = l16 > 4 * J + 3 ? l : 0.0f;
        const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
        x = x - __builtin_amdgcn_mfma_f32_16x16x4f32(l, l, zero, 0, 0, 0);
        w = w - __builtin_amdgcn_mfma_f32_16x16x4f32(l, transposed<J>(r), zero, 0, 0, 0);
    }
}

template <bool SUBNORMAL>
__device__ __forceinline__ v4f factor_columns(v4f x)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    v4f w;
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = (4 * q + v == l16) ? 1.0f : 0.0f;
    factor_four<SUBNORMAL, 0>(x, w);
    factor_four<SUBNORMAL, 1>(x, w);
    factor_four<SUBNORMAL, 2>(x, w);
    factor_four<SUBNORMAL, 3>(x, w);
    return w;
}

// the diagonal block of step p, finished: D, its Cholesky factor's inverse, into S, X and D
__device__ __forceinline__ void factor_block(DiagLds& t, int p, v4f x)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    v4f w = factor_columns<false>(x);
    // (a subnormal pivot, or one that is not positive, leaves infinities or NaNs; two selects per column in the chain instead cost
    // 45 us at K = 4096)
    if (__builtin_expect(__any(!(fabsf(w[0]) + fabsf(w[1]) + fabsf(w[2]) + fabsf(w[3]) < INFINITY)), 0)) w = factor_columns<true>(x);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        w[v] = (4 * q + v >= l16) ? w[v] : 0.0f;
        t.D[tile_at(l16, 4 * q + v)] = w[v];   // (the transpose of D in a tile's order)
    }
    put_tile(t.S + tile_index(p, p) * TF, w);
    put_tile(t.X[p & 1][p], w);
}

// L_ip^T = D S_ip^T
__device__ __forceinline__ v4f factor_rows(const DiagLds& t, int p, int i)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const float* tile = t.S + tile_index(i, p) * TF;
    v4f s;
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = tile[tile_at(l16, 4 * q + v)];
    return product(get_tile(t.D), s);
}

// A diagonal block of 36 tiles -> its Cholesky factor's inverse in t.S, eight waves.  Wave 0 walks the serial chain: the diagonal
// tile of 16 columns, its factor and inverse D, then only what the next diagonal tile waits for.  The other seven take the rest
// of step p meanwhile: the seven products with D (rows of the inverse to the left, columns of the factor below), then the
// elimination of all later rows.  Each of them keeps five tiles in registers from the first step to the last (wave u + 1 tiles
// 1 + u, 8 + u, ...; wave 0 begins with tile 0) and writes to LDS what the next step takes from there.
constexpr int kKept = 5;
static_assert(1 + kKept * (NS - 1) == TILES, "all tiles are kept by someone");
__device__ __forceinline__ int kept_tile(int wave, int e) { return wave ? wave + (NS - 1) * e : 0; }

__device__ __forceinline__ void invert_factor(DiagLds& t, v4f (&x)[kKept])
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), u = wave - 1;
    int row[kKept], col[kKept];
    if (wave == 0) {
        factor_block(t, 0, x[0]);
    } else {
#pragma unroll
        for (int e = 0; e < kKept; ++e) {
            const int n = kept_tile(wave, e);
            row[e] = tile_row(n);
            col[e] = n - tile_index(row[e], 0);
            put_tile(t.S + n * TF, x[e]);
        }
    }
    for (int p = 0; p < NS; ++p) {
        float(*X)[TF] = t.X[p & 1];
        __syncthreads();  // D of step p is there, step p - 1 has been eliminated everywhere
        if (wave == 0) {
            v4f d = v4f{0.f, 0.f, 0.f, 0.f};
            if (p + 1 < NS) {
                const v4f old = get_tile(t.S + tile_index(p + 1, p + 1) * TF);
                const v4f l = factor_rows(t, p, p + 1);
                d = old - product(l, l);
            }
            __syncthreads();
            if (p + 1 < NS) factor_block(t, p + 1, d);
            continue;
        }
        if (u < p) {
            float* s = t.S + tile_index(p, u) * TF;
            const v4f r = product(get_tile(t.D), get_tile(s));
            put_tile(s, r);
            put_tile(X[u], r);
        } else {
            put_tile(X[u + 1], factor_rows(t, p, u + 1));
        }
        __syncthreads();
        if (p + 1 == NS) break;
        v4f xi[kKept], xj[kKept];
#pragma unroll
        for (int e = 0; e < kKept; ++e) {
            xi[e] = get_tile(X[row[e]]);
            xj[e] = get_tile(X[col[e]]);
        }
#pragma unroll
        for (int e = 0; e < kKept; ++e) {
            if (row[e] <= p || (row[e] == p + 1 && col[e] == p + 1)) continue;   // finished; wave 0's
            const v4f r = product(xi[e], xj[e]);
            // (block column p was the factor's and becomes the inverse's: it starts from zero)
            x[e] = (col[e] == p ? v4f{0.f, 0.f, 0.f, 0.f} : x[e]) - r;
            if (row[e] == p + 1 || col[e] == p + 1 || (row[e] == p + 2 && col[e] == p + 2)) put_tile(t.S + kept_tile(wave, e) * TF, x[e]);
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------- update

// Workgroup 0: the next diagonal block, invert_factor; k == -1 starts the method with block 0.  The others: half a block each, 128 x 64,
// a 32 x 32 piece per wave, the contraction in four quarters copied into LDS, two of them at a time; two workgroups per
// compute unit.  The
// product of 24-bit values is six products of bf16 parts, the largest summed apart; it is summed from zero and subtracted once
// (with the accumulators started as M each MFMA would round at the size of M, towards zero).
// Bound: the chain in workgroup 0.  (One 128 x 128 block per workgroup and compute unit, three quarters in LDS: the blocks were the
// longer side, K = 8192 4.95 ms against 4.2; fp32 MFMAs on such blocks 5.3.)
constexpr int kUpdateStage = 12 * 3072, kUpdateLds = 2 * kUpdateStage;
static_assert(sizeof(DiagLds) <= kUpdateLds, "the diagonal block fits");
__global__ __launch_bounds__(512, 4) void update_kernel(PrepArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int next = a.k + 1;
    if (blockIdx.x == 0) {
        DiagLds& d = *reinterpret_cast<DiagLds*>(smem);
        float* const Md = a.M + (int64_t)next * NB * (a.Kp + 1);
        v4f x[kKept];
#pragma unroll
        for (int e = 0; e < kKept; ++e) {
            if (wave == 0 && e > 0) break;
            const int t = kept_tile(wave, e), i = tile_row(t), j = t - tile_index(i, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) x[e][v] = Md[(int64_t)(SB * i + 4 * q + v) * a.Kp + SB * j + l16];
        }
        invert_factor(d, x);
        // D: four values of a row per lane, in M and, as tiles, for the panel; zeros above
#pragma unroll
        for (int e = 0; e < 5; ++e) {
            const int t = wave + 8 * e;
            if (t >= TILES) break;
            const int i = tile_row(t), j = t - tile_index(i, 0);
            v4f row;
#pragma unroll
            for (int v = 0; v < 4; ++v) row[v] = d.S[t * TF + tile_at(l16, 4 * q + v)];
            *reinterpret_cast<v4f*>(Md + (int64_t)(SB * i + l16) * a.Kp + SB * j + 4 * q) = row;
            *reinterpret_cast<v4f*>(a.DT + t * 256 + lane * 4) = row;
        }
        for (int t = wave; t < TILES - NS; t += 8) {   // (the strict lower triangle, mirrored)
            const int i = tile_row(t), j = t - tile_index(i, 0);
            *reinterpret_cast<v4f*>(Md + (int64_t)(SB * j + l16) * a.Kp + SB * (i + 1) + 4 * q) = v4f{0.f, 0.f, 0.f, 0.f};
        }
        return;
    }
    // block (i, j): rows next, next + 1, ... with i + 1 blocks each, the diagonal block of the first of them left out
    const int t = ((int)blockIdx.x - 1) >> 1, half = (blockIdx.x - 1) & 1, p = t < next ? t : t + 1;
    const int64_t n = p + (int64_t)next * (next + 1) / 2;
    int i = (int)((sqrtf(8.0f * (float)n + 1.0f) - 1.0f) * 0.5f);
    while ((int64_t)i * (i + 1) / 2 > n) --i;
    while ((int64_t)(i + 1) * (i + 2) / 2 <= n) ++i;
    const int j = (int)(n - (int64_t)i * (i + 1) / 2);
    const int blocks = panel_blocks(a), wr = (wave >> 1) * 2, wc = (wave & 1) * 2;   // first 16-wide block of the piece
    // the column operand is the MFMA's A: a lane owns four neighbouring columns of a row
    float* const C = a.M + (int64_t)(i * NB + wr * SB + l16) * a.Kp + j * NB + (half * 4 + wc) * SB + 4 * q;
    v4f old[2][2], low[2][2], high[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            low[x][y] = high[x][y] = old[x][y] = v4f{0.f, 0.f, 0.f, 0.f};
            if (j != a.k) old[x][y] = *reinterpret_cast<const v4f*>(C + (int64_t)(SB * x) * a.Kp + SB * y);
        }
    const bool own = j == a.k;
    char* const A = a.P + operand_at(0, blocks, panel_block(a, i));
    char* const B = a.P + operand_at(0, blocks, panel_block(a, j) + half * 4);   // (unused if own)
    // the copies of a quarter, 1 KB each: 24 of rows, 12 of columns; a wave takes five, the last of some twice (the same data).
    // X_k = D is not in the panel: it is split here, from M, by four waves.
    constexpr int OPS = 5;
    auto issue = [&](int w) {
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(A + operand_at(w, blocks, 0), 0, NS * 3072, 0x00020000);
        char* const base = smem + (w & 1) * kUpdateStage;
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const int c = it * 8 + wave;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(base + c * 1024), 16, lane * 16, c * 1024, 0, 0);
        }
        if (own) {
            if (wave < NS / 2) {
                const float* D = a.M + (int64_t)(a.k * NB + 4 * q) * a.Kp + a.k * NB + (half * 4 + wave) * SB + l16;
                v4f d[2];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    d[0][v] = D[(int64_t)(SB * w + v) * a.Kp];
                    d[1][v] = D[(int64_t)(SB * (NS - 1 - w) + v) * a.Kp];
                }
                put_operand(base + (NS + wave) * 3072, d[0], d[1]);
            }
            return;
        }
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(B + operand_at(w, blocks, 0), 0, NS / 2 * 3072, 0x00020000);
#pragma unroll
        for (int it = 3; it < OPS; ++it) {
            const int c = min(it * 8 + wave, 35);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(base + c * 1024), 16, lane * 16, (c - 24) * 1024, 0, 0);
        }
    };
    auto multiply = [&](int w) {
        const char* base = smem + (w & 1) * kUpdateStage + lane * 16;
        v8bf u[3][2], e[3][2];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u[k][h] = *reinterpret_cast<const v8bf*>(base + (NS + wc + h) * 3072 + k * 1024);
                e[k][h] = *reinterpret_cast<const v8bf*>(base + (wr + h) * 3072 + k * 1024);
            }
        // (part of the column, part of the row): 2^-16, 2^-8 of the product, then 1
        constexpr int order[6][2] = {{2, 0}, {1, 1}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int s = 0; s < 6; ++s)
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    v4f& d = s < 5 ? low[x][y] : high[x][y];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[order[s][0]][y], e[order[s][1]][x], d, 0, 0, 0);
                }
    };
    issue(0);
    issue(1);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < 3 && !own) wait_vmcnt<OPS>();
        else wait_vmcnt<0>();
        wait_lgkmcnt0();
        block_barrier();   // quarter w has landed
        multiply(w);
        if (w < 2) {
            wait_lgkmcnt0();
            block_barrier();   // it has been read
            issue(w + 2);
        }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) *reinterpret_cast<v4f*>(C + (int64_t)(SB * x) * a.Kp + SB * y) = old[x][y] - (high[x][y] + low[x][y]);
}

constexpr size_t kPanelBytes = NB * 6;   // per column
inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }
inline int64_t padded(int64_t K) { return (K + NB - 1) / NB * NB; }

}  // namespace

size_t gptq_prepare_workspace_bytes(int64_t K)
{
    // The 2.5 K^2 floats that callers of this entry point are told to expect, or what they are told for few columns: M, 128 rows of it, a block
    // of it, the diagonal, the mean.  launch_gptq_prepare needs M, the panel (6 bytes for a value of 128 rows, all blocks but one), 36 KB
    // of tiles, the diagonal and the mean, which is less at every K.
    const size_t Kp = (size_t)padded(K), k = (size_t)K;
    return std::max(Kp * Kp * 4 + NB * Kp * 4 + NB * NB * 4 + align256(k * 4) + 256, align256(k * k * 10));
}

hipError_t launch_gptq_prepare(const float* H, int64_t K64, float damp, bool use_order, int* perm, float* U, void* workspace,
                               hipStream_t st)
{
    if (K64 <= 0 || K64 > 24576) return hipErrorInvalidValue;  // (a row of H is staged in LDS)
    const int K = (int)K64;
    const int64_t Kp = padded(K);
    char* ws = static_cast<char*>(workspace);
    PrepArgs a{};
    a.Kp = (int)Kp;
    a.nt = (int)(Kp / NB);
    a.M = reinterpret_cast<float*>(ws);
    ws += (size_t)Kp * Kp * 4;
    a.P = ws;
    ws += kPanelBytes * (size_t)(Kp - NB);
    a.DT = reinterpret_cast<float*>(ws);
    ws += TILES * 1024;
    float* diag = reinterpret_cast<float*>(ws);
    ws += align256((size_t)K * 4);
    float* mean = reinterpret_cast<float*>(ws);

    hipLaunchKernelGGL(diag_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, H, K, diag, perm);
    hipLaunchKernelGGL(order_kernel, dim3((unsigned)((K + 3) / 4 + 1)), dim3(256), 0, st, (const float*)diag, K, use_order ? 1 : 0, perm, mean);
    static LdsAttrOnce lds_once;
    if ((size_t)K * 4 > 48 * 1024) {
        const hipError_t le = lds_once.ensure(reinterpret_cast<const void*>(gather_kernel), 24576 * 4);
        if (le != hipSuccess) return le;
    }
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)Kp), dim3(256), (size_t)K * 4, st, H, (const int*)perm, (const float*)mean, damp, K, (int)Kp, a.M);
    a.k = -1;
    static LdsAttrOnce update_once;
    const hipError_t ue = update_once.ensure(reinterpret_cast<const void*>(update_kernel), kUpdateLds);
    if (ue != hipSuccess) return ue;
    hipLaunchKernelGGL(update_kernel, dim3(1), dim3(512), kUpdateLds, st, a);
    for (a.k = 0; a.k < a.nt; ++a.k) {
        if (a.nt > 1) hipLaunchKernelGGL(panel_kernel, dim3((unsigned)((a.nt - 1) * (NB / PW) + (a.k + 1 < a.nt ? TILES : 0))), dim3(256), 0, st, a);
        if (a.k + 1 == a.nt) break;
        const int64_t tiles = (int64_t)a.nt * (a.nt + 1) / 2 - (int64_t)(a.k + 1) * (a.k + 2) / 2;
        hipLaunchKernelGGL(update_kernel, dim3((unsigned)(1 + 2 * (tiles - 1))), dim3(512), kUpdateLds, st, a);
    }
    hipLaunchKernelGGL(reverse_kernel, dim3((unsigned)K), dim3(256), 0, st, (const float*)a.M, K, (int)Kp, U);
    return hipGetLastError();
}

}  // namespace fp4mr
