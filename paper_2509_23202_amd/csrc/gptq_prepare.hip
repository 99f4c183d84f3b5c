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
//   panel    L_ik = M_ik D^T  (i > k, into a scratch panel),  M_kj <- D M_kj  (j < k),  M_kk <- D
//   update   M_ij <- M_ij - L_ik X_j  for all i > k, j <= i, where X_j = M_kj (j <= k; M_ik counts as zero) or L_jk^T (j > k)
// and the first workgroup of the update takes the next diagonal block: it updates it, factors it and inverts the factor
// while the others work, so the only serial chain of the method -- K columns, one behind the other -- runs beside the
// products instead of between them.  Two launches per 128 columns.  The diagonal block is treated by the same elimination,
// 16 columns at a time.  All in fp32, products on the fp32 MFMA (v_mfma_f32_16x16x4_f32).
//
// Bound by that chain: [4096, 4096] takes 1.5 ms, per 128 columns 8.7 us of panel and 31 - 40 us of update, of which the
// diagonal block is 4 us of loads, 4 us of product and 19 us of elimination.  (6.3 ms with 64-column blocks, one wave per
// diagonal block between the products (47 us each) and an inversion by recursive doubling behind the factorization.)
#include "device_util.hpp"
#include "internal.hpp"

#include <algorithm>
#include <cmath>

namespace fp4mr {
namespace {

constexpr int NB = 128;        // block size of the elimination
constexpr int SB = 16;         // columns per step inside a diagonal block
constexpr int NS = NB / SB;    // such steps
constexpr int LD = NB + 16;    // LDS row of 128 values: 16 mod 64 banks, so the four k-rows of an MFMA operand do not meet
constexpr int PW = 32;         // columns per workgroup of the panel kernel

struct PrepArgs {
    float* M;        // [Kp, Kp], lower block triangle used
    float* LT;       // [NB, Kp]: the panel L_ik, contraction index first
    float* DT;       // [NB, NB]: D transposed
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

// ---------------------------------------------------------------- panel

// A workgroup takes 32 columns of either half: rows k of M to the left of the diagonal block (B = M_kj as it lies), or rows of
// M below it (B = M_ik^T, transposed on its way into LDS); out = D B, 128 x 32, one 32 x 32 piece per wave.
__global__ __launch_bounds__(256) void panel_kernel(PrepArgs a)
{
    __shared__ __attribute__((aligned(16))) float As[NB][LD];       // [contraction][row of D]
    __shared__ float Bs[NB][PW + 16];                               // [contraction][column]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int blk = blockIdx.x / (NB / PW), sub = (blockIdx.x % (NB / PW)) * PW;
    const bool left = blk < a.k;
    const int k0 = a.k * NB;
    const int c0 = (left ? blk : blk + 1) * NB + sub;  // first column of M_kj, or first row of M_ik
    float4 d[16];
#pragma unroll
    for (int it = 0; it < 16; ++it) d[it] = reinterpret_cast<const float4*>(a.DT)[it * 256 + tid];
    float4 m[4];
    if (left) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int idx = it * 256 + tid;  // 8 float4 per row of 32
            m[it] = *reinterpret_cast<const float4*>(a.M + (int64_t)(k0 + idx / 8) * a.Kp + c0 + (idx % 8) * 4);
        }
    } else {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int idx = it * 256 + tid;  // 32 float4 per row of 128
            m[it] = *reinterpret_cast<const float4*>(a.M + (int64_t)(c0 + idx / 32) * a.Kp + k0 + (idx % 32) * 4);
        }
    }
#pragma unroll
    for (int it = 0; it < 16; ++it) {
        const int idx = it * 256 + tid;
        *reinterpret_cast<float4*>(&As[idx / 32][(idx % 32) * 4]) = d[it];
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int idx = it * 256 + tid;
        const float v[4] = {m[it].x, m[it].y, m[it].z, m[it].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (left) Bs[idx / 8][(idx % 8) * 4 + e] = v[e];
            else Bs[(idx % 32) * 4 + e][idx / 32] = v[e];
        }
    }
    __syncthreads();
    v4f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int wr = wave * 32;
    // D is lower triangular: rows wr .. wr + 31 have nothing beyond contraction index wr + 31
#pragma unroll 4
    for (int ks = 0; ks < (wr + 32) / 4; ++ks) {
        float x[2], y[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i] = As[ks * 4 + q][wr + 16 * i + l16];
#pragma unroll
        for (int j = 0; j < 2; ++j) y[j] = Bs[ks * 4 + q][16 * j + l16];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[j], acc[i][j], 0, 0, 0);
    }
    float* out = left ? a.M + (int64_t)k0 * a.Kp + c0 : a.LT + c0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(int64_t)(wr + 16 * i + 4 * q + v) * a.Kp + 16 * j + l16] = acc[i][j][v];
}

// ---------------------------------------------------------------- diagonal block

// The lower block triangle of a diagonal block in LDS: strip s (rows 16 s ..) holds its 16 (s + 1) columns at a row pitch
// that puts the four row groups of an MFMA result into different banks.
__device__ __forceinline__ int strip_pitch(int s) { return SB * (s + 1) + 4; }
__device__ __forceinline__ int strip_base(int s) { return SB * (8 * s * (s + 1) + 4 * s); }
constexpr int kStripFloats = SB * (8 * NS * (NS + 1) + 4 * NS);

struct DiagLds {
    float S[kStripFloats];
    float X[2][SB][LD];  // per step p: [contraction][column]: columns of blocks j <= p hold X_j = D S_pj (j == p: D), the others L_jp^T
};

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// x (a finished 16 x 16 diagonal block of step p, as an MFMA leaves it: column l16, rows 4 q + v) -> D, its Cholesky factor's
// inverse, into S and X; one wave.  Column j is row j as well (the block is symmetric), so the sixteen lanes of group j / 4
// hold it with the row along the lanes; scaled by 1 / L_jj, without its upper part and with zeros in the other groups, it is
// an operand whose only non-zero contraction index is j / 4, and one MFMA forms the outer product L_j L_j^T that the rest
// of the block loses -- another one L_j V_j for the inverse in the making, whose row j the same lanes hold.  No value
// travels between lanes but the pivot.
// SUBNORMAL: for pivots that are subnormal, which v_rsq_f32 takes for zero: they are moved up by 2^48 on the way.
template <bool SUBNORMAL>
__device__ __forceinline__ v4f factor_columns(v4f x)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    v4f w;
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = (4 * q + v == l16) ? 1.0f : 0.0f;
    const v4f zero = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < SB; ++j) {
        constexpr int R = SB;
        const int first = R * (j / 4);  // lane of row 0 of column j
        const float d = lane_value(x[j % 4], first + j);
        float y = SUBNORMAL && d < 0x1p-126f ? __builtin_amdgcn_rsqf(d * 0x1p48f) * 0x1p24f : __builtin_amdgcn_rsqf(d);
        y = fmaf(0.5f * y, fmaf(-d * y, y, 1.0f), y);  // (one Newton step: 1 / sqrt(d) to an ulp)
        const float r = w[j % 4] * y;
        if (j + 1 < SB) {
            const bool below = (unsigned)(lane - (first + j + 1)) < (unsigned)(R - 1 - j);
            const float l = below ? x[j % 4] * y : 0.0f;
            const float rj = (lane >> 4) == j / 4 ? r : 0.0f;
            const v4f dx = __builtin_amdgcn_mfma_f32_16x16x4f32(l, l, zero, 0, 0, 0);
            const v4f dw = __builtin_amdgcn_mfma_f32_16x16x4f32(l, rj, zero, 0, 0, 0);
            x = x - dx;
            w[j % 4] = (lane >> 4) == j / 4 ? r : w[j % 4];
            w = w - dw;
        } else {
            w[j % 4] = (lane >> 4) == j / 4 ? r : w[j % 4];
        }
    }
    return w;
}

__device__ __forceinline__ void factor_block(DiagLds& t, int p, v4f x)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    v4f w = factor_columns<false>(x);
    // (a subnormal pivot, or one that is not positive, leaves infinities or NaNs; two selects per column in the chain instead cost
    // 45 us at K = 4096)
    if (__builtin_expect(__any(!(fabsf(w[0]) + fabsf(w[1]) + fabsf(w[2]) + fabsf(w[3]) < INFINITY)), 0)) w = factor_columns<true>(x);
    float* s = t.S + strip_base(p) + 4 * q * strip_pitch(p) + SB * p + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float d = (4 * q + v >= l16) ? w[v] : 0.0f;
        s[v * strip_pitch(p)] = d;
        t.X[p & 1][4 * q + v][SB * p + l16] = d;
    }
}

// D (a row block of 16 with the contraction along the registers) times what `b` points to, 16 x 16: b[k] is the lane's column
// at contraction index 4 q + k, so an MFMA takes the contraction in the order q, q + 4, ... on both sides
__device__ __forceinline__ v4f times_d(const DiagLds& t, int p, const float (&b)[4])
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const float4 d = *reinterpret_cast<const float4*>(t.S + strip_base(p) + l16 * strip_pitch(p) + SB * p + 4 * q);
    v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.x, b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.y, b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.z, b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.w, b[3], acc, 0, 0, 0);
    return acc;
}

// L_ip^T = D S_ip^T: contraction index 4 q + v, row l16 of block row i
__device__ __forceinline__ v4f factor_rows(const DiagLds& t, int p, int i)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const float4 s = *reinterpret_cast<const float4*>(t.S + strip_base(i) + l16 * strip_pitch(i) + SB * p + 4 * q);
    const float b[4] = {s.x, s.y, s.z, s.w};
    return times_d(t, p, b);
}

// The block in t.S (its Cholesky factor's inverse replaces it), eight waves.  Wave 0 walks the serial chain: the diagonal
// block of 16 columns, its factor and inverse D, then only what the next diagonal block waits for.  The other seven take
// the rest of step p meanwhile: the seven products with D (rows of the inverse to the left, columns of the factor
// below), then the elimination of all later rows.
__device__ __forceinline__ void invert_factor(DiagLds& t)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    auto block = [&](int i, int j) { return t.S + strip_base(i) + 4 * q * strip_pitch(i) + SB * j + l16; };
    if (wave == 0) {
        v4f x;
        const float* s = block(0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = s[v * strip_pitch(0)];
        factor_block(t, 0, x);
    }
    for (int p = 0; p < NS; ++p) {
        float(*X)[LD] = t.X[p & 1];
        __syncthreads();  // D of step p is there, step p - 1 has been eliminated everywhere
        if (wave == 0) {
            v4f x = v4f{0.f, 0.f, 0.f, 0.f};
            if (p + 1 < NS) {
                const v4f l = factor_rows(t, p, p + 1);
                v4f acc = x;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(l[v], l[v], acc, 0, 0, 0);
                const float* s = block(p + 1, p + 1);
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = s[v * strip_pitch(p + 1)] - acc[v];
            }
            __syncthreads();
            if (p + 1 < NS) factor_block(t, p + 1, x);
        } else {
            const int u = wave - 1;
            if (u < p) {
                float* s = block(p, u);
                float b[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) b[v] = s[v * strip_pitch(p)];
                const v4f r = times_d(t, p, b);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[v * strip_pitch(p)] = r[v];
                    X[4 * q + v][SB * u + l16] = r[v];
                }
            } else {
                const v4f r = factor_rows(t, p, u + 1);
#pragma unroll
                for (int v = 0; v < 4; ++v) X[4 * q + v][SB * (u + 1) + l16] = r[v];
            }
            __syncthreads();
            // one block column per wave (the last two, of two tiles and one, share a wave), two tiles at a time
            for (int j = u; j < (u == NS - 2 ? NS : u + 1); ++j) {
                float xj[4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) xj[ks] = X[ks * 4 + q][SB * j + l16];
                // (the diagonal tile of row p + 1 is wave 0's)
                for (int i = max(p + 1, j) + (j == p + 1 ? 1 : 0); i < NS; i += 2) {
                    const int i2 = min(i + 1, NS - 1);
                    float* s[2] = {block(i, j), block(i2, j)};
                    const int pitch[2] = {strip_pitch(i), strip_pitch(i2)};
                    v4f old[2], acc[2];
                    float xi[2][4];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) old[e][v] = s[e][v * pitch[e]];
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) xi[e][ks] = X[ks * 4 + q][SB * (e ? i2 : i) + l16];
                        acc[e] = v4f{0.f, 0.f, 0.f, 0.f};
                        // (block column p was the factor's and becomes the inverse's: it starts from zero)
                        if (j == p) old[e] = acc[e];
                    }
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int e = 0; e < 2; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi[e][ks], xj[ks], acc[e], 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int v = 0; v < 4; ++v) s[e][v * pitch[e]] = old[e][v] - acc[e][v];
                }
            }
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------- update

// Workgroup 0: the next diagonal block (lower 16 x 16 tiles of its product only, one strip of rows per wave), then
// invert_factor; k == -1 starts the method with block 0 as it is.  The others: one 128 x 128 block each, a 64 x 32 piece per
// wave, contraction 32 at a time through LDS with the next 32 in flight.  Every product is summed from zero and subtracted
// once: with the accumulators started as M (one pass over registers less) each of the 32 MFMAs rounds at the size of M,
// towards zero, and the factor came out eight times less accurate (2.7e-4 against 3.5e-5 at K = 4096, condition 1.7e4).
__global__ __launch_bounds__(512, 4) void update_kernel(PrepArgs a)
{
    constexpr int KC = 32;
    union Lds {
        struct { float A[KC][LD]; float B[KC][LD]; } u;
        float L[NB][LD];
        DiagLds d;
    };
    __shared__ __attribute__((aligned(16))) Lds lds;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int k0 = a.k * NB, next = a.k + 1;
    if (blockIdx.x == 0) {
        __builtin_amdgcn_s_setprio(3);  // (the chain of the whole method: ahead of a neighbour's products on this compute unit)
        float* const Md = a.M + (int64_t)next * NB * (a.Kp + 1);
        // strips 0 .. 7 have 1 .. 8 tiles: a SIMD's two waves (w, w + 4) share nine
        const int strip = wave < 4 ? wave : 11 - wave;
        v4f old[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            old[j] = v4f{0.f, 0.f, 0.f, 0.f};
            if (j <= strip) {
#pragma unroll
                for (int v = 0; v < 4; ++v) old[j][v] = Md[(int64_t)(SB * strip + 4 * q + v) * a.Kp + SB * j + l16];
            }
        }
        if (a.k >= 0) {
            v4f l[8];
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int idx = it * 512 + tid;
                l[it] = *reinterpret_cast<const v4f*>(a.LT + (int64_t)(idx / 32) * a.Kp + next * NB + (idx % 32) * 4);
            }
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int idx = it * 512 + tid;
                *reinterpret_cast<v4f*>(&lds.L[idx / 32][(idx % 32) * 4]) = l[it];
            }
            __syncthreads();
            v4f acc[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
            for (int ks = 0; ks < NB / 4; ++ks) {
                const float* Lk = lds.L[ks * 4 + q] + l16;
                const float x = Lk[SB * strip];
#pragma unroll
                for (int j = 0; j < NS; ++j)
                    if (j <= strip) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, Lk[SB * j], acc[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NS; ++j) old[j] = old[j] - acc[j];
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < NS; ++j)
            if (j <= strip) {
#pragma unroll
                for (int v = 0; v < 4; ++v) lds.d.S[strip_base(strip) + (4 * q + v) * strip_pitch(strip) + SB * j + l16] = old[j][v];
            }
        __syncthreads();
        invert_factor(lds.d);
#pragma unroll 4
        for (int idx = tid; idx < NB * NB; idx += 512) {
            const int r = idx / NB, c = idx % NB;
            Md[(int64_t)r * a.Kp + c] = (c <= r) ? lds.d.S[strip_base(r / SB) + (r % SB) * strip_pitch(r / SB) + c] : 0.0f;
            a.DT[idx] = (c >= r) ? lds.d.S[strip_base(c / SB) + (c % SB) * strip_pitch(c / SB) + r] : 0.0f;  // [contraction r][row c]
        }
        return;
    }
    // block (i, j): rows next, next + 1, ... with i + 1 blocks each, the diagonal block of the first of them left out
    const int p = (int)blockIdx.x - 1 < next ? blockIdx.x - 1 : blockIdx.x;
    const int64_t n = p + (int64_t)next * (next + 1) / 2;
    int i = (int)((sqrtf(8.0f * (float)n + 1.0f) - 1.0f) * 0.5f);
    while ((int64_t)i * (i + 1) / 2 > n) --i;
    while ((int64_t)(i + 1) * (i + 2) / 2 <= n) ++i;
    const int j = (int)(n - (int64_t)i * (i + 1) / 2);
    const float* A = a.LT + i * NB;
    const float* B = (j > a.k) ? a.LT + j * NB : a.M + (int64_t)k0 * a.Kp + j * NB;
    const int wr = (wave >> 2) * 64, wc = (wave & 3) * 32;
    float* const C = a.M + (int64_t)(i * NB + wr + 4 * q) * a.Kp + j * NB + wc + l16;
    v4f acc[4][2], old[4][2];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = old[x][y] = v4f{0.f, 0.f, 0.f, 0.f};
    if (j != a.k) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int y = 0; y < 2; ++y) old[x][y][v] = C[(int64_t)(16 * x + v) * a.Kp + 16 * y];
    }
    v4f ra[2], rb[2];
    auto fetch = [&](int kc) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int idx = it * 512 + tid;
            const int64_t off = (int64_t)(kc + idx / 32) * a.Kp + (idx % 32) * 4;
            ra[it] = *reinterpret_cast<const v4f*>(A + off);
            rb[it] = *reinterpret_cast<const v4f*>(B + off);
        }
    };
    fetch(0);
    for (int kc = 0; kc < NB; kc += KC) {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int idx = it * 512 + tid;
            *reinterpret_cast<v4f*>(&lds.u.A[idx / 32][(idx % 32) * 4]) = ra[it];
            *reinterpret_cast<v4f*>(&lds.u.B[idx / 32][(idx % 32) * 4]) = rb[it];
        }
        __syncthreads();
        if (kc + KC < NB) fetch(kc + KC);
#pragma unroll
        for (int ks = 0; ks < KC / 4; ++ks) {
            float x[4], y[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = lds.u.A[ks * 4 + q][wr + 16 * e + l16];
#pragma unroll
            for (int e = 0; e < 2; ++e) y[e] = lds.u.B[ks * 4 + q][wc + 16 * e + l16];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int f = 0; f < 2; ++f) acc[e][f] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[f], acc[e][f], 0, 0, 0);
        }
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int y = 0; y < 2; ++y) C[(int64_t)(16 * x + v) * a.Kp + 16 * y] = old[x][y][v] - acc[x][y][v];
}

inline size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }
inline int64_t padded(int64_t K) { return (K + NB - 1) / NB * NB; }

}  // namespace

size_t gptq_prepare_workspace_bytes(int64_t K)
{
    // M; the panel; the diagonal block's inverse; the diagonal; the mean.  Never less than the 2.5 K^2 floats that callers of
    // this entry point are told to expect.
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
    a.LT = reinterpret_cast<float*>(ws);
    ws += (size_t)NB * Kp * 4;
    a.DT = reinterpret_cast<float*>(ws);
    ws += (size_t)NB * NB * 4;
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
    hipLaunchKernelGGL(update_kernel, dim3(1), dim3(512), 0, st, a);
    for (a.k = 0; a.k < a.nt; ++a.k) {
        if (a.nt > 1) hipLaunchKernelGGL(panel_kernel, dim3((unsigned)((a.nt - 1) * (NB / PW))), dim3(256), 0, st, a);
        if (a.k + 1 == a.nt) break;
        const int64_t tiles = (int64_t)a.nt * (a.nt + 1) / 2 - (int64_t)(a.k + 1) * (a.k + 2) / 2;
        // Up to two blocks per compute unit the chain in workgroup 0 is the longer side, and unused dynamic LDS that keeps a
        // second workgroup off its compute unit shortens it (41 -> 34 us at 390 blocks); with more blocks two per unit win.
        const unsigned lone = tiles <= 2 * compute_units() ? 12288 : 0;
        hipLaunchKernelGGL(update_kernel, dim3((unsigned)tiles), dim3(512), lone, st, a);
    }
    hipLaunchKernelGGL(reverse_kernel, dim3((unsigned)K), dim3(256), 0, st, (const float*)a.M, K, (int)Kp, U);
    return hipGetLastError();
}

}  // namespace fp4mr
