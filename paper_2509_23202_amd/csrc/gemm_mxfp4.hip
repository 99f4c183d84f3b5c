// MXFP4 W4A4 GEMM on the CDNA4 block-scaled FP4 MFMA (arXiv 2509.23202, Section 4.2 item 2: the FP4 matmul
// Q(W H) Q(X H)^T with hardware-applied group scales).
//
//   out[m,n] = sum_k  2^(sa[m,k/32]-127) * 2^(sw[n,k/32]-127) * a[m,k] * w[n,k]
//
// v_mfma_scale_f32_16x16x128_f8f6f4 multiplies a 16x128 by a 128x16 FP4 tile; every lane supplies 32 consecutive
// K-elements of one row (16 bytes) and one E8M0 byte that scales exactly those 32 elements -- the MXFP4 group.
// Both operands arrive in "GEMM layout": 1 KB fragments already in lane order (layout.hpp), so a fragment moves
// global -> LDS with one 16-byte direct-to-LDS load per lane and LDS -> registers with one conflict-free
// ds_read_b128 per lane; no re-layout pass runs between the quantizer and the GEMM.  (Direct-to-LDS loads write
// lane l's bytes at LDS base + 16*l, which is exactly the fragment order.)
//
// Roles are swapped on purpose: the W fragment is the MFMA's A operand (rows = n) and the X fragment its B
// operand (columns = m).  A lane then owns four consecutive n of one m, i.e. one 8-byte bf16x4 store.
//
// Block tile BM x BN, K-step 128, STAGES-deep LDS ring fed by direct-to-LDS loads (tracked with vmcnt), one
// barrier per K-step, or per two with eight stages.  Scales take the same route into a single LDS buffer: with four and more stages one 16-byte
// copy per pair of row-blocks and 8 K-steps, with three stages one 4-byte copy per row-block and 4 K-steps.
#include "device_util.hpp"
#include "internal.hpp"
#include "layout.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

namespace fp4mr {
namespace {

struct GemmArgs {
    const uint8_t* a_codes;
    const uint8_t* a_scales;
    const uint8_t* w_codes;
    const uint8_t* w_scales;
    void* out;
    int64_t M, N, K;
    int tiles_m, tiles_n;
    float alpha;  // factor on the result: powers of 4/3 for operands whose scales carry the tensor-level 4/3, else 1
    int split_steps;  // split-K launches: K-steps per split (a multiple of 8); blockIdx.y is the split, out the fp32 partials
};

typedef const __attribute__((address_space(1))) void global_void;

template <int OPSEL>
__device__ __forceinline__ v4f mfma_fp4(const v4i& a, const v4i& b, const v4f& c, uint32_t sa, uint32_t sb)
{
    const v8i a8 = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
    const v8i b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
    // cbsz = blgp = 4: both operands E2M1.  op_sel picks byte OPSEL of each scale register.
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a8, b8, c, 4, 4, OPSEL, (int)sa, OPSEL, (int)sb);
}

__device__ __forceinline__ void remap_block(int bid, int nblocks, int tiles_m, int tiles_n, int& tm, int& tn)
{
    // Workgroups are dealt round-robin to the 8 XCDs.  Give every XCD one contiguous range of logical tile
    // ids, and order logical ids in bands of GM tile-rows, so the tiles that share an L2 share operands.
    const int per = nblocks >> 3, rem = nblocks & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    const int L = (xcd < rem) ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    constexpr int GM = 4;
    const int band = GM * tiles_n;
    const int gidx = L / band;
    const int first_m = gidx * GM;
    const int gsz = min(tiles_m - first_m, GM);
    const int in_band = L - gidx * band;
    tm = first_m + in_band % gsz;
    tn = in_band / gsz;
}

// Four-wave workgroups with a three-stage ring are sized so that two of them share a compute unit (registers: 256 per
// wave; LDS: under 80 KB): while one converts and stores its tile the other keeps the matrix pipes busy.
template <int BM, int BN, int WM, int WN, int STAGES>
constexpr int kWgsPerCu = ((BM / WM) * (BN / WN) == 4 && STAGES == 3) ? 2 : 1;

template <int BM, int BN, int WM, int WN, int STAGES, bool OUT_F32, int RD = 2, bool PERSIST = false, bool SPLITK = false>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) __attribute__((amdgpu_waves_per_eu(kWgsPerCu<BM, BN, WM, WN, STAGES>)))
void gemm_mx_kernel(GemmArgs g)
{
    constexpr int NWM = BM / WM, NWN = BN / WN, NW = NWM * NWN;
    constexpr int FX = BM / 16, FW = BN / 16, F = FX + FW;  // fragments per stage
    constexpr int LPW = (F + NW - 1) / NW;                  // fragment loads per wave per stage
    constexpr int TM = WM / 16, TN = WN / 16;               // MFMA tiles per wave
    constexpr int STAGE_BYTES = F * 1024;
    // PAIR: one barrier, and one wait for LDS reads, per two K-steps, for a stage less on its way (128 x 128 tiles, N = 4096, M = 400:
    // K = 4096 11.2 -> 10.5 us, 14336 27.8 -> 26.2, of which 11 ns a step; with six or seven stages the stages missing cost more than that).
    constexpr bool PAIR = STAGES == 8 && !PERSIST;
    constexpr int LEAD = PAIR ? STAGES - 2 : STAGES - 1;    // a step requests the stage that many steps behind its own
    static_assert(STAGES >= 3 && STAGES <= 8, "ring bookkeeping is written for 3 to 8 stages");

    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int lane = threadIdx.x & 63;
    // the wave index is uniform across the wavefront: telling the compiler keeps every fragment base address,
    // LDS offset and tile coordinate in scalar registers (the vector file is needed for accumulators and fragments)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave % NWM, wn = wave / NWM;
    const uint32_t lane16 = (uint32_t)lane * 16u, lane4 = (uint32_t)lane * 4u;

    // PERSIST: the grid is one workgroup per compute unit and a workgroup walks the tiles blockIdx.x,
    // blockIdx.x + gridDim.x, ...; otherwise the grid has one workgroup per tile and the loop below runs once.
    const int ntiles = g.tiles_m * g.tiles_n;
    int tile = blockIdx.x;

    const int64_t KC = g.K >> 7;            // K-steps (of a row-block in memory)
    const int64_t KS = (g.K + 511) >> 9;    // scale super-steps (likewise)
    // SPLITK: this workgroup multiplies K-steps kt0 .. kt0 + KT - 1 only (kt0 a multiple of 8: whole scale batches) and
    // writes its fp32 partial tile to slice blockIdx.y of the output, which a reduction kernel adds up in split order
    static_assert(!SPLITK || (OUT_F32 && !PERSIST), "split-K workgroups write fp32 partials, one tile each");
    const int kt0 = SPLITK ? (int)blockIdx.y * g.split_steps : 0;
    const int KT = SPLITK ? min(g.split_steps, (int)KC - kt0) : (int)KC;
    const int KS_rem = (int)KS - (kt0 >> 2);  // scale blocks from kt0 to the end of K

    // Operands are addressed through buffer resources: one VGPR (16 * lane) is the only per-lane address and every
    // fragment's position is a scalar offset.  Row-blocks past the end of an operand (last tile) are clamped to its
    // last row-block: the duplicates only feed output rows / columns that are never stored.
    const int a_rbs = (int)((g.M + 15) / 16), w_rbs = (int)((g.N + 15) / 16);
    auto make_rsrc = [](const uint8_t* base, int64_t bytes) {
        const uint32_t n = bytes > 0xffffffffll ? 0xffffffffu : (uint32_t)bytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), 0, (int)n, 0x00020000);
    };
    // bases at the tile's first row-block keep every scalar offset far below 2^31
    int tm, tn;                  // tile whose operands the loads below address
    __amdgpu_buffer_rsrc_t rs_ac, rs_wc, rs_as, rs_ws;
    int a_rb_last, w_rb_last;    // largest valid row-block relative to the base
    auto set_tile = [&](int t) {
        remap_block(t, ntiles, g.tiles_m, g.tiles_n, tm, tn);
        const int a_rb0 = min(tm * FX, a_rbs - 1), w_rb0 = min(tn * FW, w_rbs - 1);
        const int64_t c0 = (int64_t)kt0 * 1024, s0 = (int64_t)(kt0 >> 2) * 256;  // (0 unless SPLITK)
        rs_ac = make_rsrc(g.a_codes + (int64_t)a_rb0 * KC * 1024 + c0, (int64_t)(a_rbs - a_rb0) * KC * 1024 - c0);
        rs_wc = make_rsrc(g.w_codes + (int64_t)w_rb0 * KC * 1024 + c0, (int64_t)(w_rbs - w_rb0) * KC * 1024 - c0);
        rs_as = make_rsrc(g.a_scales + (int64_t)a_rb0 * KS * 256 + s0, (int64_t)(a_rbs - a_rb0) * KS * 256 - s0);
        rs_ws = make_rsrc(g.w_scales + (int64_t)w_rb0 * KS * 256 + s0, (int64_t)(w_rbs - w_rb0) * KS * 256 - s0);
        a_rb_last = a_rbs - 1 - a_rb0;
        w_rb_last = w_rbs - 1 - w_rb0;
    };
    set_tile(tile);

    // Scales: every (row-block, 4 K-steps) owns 256 bytes = one dword per lane.  They travel global -> LDS with
    // direct-to-LDS loads (so no VGPR is ever the target of an in-flight load inside the main loop) and are read back
    // once per 4 K-steps.
    //   SC8 (four and more stages): a batch is 8 K-steps.  One 16-byte-per-lane copy fetches 512 bytes (two
    //   consecutive 4-step blocks) of TWO row-blocks -- lanes 0..31 the first, lanes 32..63 the second; the address is
    //   per lane, the LDS side is base + 16 * lane -- so a workgroup needs (FX + FW) / 2 copies per 8 K-steps instead of
    //   2 * (FX + FW) four-byte ones.  The vector-memory path is a co-limiter of this loop (extra address traffic
    //   measured far more expensive than its bytes), which is what this saves.  One buffer: the batch of steps
    //   8b+8 .. 8b+15 is requested in step 8b+4, after every wave has read the second half of batch b into registers
    //   (end of step 8b+3, then that step's barrier), and it has landed before the read at the end of step 8b+7
    //   (loads complete in order, and step 8b+7 has waited for the stage requested in step 8b+5).
    //   Otherwise (three stages): 4-byte copies, a batch is 4 K-steps.
    constexpr bool SC8 = STAGES >= 4;
    constexpr int XP = (FX + 1) / 2, WP = (FW + 1) / 2;    // pairs of row-blocks
    constexpr int NS = SC8 ? (XP + WP + NW - 1) / NW : LPW; // scale loads per wave per batch
    constexpr int SCALE_BYTES = SC8 ? (XP + WP) * 1024 : F * 256;
    static_assert(NS <= LPW, "a scale load is issued in front of a fragment load of the same step");
    // One scale buffer up to five stages.  From six stages on the stage a step waits for was requested more than four steps
    // earlier, so a batch requested in step 8b+4 would no longer be covered by the wait of step 8b+7 (loads complete in
    // issue order: a wait for stage kt+1 covers what was requested before it): the batch is then requested in step 8b+0,
    // into the other of TWO buffers (the one whose batch was last read at the end of step 8b-5).
    constexpr int SD = (SC8 && STAGES >= 6) ? 2 : 1;
    char* const scale_ring = smem + STAGES * STAGE_BYTES;
    const int kc_bytes = (int)KC * 1024, ks_bytes = (int)KS * 256;

    v4f acc[TN][TM];
    uint32_t sx[TM], sw[TN];
    // Software pipeline of the LDS reads: the X fragments of step kt+1 are read into the other half of xf[2][.]
    // while step kt computes, and the W fragments run through a 4-deep register ring two groups of TM MFMAs ahead
    // of their use -- so no MFMA waits on LDS latency, at a cost of 2*TM*4 + 16 fragment registers.
    // W-fragment register ring; RD = how many MFMA groups ahead it is filled (three or two slots when TN is not a multiple of 4)
    constexpr int RING = TN == 2 ? 2 : (TN % 4 != 0) ? 3 : 4;
    v4i xf[2][TM], wring[RING];
    static_assert(TN % RING == 0 && RD < RING && RD <= TN, "the W-fragment ring index must be static");
    // every wave issues exactly LPW fragment loads per stage and NS scale loads per batch so that the vmcnt
    // bookkeeping is uniform; when F is not a multiple of NW the spare slots re-copy the last fragment (same bytes
    // to the same place)
    // which operand load slot i of this wave belongs to: known at compile time (i is a constant after unrolling)
    // whenever the X fragments divide evenly among the waves, which keeps the step body free of branches
    auto is_x = [&](int f, int i) { return (FX % NW == 0) ? (i < FX / NW) : (f < FX); };
    auto issue_scale_one = [&](int ss, int i) {
        if constexpr (SC8) {
            // ss = the batch: 4-step blocks 2 * ss and 2 * ss + 1 (past the end: the last block again; what lies behind it
            // in the 512 bytes is never used, and reads beyond the operand return zeros)
            const int blk = min(2 * ss, KS_rem - 1);
            const int p = min(wave + i * NW, XP + WP - 1);
            const uint32_t half = (uint32_t)lane >> 5, col = ((uint32_t)lane & 31u) * 16u;
            if ((XP % NW == 0) ? (i < XP / NW) : (p < XP)) {
                const uint32_t rb = (uint32_t)min(2 * p + (int)half, a_rb_last);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_as, (lds_void*)(scale_ring + (SD == 2 ? (ss & 1) * SCALE_BYTES : 0) + p * 1024), 16, rb * (uint32_t)ks_bytes + col, blk * 256, 0, 0);
            } else {
                const uint32_t rb = (uint32_t)min(2 * (p - XP) + (int)half, w_rb_last);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ws, (lds_void*)(scale_ring + (SD == 2 ? (ss & 1) * SCALE_BYTES : 0) + p * 1024), 16, rb * (uint32_t)ks_bytes + col, blk * 256, 0, 0);
            }
            return;
        }
        char* base = scale_ring;
        ss = ss < KS_rem ? ss : KS_rem - 1;  // the batch past the end re-reads the last one
        const int f = min(wave + i * NW, F - 1);
        if (is_x(f, i)) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_as, (lds_void*)(base + f * 256), 4, lane4, min(f, a_rb_last) * ks_bytes + ss * 256, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ws, (lds_void*)(base + f * 256), 4, lane4, min(f - FX, w_rb_last) * ks_bytes + ss * 256, 0, 0);
    };
    auto issue_frag_one = [&](int kt, char* base, int i) {
        const int f = min(wave + i * NW, F - 1);
        if (is_x(f, i)) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ac, (lds_void*)(base + f * 1024), 16, lane16, min(f, a_rb_last) * kc_bytes + kt * 1024, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_wc, (lds_void*)(base + f * 1024), 16, lane16, (min(f - FX, w_rb_last)) * kc_bytes + kt * 1024, 0, 0);
    };
    auto issue_scales = [&](int ss) {
#pragma unroll
        for (int i = 0; i < NS; ++i) issue_scale_one(ss, i);
    };
    auto read_scales = [&](int64_t ss, uint32_t (&dx)[TM], uint32_t (&dw)[TN]) {  // ss = 4-step block
        if constexpr (SC8) {
            // a row-block's 512 bytes: even block, odd block (two buffers: batch ss / 2 is in buffer (ss / 2) % 2)
            const char* base = scale_ring + (SD == 2 ? (int)((ss >> 1) & 1) * SCALE_BYTES : 0) + (ss & 1) * 256;
#pragma unroll
            for (int j = 0; j < TM; ++j) dx[j] = *(reinterpret_cast<const uint32_t*>(base + (wm * TM + j) * 512) + lane);
#pragma unroll
            for (int i = 0; i < TN; ++i) dw[i] = *(reinterpret_cast<const uint32_t*>(base + (2 * XP + wn * TN + i) * 512) + lane);
        } else {
            const char* base = scale_ring;
#pragma unroll
            for (int j = 0; j < TM; ++j) dx[j] = *(reinterpret_cast<const uint32_t*>(base + (wm * TM + j) * 256) + lane);
#pragma unroll
            for (int i = 0; i < TN; ++i) dw[i] = *(reinterpret_cast<const uint32_t*>(base + (FX + wn * TN + i) * 256) + lane);
        }
    };
    auto read_x = [&](int kt, auto ptag, int j) {
        constexpr int P = decltype(ptag)::value;
        xf[P][j] = *(reinterpret_cast<const v4i*>(smem + (kt % STAGES) * STAGE_BYTES + (wm * TM + j) * 1024) + lane);
    };
    auto read_w = [&](int kt, int i) {  // into ring slot i % 4 (i is a compile-time constant after unrolling)
        wring[i % RING] = *(reinterpret_cast<const v4i*>(smem + (kt % STAGES) * STAGE_BYTES + (FX + wn * TN + i) * 1024) + lane);
    };

    // prologue of a tile: scales of super-step 0 and LEAD stages on their way into ring slots 0 .. LEAD-1
    auto issue_prologue = [&]() {
        issue_scales(0);
#pragma unroll
        for (int s = 0; s < LEAD; ++s) {
#pragma unroll
            for (int i = 0; i < LPW; ++i) issue_frag_one(min(s, KT - 1), smem + s * STAGE_BYTES, i);
        }
    };
    issue_prologue();
    wait_vmcnt<(LEAD - 1) * LPW>();

    // One K-step.  J = kt % 8 (SC8) or kt % 4: J & 3 selects the scale byte (op_sel), J & 1 the X register half.
    //   top:    stage kt+1 must have landed (this wave's copies: vmcnt; everybody's: barrier).  The same barrier
    //           says that every wave is done reading stage kt-1, whose LDS buffer is refilled with stage kt+STAGES-1.
    //   vmcnt:  allowed in flight = the STAGES-3 stages after kt+1, plus one scale batch when it was issued after
    //           stage kt+1's loads (batches go out at J == 0, ahead of that step's fragment loads).
    // PAIR: an even step waits for the stages kt+1 and kt+2 of itself and of the odd step behind it, which has no wait of its own; the
    // barrier says that stages kt-2 and kt-1 have been read, whose slots the two steps refill with stages kt+STAGES-2 and
    // kt+STAGES-1; STAGES-5 stages may be in flight.  A scale batch (requested in step 8b) has landed for step 8b+6.
    constexpr int NST = TM * (16 * (WN / 8) / 64);  // store instructions a wave issues for one interior output tile
    static_assert((STAGES - 2) * LPW + NST < 64 && (STAGES - 3) * LPW + NS + NST < 64, "vmcnt is a 6-bit counter");
    bool pend = false;  // persistent workgroups: the previous tile's stores may be outstanding at the top of this tile
    constexpr int XPG = (TM + TN - 1) / TN;  // X-fragment reads folded in front of each group of TM MFMAs
    // The LDS reads for "the next step" are unconditional: in the very last step they fetch stale bytes of the ring
    // that nothing consumes, which keeps the step body free of branches (and of a second copy of the code).
    auto step = [&](int kt, auto jtag, auto wtag) {
        constexpr int J = decltype(jtag)::value;
        constexpr int SKEW = (2 * decltype(wtag)::value) % TM;  // MFMA index inside a group after which this wave issues its loads
        constexpr int P = J & 1;
        constexpr int JB = (SC8 && SD == 1) ? 4 : 0;  // the step of a period that requests the next scale batch
        constexpr int PER = SC8 ? 8 : 4;                // steps per scale batch
        // the batch was requested 1 .. FLYING steps ago, i.e. behind the loads of the stage this step waits for
        constexpr int FLYING = PAIR ? STAGES - 5 : STAGES - 3;
        constexpr bool batch_after = ((J - JB - 1 + PER) % PER) <= FLYING - 1;
        constexpr int ALLOWED = FLYING * LPW + (batch_after ? NS : 0);
        if constexpr (PERSIST && J <= STAGES - 3) {
            // first steps of a follow-on tile, as long as the stage they wait for (kt + 1) is one of the STAGES - 1 that
            // were prefetched: the previous tile's NST output stores were issued after those and may still be in flight
            // (vector memory operations complete in issue order, so the stages in front of the stores can be waited for
            // without waiting for the stores)
            if (pend && kt <= STAGES - 3) wait_vmcnt<ALLOWED + NST>(); else wait_vmcnt<ALLOWED>();
        } else if constexpr (!PAIR || J % 2 == 0) {
            wait_vmcnt<ALLOWED>();
        }
        if constexpr (!PAIR || J % 2 == 0) {
            wait_lgkmcnt0();
            block_barrier();
        }
        // The global -> LDS loads of stage kt+LEAD (and, at J == 0, of the next scale batch) are spread over the
        // groups of MFMAs: a wave issues in order, and a burst of vector-memory instructions at the top of the step
        // would hold its MFMAs back while the CU's single address unit works through all four waves' bursts.
        // Past the last stage the loads re-copy stage KT-1 into a ring slot nobody reads any more: the step body stays
        // free of branches (which would let the compiler pull the MFMAs away from the loads they are meant to cover)
        // and the vmcnt bookkeeping needs no special case for the tail.
        const int kt_load = min(kt + LEAD, KT - 1);
        char* const load_base = smem + ((kt + LEAD) % STAGES) * STAGE_BYTES;
        constexpr int DPG = (LPW + TN - 1) / TN;  // loads per group
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            // W fragment two groups ahead (wraps into the next step), X fragments of the next step
            if (i + RD < TN) read_w(kt, i + RD);
            else read_w(kt + 1, i + RD - TN);
#pragma unroll
            for (int j = i * XPG; j < (i + 1) * XPG && j < TM; ++j) read_x(kt + 1, std::integral_constant<int, 1 - P>{}, j);
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                acc[i][j] = mfma_fp4<(J & 3)>(wring[i % RING], xf[P][j], acc[i][j], sw[i], sx[j]);
                if (j == SKEW) {
                    // the four waves of a workgroup run in lockstep (one barrier per step); issuing their loads at
                    // different points of the group keeps them from queueing up behind each other at the CU's one
                    // address unit while their MFMA pipes run dry
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int d = i * DPG; d < (i + 1) * DPG && d < LPW; ++d) {
                        if constexpr (J == JB) {
                            if (d < NS) issue_scale_one(SC8 ? (kt >> 3) + 1 : (kt >> 2) + 1, d);
                        }
                        issue_frag_one(kt_load, load_base, d);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // keep the instruction scheduler from hoisting the later groups' LDS reads up here: that would rebuild a
            // full second copy of the W fragments in registers
            __builtin_amdgcn_sched_barrier(0);
        }
        // scales of the next four steps (their batch landed before this step's barrier)
        if constexpr ((J & 3) == 3) read_scales((kt >> 2) + 1, sx, sw);
    };

    auto main_loop = [&](auto wtag) {
        for (int kt0 = 0; kt0 < KT; kt0 += (SC8 ? 8 : 4)) {
            step(kt0, std::integral_constant<int, 0>{}, wtag);
            if (kt0 + 1 < KT) step(kt0 + 1, std::integral_constant<int, 1>{}, wtag);
            if (kt0 + 2 < KT) step(kt0 + 2, std::integral_constant<int, 2>{}, wtag);
            if (kt0 + 3 < KT) step(kt0 + 3, std::integral_constant<int, 3>{}, wtag);
            if constexpr (SC8) {
                if (kt0 + 4 < KT) step(kt0 + 4, std::integral_constant<int, 4>{}, wtag);
                if (kt0 + 5 < KT) step(kt0 + 5, std::integral_constant<int, 5>{}, wtag);
                if (kt0 + 6 < KT) step(kt0 + 6, std::integral_constant<int, 6>{}, wtag);
                if (kt0 + 7 < KT) step(kt0 + 7, std::integral_constant<int, 7>{}, wtag);
            }
        }
    };

    // The epilogue transposes 16 output rows of the wave tile at a time through a staging area in the last ring
    // slot; the other slots are free for the next tile's prologue loads while the stores drain.
    constexpr int CPR = WN / 8;                  // 16-byte chunks per staged row
    constexpr int STAGING = 16 * WN * 2;         // bytes per wave
    constexpr bool STAGED = !OUT_F32 && NW * STAGING <= STAGE_BYTES && (CPR == 8 || CPR == 12 || CPR == 16);
    constexpr int SWZ = (CPR == 12) ? 3 : CPR - 1;  // chunk swizzle mask: XOR stays inside an aligned group of SWZ + 1 chunks

    for (;;) {
        // stage 0 and the first scale batch have landed (this wave's copies: the vmcnt wait before this point)
        block_barrier();
        read_scales(0, sx, sw);
#pragma unroll
        for (int j = 0; j < TM; ++j) read_x(0, std::integral_constant<int, 0>{}, j);
#pragma unroll
        for (int i = 0; i < RD; ++i) read_w(0, i);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

        if constexpr (SC8) {
            // (the eight-step period doubles the loop body: one copy of it, every wave issuing its loads at the same
            // point of an MFMA group; the per-wave skew below measured within noise)
            main_loop(std::integral_constant<int, 0>{});
        } else {
            switch (wave & 3) {
                case 0: main_loop(std::integral_constant<int, 0>{}); break;
                case 1: main_loop(std::integral_constant<int, 1>{}); break;
                case 2: main_loop(std::integral_constant<int, 2>{}); break;
                default: main_loop(std::integral_constant<int, 3>{}); break;
            }
        }
        wait_vmcnt<0>();  // the clamped loads of the last steps
        wait_lgkmcnt0();
        block_barrier();  // every wave is done with the operand ring, and nothing is in flight into it

        const int64_t m0 = (int64_t)tm * BM + wm * WM, n0 = (int64_t)tn * BN + wn * WN;  // this wave's output tile
        const bool interior = (int64_t)(tm + 1) * BM <= g.M && (int64_t)(tn + 1) * BN <= g.N;  // no lane is masked off
        const int next = tile + (int)gridDim.x;
        const bool more = PERSIST && next < ntiles;
        pend = false;
        if (more) {
            // the next tile's first stages travel while this tile's results are converted and stored
            set_tile(next);
            issue_prologue();
        }

        // A lane owns out[m][n..n+3] with m = m0 + 16*j + lane%16, n = n0 + 16*i + 4*(lane/16): stored directly that
        // is 16 rows x 32 bytes per instruction.  For bf16 output the rows go through LDS first so that every store
        // instruction writes 16 bytes per lane in whole rows.  A staged row is WN*2 bytes with its 16-byte chunks
        // XOR-swizzled by the row number: the 8-byte writes of a half-wave and the 16-byte reads of a quarter-wave
        // then both spread over all banks.
        // the lane-dependent address arithmetic of the epilogue is tied to a value defined here, so that the compiler
        // cannot hoist it above the tile loop and carry it (in registers the main loop needs) through every K-step
        int el = lane;
        asm volatile("" : "+v"(el));
        if (g.alpha != 1.0f) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) acc[i][j] *= g.alpha;
        }
        if (STAGED && (g.N & 7) == 0) {
            char* const mine = smem + (STAGES - 1) * STAGE_BYTES + wave * STAGING;
            typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
            const int wr = el & 15, wq = el >> 4;
#pragma unroll
            for (int j = 0; j < TM; ++j) {
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const v4f v = acc[i][j];
                    const v4bf p = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                    const int ch = (2 * i + (wq >> 1)) ^ (wr & SWZ);
                    *reinterpret_cast<v4bf*>(mine + wr * (WN * 2) + ch * 16 + (wq & 1) * 8) = p;
                }
#pragma unroll
                for (int it = 0; it < 16 * CPR / 64; ++it) {
                    const int c = it * 64 + el;
                    const int row = c / CPR, ch = c % CPR;
                    const v4i v = *reinterpret_cast<const v4i*>(mine + row * (WN * 2) + ((ch ^ (row & SWZ)) * 16));
                    const int64_t m = m0 + 16 * j + row, n = n0 + ch * 8;
                    // an interior tile issues exactly NST stores per wave (what the follow-on tile's vmcnt allowance counts)
                    if (interior || (m < g.M && n < g.N)) __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(static_cast<__bf16*>(g.out) + m * g.N + n));
                }
            }
            pend = more && interior;
        } else {
            // direct stores (fp32 output, or N not a multiple of 8)
            const int64_t m_base = m0 + (el & 15);
            const int64_t n_base = n0 + (el >> 4) * 4;
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const int64_t m = m_base + 16 * j;
                if (m >= g.M) continue;
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int64_t n = n_base + 16 * i;
                    if (n >= g.N) continue;
                    const v4f v = acc[i][j];
                    if constexpr (OUT_F32) {
                        float* o = static_cast<float*>(g.out) + (SPLITK ? (int64_t)blockIdx.y * g.M * g.N : 0) + m * g.N + n;
                        if (n + 3 < g.N && (g.N & 3) == 0) {
                            *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
                        } else {
                            for (int e = 0; e < 4; ++e)
                                if (n + e < g.N) o[e] = v[e];
                        }
                    } else {
                        __bf16* o = static_cast<__bf16*>(g.out) + m * g.N + n;
                        typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
                        if (n + 3 < g.N && (g.N & 3) == 0) {
                            v4bf p = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                            *reinterpret_cast<v4bf*>(o) = p;
                        } else {
                            for (int e = 0; e < 4; ++e)
                                if (n + e < g.N) o[e] = (__bf16)v[e];
                        }
                    }
                }
            }
        }
        if (!more) break;
        tile = next;
        // Stage 0 and the scale batch of the next tile were issued before this tile's stores: after an interior tile
        // (exact store count) wait for them only and let the stores drain under the first K-steps; otherwise wait for
        // everything.
        if (pend) wait_vmcnt<(STAGES - 2) * LPW + NST>(); else wait_vmcnt<0>();
    }
}


// out[i] = alpha * (partial[0][i] + partial[1][i] + ...), the splits added in their order (deterministic), as bf16 or fp32; V
// neighbouring values per thread (four where mn and `partial` allow it), all splits' loads on their way together
template <bool OUT_F32, int V>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int64_t mn, float alpha, void* out)
{
    constexpr int kMost = 8;   // splits (plan_mx)
    typedef float vec __attribute__((ext_vector_type(V)));
    typedef __bf16 vecb __attribute__((ext_vector_type(V)));
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= mn) return;
    vec x[kMost];
#pragma unroll
    for (int p = 0; p < kMost; ++p)
        if (p < splits) x[p] = *reinterpret_cast<const vec*>(partial + (int64_t)p * mn + i);
    vec s = x[0];
#pragma unroll
    for (int p = 1; p < kMost; ++p)
        if (p < splits) s += x[p];
    s *= alpha;
    if constexpr (OUT_F32) *reinterpret_cast<vec*>(static_cast<float*>(out) + i) = s;
    else *reinterpret_cast<vecb*>(static_cast<__bf16*>(out) + i) = __builtin_convertvector(s, vecb);
}

template <int V>
void launch_splitk_reduce(const float* partial, int splits, int64_t mn, float alpha, void* out, bool out_f32, hipStream_t st)
{
    const dim3 grid((unsigned)((mn + 256 * V - 1) / (256 * V)));
    if (out_f32) hipLaunchKernelGGL((splitk_reduce_kernel<true, V>), grid, dim3(256), 0, st, partial, splits, mn, alpha, out);
    else hipLaunchKernelGGL((splitk_reduce_kernel<false, V>), grid, dim3(256), 0, st, partial, splits, mn, alpha, out);
}

// the tile shapes that have a split-K instantiation: the small ones, and with four stages 128 x 128, 256 x 128 and 256 x 256
constexpr bool tile_splits(int bm, int bn, int stages) { return (bm <= 96 && bn <= 128) || (stages == 4 && ((bm == 128 && bn == 128) || (bm == 256 && bn != 192))); }

// splits > 1: every tile is computed by `splits` workgroups, split y taking K-steps y * split_steps .. and writing its
// fp32 partial tile to slice y of `partial`; the caller then runs splitk_reduce_kernel
template <int BM, int BN, int WM, int WN, int STAGES, int RD = 2, bool PERSIST = false>
hipError_t launch_variant(const GemmArgs& g0, bool out_f32, hipStream_t st, int splits = 1, int split_steps = 0, float* partial = nullptr)
{
    GemmArgs g = g0;
    g.tiles_m = (int)((g.M + BM - 1) / BM);
    g.tiles_n = (int)((g.N + BN - 1) / BN);
    if (splits > 1) {
        if constexpr (tile_splits(BM, BN, STAGES)) {
            constexpr int threads_s = (BM / WM) * (BN / WN) * 64;
            constexpr size_t lds_s = (size_t)STAGES * (BM + BN) / 16 * 1024 +
                                     (STAGES >= 4 ? (size_t)((BM / 16 + 1) / 2 + (BN / 16 + 1) / 2) * 1024 * (STAGES >= 6 ? 2 : 1) : (size_t)(BM + BN) / 16 * 256);
            g.out = partial;
            g.alpha = 1.0f;
            g.split_steps = split_steps;
            static LdsAttrOnce raised_s;
            auto k = gemm_mx_kernel<BM, BN, WM, WN, STAGES, true, RD, false, true>;
            hipError_t es;
            if ((es = raised_s.ensure(reinterpret_cast<const void*>(k), (int)lds_s)) != hipSuccess) return es;
            hipLaunchKernelGGL(k, dim3((unsigned)(g.tiles_m * g.tiles_n), (unsigned)splits), dim3(threads_s), lds_s, st, g);
            if ((es = hipGetLastError()) != hipSuccess) return es;
            const int64_t mn = g.M * g.N;
            if (mn % 4 == 0) launch_splitk_reduce<4>(partial, splits, mn, g0.alpha, g0.out, out_f32, st);   // (both buffers begin at multiples of 16 bytes)
            else launch_splitk_reduce<1>(partial, splits, mn, g0.alpha, g0.out, out_f32, st);
            return hipGetLastError();
        } else {
            return hipErrorInvalidValue;
        }
    }
    constexpr int threads = (BM / WM) * (BN / WN) * 64;
    // operand ring + scale buffer (four and more stages: 1 KB per pair of row-blocks; three stages: 256 B per row-block)
    constexpr size_t lds = (size_t)STAGES * (BM + BN) / 16 * 1024 +
                           (STAGES >= 4 ? (size_t)((BM / 16 + 1) / 2 + (BN / 16 + 1) / 2) * 1024 * (STAGES >= 6 ? 2 : 1) : (size_t)(BM + BN) / 16 * 256);
    const int ntiles = g.tiles_m * g.tiles_n;
    int nwg = ntiles;
    if (PERSIST) {
        nwg = std::min(ntiles, compute_units() * kWgsPerCu<BM, BN, WM, WN, STAGES>);
        // the grid cap option (a testing aid: a small grid walks many tiles per workgroup)
        if (options().gemm_grid > 0) nwg = std::min(nwg, options().gemm_grid);
    }
    const dim3 grid((unsigned)nwg);
    hipError_t e;
    // the dynamic-LDS limit of a kernel is raised once per device, not on every launch
    static LdsAttrOnce raised[2];
    if (out_f32) {
        auto k = gemm_mx_kernel<BM, BN, WM, WN, STAGES, true, RD, PERSIST>;
        if ((e = raised[1].ensure(reinterpret_cast<const void*>(k), (int)lds)) != hipSuccess) return e;
        hipLaunchKernelGGL(k, grid, dim3(threads), lds, st, g);
    } else {
        auto k = gemm_mx_kernel<BM, BN, WM, WN, STAGES, false, RD, PERSIST>;
        if ((e = raised[0].ensure(reinterpret_cast<const void*>(k), (int)lds)) != hipSuccess) return e;
        hipLaunchKernelGGL(k, grid, dim3(threads), lds, st, g);
    }
    return hipGetLastError();
}

// What a launch of one of the tile shapes takes: rounds of workgroups over the chip times (a tile's fixed cost + K-steps times a
// step, which grows with the share of the chip that is busy), in microseconds; more where the output's rows are not whole
// 64-byte pieces (their stores share lines with the next row: a quarter of the launch at M = 4085, N = 9224, K = 1024).  Fitted to
// launches of every shape on 806 products with cold weights (as many copies in turn as fill 400 MB: what a model's layers see)
// and, at a fifth of the weight, 873 with the same weights again and again (M = 65 ... 4096, N = 1024 ... 57344, K = 512 ... 28672), for
// the choice to lose least.  On products left out of the fit the tile taken is slower than the best of all by 0.3 % on average (97
// cold ones; 7 % at most) and 0.8 % (139 warm ones; 9 %).  (A fit to warm weights alone took 128 x 128 and 160 x 128 tiles with four stages where the
// eight-stage ring keeps twice the bytes in flight: N = K = 8192, M = 394, cold: 22.3 -> 26.4 us.)
struct TileCost {
    int variant, bm, bn, per_cu;       // per_cu: workgroups a compute unit holds
    double fixed, step, step_busy, once, ragged;
    double alone, alone_step, alone_busy;   // (two to a compute unit:) fixed cost and step of one that has it to itself
};
// The shapes differ in how they round off.  128 rows or columns less than a square tile's mean more tiles of less arithmetic per
// byte; 192 and 160 rows fill in between (M = 1111: 192 x 128 tiles on 192 compute units where 256 x 128 had 160, N = 4096,
// K = 14336: 45.5 -> 38.0 us, K = 4096: 17.0 -> 12.9; 192 x 256, N = 28672, K = 4096: 72 -> 68; M = 600, N = K = 8192, 160 x 128:
// 28.9 -> 23.4; M = 300, N = 57344, K = 8192, 192 x 256: 102 -> 82).  256 x 128 has eight waves of 64 x 64: two to a SIMD, one's LDS
// reads under the other's products, against four of 128 x 64 M = 1111, N = 4096, K = 14336: 45.5 -> 41.0 us.  128 x 256 with two
// workgroups per compute unit overlaps one's start-up and stores with the other's main loop: where a tile is not much longer
// than those (M = 2166, N = 10968, K = 1024: 26.5 us, the best of the others 30.0; M = 1104, N = 26544, K = 1536: 38.4 against 42.5).
// Where 128 x 128 tiles leave compute units without one, what a step takes is its copies: 128 tiles in two rows, one to a compute unit, 30 ns
// and 10 a KB where W comes from the last-level cache, 16 a KB where it comes from HBM (64 x 64 / 64 x 128 / 128 x 128, 8 / 12 / 16 KB a step:
// 112 / 133 / 197 and 152 / 223 / 285 ns).  Tiles
// of 64 or 96 rows and 64 or 128 columns put more units to work on fewer bytes each (N = K = 2048, M = 201: 6.8 -> 5.0 us; N = 1024, K = 2816:
// 7.8 -> 5.5; N = 6144, K = 4096: 11.1 -> 9.6; N = K = 8192: 21.8 -> 17.9).  Their four rows were fitted to 9996 products with cold weights (M = 65
// ... 4096, N = 512 ... 28672, K = 1024 ... 28672), on the scale of the others, and once more, with those of the eight-stage 128 x 128 tiles, the
// parts and the streaming kernels' prices, to 32735 on three cards (M = 17 ... 900, N = 512 ... 32768, K = 1024 ... 28672), for the choice to lose least
// and for few products to lose by the change.  What was taken lost 1.1 % on the best way on average and more than 5 % on 3006 products; now 0.65 % and
// 1503 (0.7 % on the 8100 left out of the fit).  2923 products go another way, at 0.95 of their time on average, 41 of them more than 5 % slower.
constexpr TileCost kTileCosts[] = {
    {2, 128, 128, 2, 3.539, 0.307, 0.207, 0.890, 1.100, 2.998, 0.227, 0.525},
    {18, 128, 128, 1, 2.990, 0.193, 0.099, 1.057, 1.501},   // one workgroup per compute unit, eight-stage ring
    {17, 128, 128, 1, 2.916, 0.230, 0.068, 1.215, 0.609},
    {5, 256, 128, 1, 3.755, 0.305, 0.153, 0.861, 2.861},
    {6, 192, 128, 1, 2.521, 0.308, 0.102, 1.515, 2.449},
    {7, 160, 128, 1, 2.538, 0.301, 0.058, 1.800, 0.928},
    {8, 192, 256, 1, 5.040, 0.314, 0.326, 0.790, 4.259},
    {13, 256, 192, 1, 6.292, 0.286, 0.350, 0.529, 4.097},
    {10, 256, 256, 1, 6.891, 0.365, 0.430, 0.314, 4.451},
    {11, 256, 256, 1, 6.536, 0.454, 0.293, 1.470, 4.683},   // persistent: the next tile's first stages and the stores overlap
    {15, 128, 256, 2, 5.720, 0.475, 0.516, 0.119, 1.977, 5.139, 0.452, 0.275},
    {16, 128, 256, 2, 5.883, 0.607, 0.367, 1.472, 1.613, 2.756, 0.456, 0.314},   // persistent
    {1, 64, 64, 2, 1.320, 0.134, 0.101, 2.941, 0.000, 0.147, 0.132, 0.162},     // these four with an eight-stage ring
    {4, 64, 128, 1, 0.640, 0.164, 0.045, 3.000, 0.509},
    {9, 96, 128, 1, 1.679, 0.182, 0.064, 2.467, 0.408},
    {12, 96, 64, 1, 2.334, 0.153, 0.006, 1.770, 0.000},
};
// larger tiles in parts, priced from such runs
constexpr TileCost kSplitCosts[] = {
    {2, 128, 128, 2, 2.862, 0.331, 0.261, 0.302, 0.000, 1.141, 0.250, 0.277},
    {5, 256, 128, 1, 8.639, 0.122, 0.338, 0.000, 0.000},
    {10, 256, 256, 1, 7.046, 0.499, 0.323, 0.000, 0.000},
};

double tile_cost(const TileCost& c, int64_t tiles, int64_t kt, bool ragged, int cus)
{
    const int64_t slots = (int64_t)cus * c.per_cu, full = tiles / slots, rest = tiles % slots;
    double t = c.once + (double)full * (c.fixed + (double)kt * (c.step + c.step_busy));
    if (ragged) t += c.ragged * (double)tiles / (double)slots;
    if (rest > 0 && c.per_cu == 2 && rest <= cus) t += c.alone + (double)kt * c.alone_step * (1.0 + c.alone_busy * (double)rest / (double)cus);
    else if (rest > 0) t += c.fixed + (double)kt * (c.step + c.step_busy * (double)rest / (double)slots);
    return t;
}

// (the least of K: two parts of sixteen K-steps)
bool may_split(int64_t M, int64_t K) { return M > 64 && K >= 32 * 128; }

}  // namespace

// The cheapest way of a product: the tiles of the table above (variant: a number of launch_gemm_mxfp4's switch), with more than 64 tokens and
// room for partials also as a split-K run, or the streaming kernels (variant 0), which have a price of their own (gemm_stream_us).
// With few tiles and a long K -- batched decoding against a narrow layer -- a handful of compute units each stream a long K range alone.
// Every tile's K range can then be cut into up to eight parts of at least 16 K-steps (whole scale batches of eight), each part one
// workgroup of as many tiles.  Priced as as many tiles of as many steps, which share their start, and 3.8 us + bytes at 4.3 TB/s (written and
// read) for the partials and their sum's launch; a split has to win 4 %.  Of 2208 products with K from 4096 to 28672, parts of up to 96 rows
// were the best way in 749, 1.26 times as fast as the best unsplit one on average.  Parts of larger tiles are where more than half the units have a small
// tile and none could have a second part of one, K >= 16384 mostly (three parts of 128 x 128, M = 119, N = 8320, K = 24576: 39.6 us, unsplit 64 x 128 52.2; four of
// 256 x 128, M = 230, N = 6248, K = 26752: 41.7, 49.0; three of 256 x 256, M = 220, N = 17152, K = 28416: 90, unsplit 256 x 128 104).
MxPlan plan_mx(int64_t M, int64_t N, int64_t K, size_t room)
{
    MxPlan p{0, 1, 0};
    if (M <= 16) return p;
    // (more than 32 tokens on a very wide layer: 64 x 256 tiles, whose time hardly grows with the token count; N = 57344, K = 14336, M = 48:
    // 87 us, streamed 113; K = 6144, M = 64: 39 and 45)
    if (M > 32 && M <= 64 && N >= 40960 && K > 4096) return MxPlan{3, 1, 0};
    const double stream = gemm_stream_us(M, N, K);
    if (stream == 0.0) return p;
    const int cus = compute_units();
    const int64_t kt = K >> 7;
    auto tiles = [&](const TileCost& c) { return ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn); };
    // Up to 64 tokens both prices are rough where they are close (and the tiles were not timed beyond N = 32768): tiles have to win a
    // fifth.  Of 7463 products of 20 to 64 tokens 0.96 of the streaming kernels' time on average; K = 1024, N > 8192 0.8.
    if (M <= 64 && N > 32768) return p;
    double best = M <= 64 ? stream / 1.2 : stream;
    for (const TileCost& c : kTileCosts) {
        if (M <= 64 && c.bm != 64) continue;
        const int64_t t = tiles(c);
        if ((c.variant == 17 || c.variant == 18) && t > cus) continue;
        // (persistent workgroups: only where there is a next tile, and not for a ragged few rounds, where one workgroup per tile, which
        // the hardware hands to whichever unit is free, measured up to 5 % faster: N = 28672, K = 4096, M = 994: 63.4 against 66.8 us)
        if (c.variant == 11 && (t <= cus || (t % cus != 0 && t < 3 * (int64_t)cus))) continue;
        if (c.variant == 16 && t <= 2 * (int64_t)cus) continue;
        const double us = tile_cost(c, t, kt, N % 32 != 0, cus);
        if (us < best) {
            best = us;
            p.variant = c.variant;
        }
    }
    if (!may_split(M, K)) return p;
    best *= 0.96;
    auto parts = [&](const TileCost& c, double share, double launch, double us_per_mb) {
        const int64_t t = tiles(c), s_max = std::min<int64_t>(std::min<int64_t>((int64_t)cus * c.per_cu / t, kt / 16), 8);
        for (int64_t s = 2; s <= s_max; ++s) {
            const int64_t st = ((kt + s - 1) / s + 7) / 8 * 8;
            const int64_t n = (kt + st - 1) / st;  // parts of st steps that cover K (the last may be shorter)
            const double bytes = (double)n * (double)M * (double)N * 4.0;
            if (n < 2 || bytes > (double)room) continue;
            const double us = share * tile_cost(c, t * n, st, false, cus) + launch + us_per_mb * bytes * 1e-6;
            if (us < best) {
                best = us;
                p = MxPlan{c.variant, (int)n, (int)st};
            }
        }
    };
    for (const TileCost& c : kTileCosts)
        if (c.bm <= 96 && c.bn <= 128) parts(c, 0.811, 3.83, 0.467);
    for (const TileCost& c : kSplitCosts) parts(c, 1.0, 8.55, 0.205);
    return p;
}

// bytes of fp32 partials a split-K run of this product needs (0: the product is not split)
size_t gemm_mx_split_k_bytes(int64_t M, int64_t N, int64_t K)
{
    if (!may_split(M, K)) return 0;
    const MxPlan p = plan_mx(M, N, K, SIZE_MAX);
    return p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N * 4 : 0;
}

// plan: of plan_mx, with a tile configuration, or any such (variant 1 ..) in one part; partial: room for a split run's partials
hipError_t launch_gemm_mxfp4(const void* a_codes, const void* a_scales, const void* w_codes, const void* w_scales,
                             int64_t M, int64_t N, int64_t K, void* out, bool out_f32, const MxPlan& plan, float alpha, void* partial,
                             hipStream_t st)
{
    GemmArgs g{};
    g.alpha = alpha;
    g.a_codes = static_cast<const uint8_t*>(a_codes);
    g.a_scales = static_cast<const uint8_t*>(a_scales);
    g.w_codes = static_cast<const uint8_t*>(w_codes);
    g.w_scales = static_cast<const uint8_t*>(w_scales);
    g.out = out;
    g.M = M;
    g.N = N;
    g.K = K;
    const int splits = plan.splits, split_steps = plan.steps;
    float* const pp = static_cast<float*>(partial);
    switch (plan.variant) {
        case 1: return launch_variant<64, 64, 32, 32, 8, 1>(g, out_f32, st, splits, split_steps, pp);
        case 2: return launch_variant<128, 128, 64, 64, 4>(g, out_f32, st, splits, split_steps, pp);
        case 3: return launch_variant<64, 256, 64, 64, 4>(g, out_f32, st);
        case 4: return launch_variant<64, 128, 32, 64, 8>(g, out_f32, st, splits, split_steps, pp);
        case 5: return launch_variant<256, 128, 64, 64, 4>(g, out_f32, st, splits, split_steps, pp);
        case 6: return launch_variant<192, 128, 48, 64, 4>(g, out_f32, st);
        case 7: return launch_variant<160, 128, 80, 64, 4>(g, out_f32, st);
        case 8: return launch_variant<192, 256, 96, 64, 4>(g, out_f32, st);
        case 9: return launch_variant<96, 128, 48, 64, 8>(g, out_f32, st, splits, split_steps, pp);
        case 10: return launch_variant<256, 256, 64, 128, 4, 3>(g, out_f32, st, splits, split_steps, pp);
        case 11: return launch_variant<256, 256, 64, 128, 4, 3, true>(g, out_f32, st);
        case 12: return launch_variant<96, 64, 48, 32, 8, 1>(g, out_f32, st, splits, split_steps, pp);
        case 13: return launch_variant<256, 192, 64, 96, 4, 2>(g, out_f32, st);
        case 14: return launch_variant<256, 192, 64, 96, 4, 2, true>(g, out_f32, st);
        case 15: return launch_variant<128, 256, 64, 128, 3, 3>(g, out_f32, st);
        case 16: return launch_variant<128, 256, 64, 128, 3, 3, true>(g, out_f32, st);
        case 17: return launch_variant<128, 128, 64, 64, 8>(g, out_f32, st);
        case 18: return launch_variant<128, 128, 32, 64, 8>(g, out_f32, st);
        default: return hipErrorInvalidValue;
    }
}

// compute units of the current device (asked of the runtime once per device; which one is current, 54 ns of the smallest calls' 4.5 us, only where a
// process sees more than one)
int compute_units()
{
    static const bool one_device = [] {
        int n = 0;
        return hipGetDeviceCount(&n) == hipSuccess && n == 1;
    }();
    static std::atomic<int> cached[64] = {};
    int dev = 0;
    if (!one_device && (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

}  // namespace fp4mr
