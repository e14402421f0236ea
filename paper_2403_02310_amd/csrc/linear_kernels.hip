// gfx950 kernels of libsarathi: a linear layer over the token rows of a batch (paper sections
// 2.1 and 3.1),  y[t][n] = sum_k x[t][k] * w[n][k],  bf16 in, fp32 accumulation, bf16 out.
//
// Both operands are contiguous along the contraction index k, which is the per-lane operand
// shape of v_mfma_f32_32x32x16_bf16 and v_mfma_f32_16x16x32_bf16 (a lane holds one row and 8 consecutive k).  The weight tile
// is the A operand (rows = output features) and the token tile the B operand (columns = tokens),
// so an accumulator lane holds ONE token and runs of 4 consecutive features.  Small batches write
// these as 8-byte pieces that a wavefront's accumulator tiles complete to 128 contiguous bytes;
// larger ones turn them into whole rows in LDS first.
//
// Four kernels.  linear_thin_kernel (up to 16 tokens, 32 on shorter k ranges) and linear_mid_kernel (17 to 96 tokens where k ranges are
// short next to the features): one workgroup per compute unit, nothing cut across workgroups.  linear_phased_kernel (more than 64 tokens otherwise): four wavefronts, one per SIMD, each with up to 128 x 128
// results in accumulation registers; linear_kernel (up to 64 tokens otherwise): eight wavefronts, narrow token tiles, bound by
// fetching the weights.  All bring k stages of 64 (an LDS row is one full 128-byte line of its matrix row; rows of half a
// line fetch at less than half the rate: 43 against 95 GB/s per compute unit out of L2) from global memory straight into LDS
// (global_load_lds_dwordx4: no staging registers).  The eight 16-byte pieces of LDS row r are XOR-swizzled with
// (r >> 1) & 7 so that the 16 lanes of a b128 operand read, which walk 16 rows at one logical piece, hit distinct banks.
//
// The non-temporal hint goes on the weights where ONE token tile covers the batch: every weight byte is then fetched
// once and the chip streams 7.0 TB/s with it against 6.2 without.  Where several token tiles share a weight tile it
// must not: lines fetched with it do not stay in L2 for the other compute units of the XCD (58 GB/s per compute unit
// against 95 for a tile shared by eight of them).
//
// Few tokens (a decode-heavy batch): one token tile covers the batch, the weights are read
// once, and the layer is bound by fetching them (section 3.1); when the grid would leave
// compute units idle the k range is cut into pieces (split-K) whose fp32 partial tiles a
// second small kernel adds up in piece order (bitwise reproducible).
//
// Workgroup -> tile mapping (lin_work_item): blockIdx % 8 selects the XCD; every XCD gets a contiguous run of work items
// (equal runs, give or take one) in an order that walks groups of four feature tiles, so that the 32 workgroups an XCD
// runs at a time share weight and token tiles in its L2.  (Dealing whole feature tiles to XCDs, n = xcd, xcd + 8, ...,
// left ten feature tiles on eight XCDs with two rounds of work on two of them: 2048 x 2560 x 8192 took 161 us, now 81.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace sarathi {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 lbf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 lbf16x4;
typedef __attribute__((ext_vector_type(4))) float lf32x4;
typedef __attribute__((ext_vector_type(16))) float lf32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t lu32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t lu32x2;
typedef lu32x4 __attribute__((aligned(8))) lu32x4_at8;  // output rows: y is promised 8-byte alignment only

constexpr int kLinStageK = 64;   // k per stage: one 128-byte line of every row
constexpr int kLinXcds = 8;
constexpr int kLinThreads = 512;
constexpr int kLinSmallTokens = 64;  // up to this many: linear_kernel, beyond: linear_phased_kernel

typedef void __attribute__((address_space(3))) *lin_lds_ptr;

// One direct global -> LDS load of 16 bytes per lane: lane l fetches base + byte_off(l) and the
// wavefront's kilobyte lands at LDS byte address lds_addr + 16 l.  Inline assembly so that the
// compiler's wait-count pass does not treat later LDS operand reads as possibly overtaken by it;
// these loads are waited for by hand, they are the only vector-memory loads of the loop.
__device__ __forceinline__ void lin_dma_load_16(const uint16_t *base, int byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(byte_off), "s"(base)
                 : "memory");
}
// The same with the non-temporal hint (weights that one workgroup alone fetches).
__device__ __forceinline__ void lin_dma_load_16_stream(const uint16_t *base, int byte_off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :
                 : "s"(lds_addr), "v"(byte_off), "s"(base)
                 : "memory");
}
// s_waitcnt with the vector-memory counter at n and the LDS counter at zero (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4 left at its maximum, lgkmcnt 11:8)
#define LIN_WAIT_LDS() __builtin_amdgcn_s_waitcnt(0xC07F)  // the LDS counter alone
#define LIN_WAIT_VMCNT_AND_LDS(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0070)

// Orders a wavefront's LDS writes before the reads of other lanes that follow (and reads before later writes).  The LDS queue
// of a wavefront is in order, so no instruction comes of it; it keeps the compiler from moving one across the other.
__device__ __forceinline__ void lin_wavefront_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// c += a b^T (16 rows x 16 columns x 32 k) in place.  Inline assembly, because it ties the result to the accumulation registers of c:
// through the builtin the compiler gives each of up to 256 results new registers and copies them back, 234 to 658 moves per
// two stages, and spills in the key loop of the largest shape (2048 x 8192 x 7168: 522 us).  The compiler does not see that this
// is a matrix instruction, so the caller keeps the distances that the hardware does not: other instructions read c from 8 wait
// states on, and the instruction reads a, b and c from 2 wait states after a vector instruction wrote them.  Whether the registers that the
// compiler chose leave them so is looked up in its assembly (tests/test_device_code.py): a copy or a spill in between gives wrong sums.
__device__ __forceinline__ void lin_mfma_in_place(lf32x4 &c, const lbf16x8 &a, const lbf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

struct LinearParams {
    const uint16_t *x;   // [T, K]
    const uint16_t *w;   // [N, K]
    uint16_t *y;         // [T, N], rows y_stride apart (linear_phased_kernel; the others: N)
    float *part;         // [splits, T, N] when splits > 1
    int32_t T, N, K;
    int32_t y_stride;
    int32_t n_tiles, t_tiles, splits;
    int32_t k_per_split;  // multiple of 64
};

struct LinearItem {
    int32_t n_tile, t_tile, split;  // n_tile < 0: nothing to do
};
// Work item of this workgroup: the XCD's run of the items, which are ordered (group of four feature tiles, k piece,
// token tile, feature tile of the group).
constexpr int kLinGroup = 4;
__device__ __forceinline__ LinearItem lin_work_item(const LinearParams &p) {
    const int items = p.n_tiles * p.t_tiles * p.splits;
    const int xcd = blockIdx.x % kLinXcds, j = blockIdx.x / kLinXcds;
    const int run = items / kLinXcds, extra = items % kLinXcds;
    if (j >= run + (xcd < extra ? 1 : 0)) return LinearItem{-1, 0, 0};
    const int it = xcd * run + min(xcd, extra) + j;
    const int per_group = kLinGroup * p.splits * p.t_tiles;
    const int group = __builtin_amdgcn_readfirstlane(it / per_group);
    int rest = it - group * per_group;
    const int width = min(kLinGroup, p.n_tiles - group * kLinGroup);
    // wave-uniform by construction; tell the compiler (its integer division goes through the vector unit)
    const int split = __builtin_amdgcn_readfirstlane(rest / (width * p.t_tiles));
    rest -= split * width * p.t_tiles;
    const int t_tile = __builtin_amdgcn_readfirstlane(rest / width);
    return LinearItem{group * kLinGroup + rest - t_tile * width, t_tile, split};
}

// Where a workgroup starts in its k range, in stages; it wraps round at the end.  Workgroups of one token tile only meet in
// memory: if all of them started at the front, every row of the weights would be read at the same k, and rows lie a power
// of two (or a small multiple of one) apart, so that all reads of a moment would fall on a few memory channels.
// 8 x 28672 x 4096: 49 us from the front, 38 staggered; 77 x 28672 x 4096: 53 and 44; 8 x 14336 x 8192: 51 and 42.  With
// several token tiles the workgroups of an XCD have to stay at the same k to share tiles in L2 (no gain measured there).
__device__ __forceinline__ int lin_first_stage(const LinearParams &p, int n_tile, int n_stages) {
    return p.t_tiles == 1 ? __builtin_amdgcn_readfirstlane((n_tile * 3) % n_stages) : 0;
}

// BM tokens per tile; WT wavefronts side by side along the tokens (the other 8 / WT along the features);
// RING stages of LDS; BN features per tile.
template <int BM, int WT, int RING, int BN>
__global__ __launch_bounds__(kLinThreads, 1) void linear_kernel(LinearParams p) {
    constexpr int KS = kLinStageK;
    constexpr int PIECES = KS / 8;              // 16-byte pieces of an LDS row
    constexpr int DMA_ROWS = 64 / PIECES;       // rows one 1 KiB load covers
    constexpr int W_ELEMS = BN * KS;
    constexpr int X_ELEMS = BM * KS;
    constexpr int STAGE = W_ELEMS + X_ELEMS;
    constexpr int W_ROWS = BN / 8;              // weight rows a wavefront moves per stage
    constexpr int W_LOADS = W_ROWS / DMA_ROWS;  // 1 KiB loads of weight rows per wavefront and stage
    constexpr int X_LOADS = BM / (8 * DMA_ROWS);  // the same for token rows
    static_assert(BM % (8 * DMA_ROWS) == 0, "every wavefront moves the same number of token rows");
    constexpr int LOADS = W_LOADS + X_LOADS;    // all loads of a wavefront per stage
    constexpr int NI = BN * WT / 256;           // 32-feature MFMA tiles per wavefront: BN features / (8 / WT wavefronts) / 32
    constexpr int NJ = BM / WT / 32;            // 32-token MFMA tiles per wavefront
    constexpr int STEPS = KS / 16;
    static_assert(NI * (8 / WT) * 32 == BN && NJ * WT * 32 == BM, "the wavefronts' tiles cover the workgroup's");
    __shared__ __attribute__((aligned(16))) uint16_t smem[RING * STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LinearItem wi = lin_work_item(p);
    if (wi.n_tile < 0) return;
    const int n_tile = wi.n_tile, t_tile = wi.t_tile, split = wi.split;
    const int n0 = n_tile * BN;
    const int t0 = t_tile * BM;
    const int k_begin = split * p.k_per_split;
    const int k_end = min(p.K, k_begin + p.k_per_split);
    const int n_stages = (k_end - k_begin) / KS;
    const int first_stage = lin_first_stage(p, n_tile, n_stages);
    auto row_key = [](int row) { return (row >> 1) & 7; };

    // ---- global -> LDS: wavefront w moves rows (BN/8)w .. of the weight tile and rows (BM/8)w .. of the token tile, 8 rows
    // a load.  Lane l of a load fills physical piece l % 8 of row l / 8 and
    // therefore fetches the logical piece that lives there.  Rows past the matrix re-read its last row.
    int w_off[W_LOADS], x_off[X_LOADS];
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) {
        const int row = wave * W_ROWS + i * DMA_ROWS + lane / PIECES;
        const int piece = (lane % PIECES) ^ row_key(row);
        w_off[i] = ((min(n0 + row, p.N - 1) - n0) * p.K + piece * 8) * 2;
    }
#pragma unroll
    for (int i = 0; i < X_LOADS; ++i) {
        const int row = (wave * X_LOADS + i) * DMA_ROWS + lane / PIECES;
        const int piece = (lane % PIECES) ^ row_key(row);
        x_off[i] = ((min(t0 + row, p.T - 1) - t0) * p.K + piece * 8) * 2;
    }
    const uint16_t *w_base = p.w + (int64_t)n0 * p.K + k_begin;
    const uint16_t *x_base = p.x + (int64_t)t0 * p.K + k_begin;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lin_lds_ptr)(smem);
    auto issue_stage = [&](int stage, int slot) {
        // stages past the range re-read the last one into a free slot: every step issues the same
        // number of loads, so one wait count serves the whole loop
        const int at = min(stage, n_stages - 1) + first_stage;
        const int s = at < n_stages ? at : at - n_stages;
        const uint32_t dst = smem_addr + (uint32_t)(slot * STAGE * 2);
        const uint16_t *wb = w_base + s * KS;
        const uint16_t *xb = x_base + s * KS;
#pragma unroll
        for (int i = 0; i < W_LOADS; ++i) lin_dma_load_16_stream(wb, w_off[i], dst + (uint32_t)((wave * W_ROWS + i * DMA_ROWS) * KS * 2));
#pragma unroll
        for (int i = 0; i < X_LOADS; ++i)
            lin_dma_load_16(xb, x_off[i], dst + (uint32_t)(W_ELEMS * 2 + (wave * X_LOADS + i) * DMA_ROWS * KS * 2));
    };

    // ---- operands: wavefront (wn, wt) owns features 32 NI wn.. and tokens 32 NJ wt.. of the tile
    const int wn = wave % (8 / WT), wt = wave / (8 / WT);
    const int r = lane & 31, g = lane >> 5;
    int a_row[NI], a_key[NI], b_row[NJ], b_key[NJ];  // element offset of the row inside a stage, and its swizzle key
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int ra = wn * (32 * NI) + i * 32 + r;
        a_row[i] = ra * KS;
        a_key[i] = row_key(ra);
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int rb = wt * (32 * NJ) + jj * 32 + r;
        b_row[jj] = W_ELEMS + rb * KS;
        b_key[jj] = row_key(rb);
    }

    lf32x16 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][jj][e] = 0.f;

    auto read_step = [&](const uint16_t *sp, int s, lbf16x8 (&a)[NI], lbf16x8 (&b)[NJ]) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            a[i] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + a_row[i] + (((2 * s + g) ^ a_key[i]) * 8)));
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
            b[jj] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + b_row[jj] + (((2 * s + g) ^ b_key[jj]) * 8)));
    };
    auto mfma_step = [&](const lbf16x8 (&a)[NI], const lbf16x8 (&b)[NJ]) {
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int i = 0; i < NI; ++i)
                acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[jj], acc[i][jj], 0, 0, 0);
    };
    lbf16x8 fa[2][NI], fb[2][NJ];  // two operand sets used in turn
#pragma unroll
    for (int i = 0; i < NI; ++i) fa[1][i] = lbf16x8{};  // the "last step of stage -1": zeros
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) fb[1][jj] = lbf16x8{};

#pragma unroll
    for (int st = 0; st < RING - 1; ++st) issue_stage(st, st);
    int slot = 0, fill_slot = RING - 1;
    for (int st = 0; st < n_stages; ++st) {
        // Stage st has landed when at most the loads of the RING-2 later stages are in flight.  The barrier
        // also says that every wavefront has its last operands of stage st-1 in registers (LDS counter at
        // zero), so the slot of stage st-1 may be overwritten by stage st+RING-1.
        LIN_WAIT_VMCNT_AND_LDS((RING - 2) * LOADS);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue_stage(st + RING - 1, fill_slot);
        const uint16_t *sp = smem + slot * STAGE;
        // STEPS is even: step s uses operand set s & 1; set 1 arrives holding the previous stage's last step
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            read_step(sp, s, fa[s & 1], fb[s & 1]);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step(fa[(s & 1) ^ 1], fb[(s & 1) ^ 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = slot + 1 == RING ? 0 : slot + 1;
        fill_slot = fill_slot + 1 == RING ? 0 : fill_slot + 1;
    }
    mfma_step(fa[1], fb[1]);
    LIN_WAIT_VMCNT_AND_LDS(0);  // the padding loads past the range must land before the workgroup's LDS is given back

    // ---- output: accumulator element e of lane (r, g) of tile (i, jj) is feature 32i + 8(e/4) + 4g + e%4, token 32jj + r
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int t = t0 + wt * (32 * NJ) + jj * 32 + r;
        if (t >= p.T) continue;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int f0 = n0 + wn * (32 * NI) + i * 32 + 4 * g;
            if (f0 >= p.N) continue;  // N is a multiple of 128, the tile may reach past it
            if (p.splits == 1) {
                uint16_t *yp = p.y + (int64_t)t * p.N + f0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const lf32x4 v = {acc[i][jj][4 * q], acc[i][jj][4 * q + 1], acc[i][jj][4 * q + 2], acc[i][jj][4 * q + 3]};
                    *reinterpret_cast<lu32x2 *>(yp + 8 * q) = __builtin_bit_cast(lu32x2, __builtin_convertvector(v, lbf16x4));
                }
            } else {
                float *pp = p.part + ((int64_t)split * p.T + t) * p.N + f0;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<lf32x4 *>(pp + 8 * q) =
                        lf32x4{acc[i][jj][4 * q], acc[i][jj][4 * q + 1], acc[i][jj][4 * q + 2], acc[i][jj][4 * q + 3]};
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// More than 64 tokens: four wavefronts in a 2 x 2 grid, one per SIMD.  A wavefront owns (A0 + A1) x (B0 + B1) blocks
// of 32 features x 32 tokens (4 x 4 in the largest shape: all 256 accumulation registers), so that a 256 x 256 tile reads
// 8 operands of 1 KiB from LDS per 16 x 32 x 32 x 16 multiply-adds; eight wavefronts of 64 x 128 read 12 (195-205 us on 2048 x 8192 x 7168).
// A block is four v_mfma_f32_16x16x32_bf16 rather than two v_mfma_f32_32x32x16_bf16 per 32 k: both issue at the matrix pipes' rate (16.3
// and 32.3 clocks), but the smaller draws less power per multiply-add, and on N(0,1) values power sets the clock: 1.93 to 2.10
// against 1.65 to 1.78 PFLOP/s where nothing else runs, 1.88 against 1.64 GHz here (2048 x 8192 x 7168 180 -> 160 us, 2048 x 14336 x
// 8192 372 -> 346; on zeros both instructions 2.46 PFLOP/s at 2.4 GHz).
//
// A stage is worked off in phases: half A0 of the wavefront's weight rows x half B0 of its token rows, A0 x B1, A1 x B1,
// A1 x B0, each over the stage's 64 k.  While a phase's MFMAs issue, the operands of the half that a later phase needs are
// read into registers (8 reads per 32 MFMAs), and the barrier at the head of the next phase then frees that half's LDS for
// the stage RING stages on.  So LDS is refilled half by half and a fetch has 1.75 stages (RING = 2) to land; waiting for
// whole stages gives it less than one of the two that 128 KiB hold, and the loop then waits for memory: 2048 x 8192 x 7168
// on all-zero data 158 us by whole stages, 121 us by halves (with the 32 x 32 instruction, as the figures below).  The matrix pipes
// are busy for 75 % of the cycles (78 % with that).
// One wavefront per SIMD leaves nobody to cover a wait, so a phase is laid out by hand: slot m issues its share of reads and
// fetches, then MFMA m, and a scheduling barrier keeps the compiler from moving them (204 other instructions per 256 MFMAs).
// Accumulators go out through LDS as whole rows (16-byte stores, 128 to 256 contiguous bytes per token and wavefront): 5 us
// less per tile than 8-byte stores from the accumulator layout.  The way out still takes 8.2 us for 256 x 256: each piece is
// a predicated read, a wait and a store in a row.  No shape spills.
// ---------------------------------------------------------------------------------------
template <int A0, int A1, int B0, int B1, int RING, bool STREAM>
__global__ __launch_bounds__(256, 1) void linear_phased_kernel(LinearParams p) {
    constexpr int KS = kLinStageK;
    constexpr int NI = A0 + A1, NJ = B0 + B1;    // MFMA tiles of a wavefront along features, tokens
    constexpr int BN = 64 * NI, BM = 64 * NJ;    // features, tokens of the workgroup's tile
    constexpr int BLOCK = 32 * KS;               // elements of 32 rows of a stage
    constexpr int STAGE = 2 * (NI + NJ) * BLOCK;
    // halves in the order in which they are read; each holds its rows for both wavefronts along its side
    constexpr int HA0 = 0, HB0 = 1, HB1 = 2, HA1 = 3;
    constexpr int kBlocks[4] = {A0, B0, B1, A1};
    constexpr int kOff[4] = {0, 2 * NI * BLOCK, 2 * (NI + B0) * BLOCK, 2 * A0 * BLOCK};
    constexpr int LOADS = 2 * (NI + NJ);         // 1 KiB loads of a wavefront per stage: two per 32-row block
    static_assert(A0 > 0 && A1 > 0 && B0 > 0 && RING >= 2, "two weight halves, one or two token halves");
    static_assert(RING * LOADS < 64, "the vector-memory counter holds 63 loads");
    static_assert(RING * STAGE * 2 <= 160 * 1024 && RING * STAGE * 2 >= 4 * 16384, "LDS of a compute unit; the output's transposition needs 16 KiB per wavefront");
    __shared__ __attribute__((aligned(16))) uint16_t smem[RING * STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LinearItem wi = lin_work_item(p);
    if (wi.n_tile < 0) return;
    const int n0 = wi.n_tile * BN, t0 = wi.t_tile * BM;
    const int k_begin = wi.split * p.k_per_split;
    const int n_stages = (min(p.K, k_begin + p.k_per_split) - k_begin) / KS;
    const int first_stage = STREAM ? lin_first_stage(p, wi.n_tile, n_stages) : 0;
    auto row_key = [](int row) { return (row >> 1) & 7; };

    // ---- global -> LDS.  LDS row l of a half of nb blocks is row l % 32 of block (l / 32) % nb of side-wavefront
    // l / (32 nb); wavefront w moves rows 16 nb w .. as 2 nb loads of 8 rows.  Rows past the matrix re-read its last row.
    const uint16_t *w_base = p.w + (int64_t)n0 * p.K + k_begin;
    const uint16_t *x_base = p.x + (int64_t)t0 * p.K + k_begin;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lin_lds_ptr)(smem);
    int off[LOADS];  // this lane's byte offsets: halves A0, B0, B1, A1 one after the other
    auto half_loads = [&](int h) { return 2 * kBlocks[h]; };
    auto first_load = [&](int h) { return 2 * ((h > 0 ? A0 : 0) + (h > 1 ? B0 : 0) + (h > 2 ? B1 : 0)); };
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const bool weights = h == HA0 || h == HA1;
        const int nb = kBlocks[h];
        const int before = h == HA1 ? A0 : h == HB1 ? B0 : 0;  // blocks of the side's first half
#pragma unroll
        for (int i = 0; i < 2 * nb; ++i) {
            const int l = wave * 16 * nb + i * 8 + lane / 8;
            const int row = l / (32 * nb) * 32 * (weights ? NI : NJ) + (before + l / 32 % nb) * 32 + l % 32;
            const int base = weights ? n0 : t0, limit = weights ? p.N : p.T;
            off[first_load(h) + i] = ((min(base + row, limit - 1) - base) * p.K + ((lane % 8) ^ row_key(l % 32)) * 8) * 2;
        }
    }
    // load i of half h of stage `stage` into ring slot `slot`; stages past the range re-read the last one, so that every
    // phase issues the same loads and one wait count serves the whole loop
    auto issue = [&](auto ht, int i, int stage, int slot) {
        constexpr int h = decltype(ht)::value;
        const int at = min(stage, n_stages - 1) + first_stage;
        const int k = (at < n_stages ? at : at - n_stages) * KS;
        const uint32_t dst = smem_addr + (uint32_t)(slot * STAGE + kOff[h] + wave * kBlocks[h] * 16 * KS) * 2 + (uint32_t)i * 1024;
        if (h == HB0 || h == HB1) lin_dma_load_16(x_base + k, off[first_load(h) + i], dst);
        else if (STREAM) lin_dma_load_16_stream(w_base + k, off[first_load(h) + i], dst);
        else lin_dma_load_16(w_base + k, off[first_load(h) + i], dst);
    };

    // ---- operands: wavefront (wn, wt) owns features 32 NI wn .. and tokens 32 NJ wt .. of the tile
    const int wn = wave & 1, wt = wave >> 1;
    const int n = lane & 15, g = lane >> 4;
    int piece[4];  // element offset of operand s (k 32 (s / 2) .., rows 16 (s % 2) ..) inside a 32-row block for this lane
#pragma unroll
    for (int s = 0; s < 4; ++s) piece[s] = (s % 2 * 16 + n) * KS + ((s / 2 * 4 + g) ^ row_key(n)) * 8;
    constexpr int BX = B0 > B1 ? B0 : B1;
    lbf16x8 fa[2][A0 > A1 ? A0 : A1][4];  // weight operands of halves A0, A1
    lbf16x8 fb[2][BX][4];                 // token operands: B0 and B1 swap sets from stage to stage
    // read q (operand q / nb, block q % nb) of half h from ring slot `slot`; tokens go to set `set`
    auto read = [&](auto ht, auto set, int q, int slot) {
        constexpr int h = decltype(ht)::value;
        constexpr int nb = kBlocks[h] > 0 ? kBlocks[h] : 1;
        const int s = q / nb, b = q % nb;
        const int side = (h == HA0 || h == HA1) ? wn : wt;
        const lbf16x8 v = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(smem + slot * STAGE + kOff[h] + (side * nb + b) * BLOCK + piece[s]));
        if (h == HA0 || h == HA1) fa[h == HA1 ? 1 : 0][b][s] = v;
        else fb[decltype(set)::value][b][s] = v;
    };
    lf32x4 acc[NI][NJ][4];  // of a 32 x 32 block: features 16 (q / 2) .., tokens 16 (q % 2) ..
    auto mfma = [&](int a, int na, int nb, int b_first, const lbf16x8 (&b_ops)[BX][4], int m) {
        const int kh = m / (na * nb * 4), e = m / 4 % (na * nb);
        const int j = e / na, i = (j & 1) ? na - 1 - e % na : e % na;  // consecutive MFMAs share an operand
        const int fi = m % 4 / 2, tj = fi ^ (m & 1);
        lf32x4 &c = acc[(a ? A0 : 0) + i][b_first + j][fi * 2 + tj];
        lin_mfma_in_place(c, fa[a][i][kh * 2 + fi], b_ops[j][kh * 2 + tj]);
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using TA0 = std::integral_constant<int, HA0>;
    using TB0 = std::integral_constant<int, HB0>;
    using TB1 = std::integral_constant<int, HB1>;
    using TA1 = std::integral_constant<int, HA1>;

    // The head of a phase: at most `keep` loads in flight, so the half about to be read has landed; this wavefront's reads
    // are in registers; and behind the barrier both hold for every wavefront.
#define LIN_PHASE_HEAD(keep)            \
    LIN_WAIT_VMCNT_AND_LDS(keep);       \
    __builtin_amdgcn_s_barrier();       \
    asm volatile("" ::: "memory")

    // Prologue: RING stages on their way, A0 and B0 of the first one into registers.
#pragma unroll
    for (int st = 0; st < RING; ++st) {
#pragma unroll
        for (int i = 0; i < half_loads(HA0); ++i) issue(TA0{}, i, st, st);
#pragma unroll
        for (int i = 0; i < half_loads(HB0); ++i) issue(TB0{}, i, st, st);
#pragma unroll
        for (int i = 0; i < half_loads(HB1); ++i) issue(TB1{}, i, st, st);
#pragma unroll
        for (int i = 0; i < half_loads(HA1); ++i) issue(TA1{}, i, st, st);
    }
    // Zeros in place while the loads are on their way, before the first barrier and far from the first MFMA (in front of the loads
    // they kept them back for a clock quad each).
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[i][j][q] = lf32x4{0.f, 0.f, 0.f, 0.f};
                asm volatile("" : "+a"(acc[i][j][q]));
            }
    LIN_PHASE_HEAD(RING * LOADS - 2 * A0);
#pragma unroll
    for (int q = 0; q < 4 * A0; ++q) read(TA0{}, S0{}, q, 0);
    LIN_PHASE_HEAD(RING * LOADS - 2 * A0 - 2 * B0);
    if constexpr (B1 > 0) {
#pragma unroll
        for (int i = 0; i < half_loads(HA0); ++i) issue(TA0{}, i, RING, 0);
    }
#pragma unroll
    for (int q = 0; q < 4 * B0; ++q) read(TB0{}, S0{}, q, 0);

    // One phase: weight half a x token half b (operand set bset).  Reads half rh from slot rslot (tokens into set rset) over
    // the first three quarters of its MFMAs, and refills half ih, whose reads the barrier closes, with stage istage.
    // Loads younger than half rh when the phase starts: RING stages less rh and less ih, which is issued next.
    auto phase = [&](auto at, auto bt, auto bset, auto rht, auto rset, int rslot, auto iht, int istage, int islot) {
        constexpr int a = decltype(at)::value, b = decltype(bt)::value, rh = decltype(rht)::value, ih = decltype(iht)::value;
        constexpr int na = a ? A1 : A0, nb = b ? B1 : B0, NM = na * nb * 8;
        constexpr int reads = 4 * kBlocks[rh], loads = 2 * kBlocks[ih];
        constexpr int span = NM * 3 / 4;
        LIN_PHASE_HEAD(RING * LOADS - 2 * kBlocks[rh] - 2 * kBlocks[ih]);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int q0 = reads * min(m, span) / span, q1 = reads * min(m + 1, span) / span;
#pragma unroll
            for (int q = 0; q < reads; ++q)
                if (q >= q0 && q < q1) read(rht, rset, q, rslot);
#pragma unroll
            for (int l = 0; l < loads; ++l)
                if (l >= loads * m / NM && l < loads * (m + 1) / NM) issue(iht, l, istage, islot);
            mfma(a, na, nb, b ? B0 : 0, fb[decltype(bset)::value], m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // The same without a second token half: A1 is read under A0 x B0, the next stage's B0 and A0 under A1 x B0, and a phase
    // refills what the other one read.  Loads younger than what it reads: RING - 1 stages.
    auto phase_one_half = [&](auto at, auto bset, auto rset, int rslot, int istage, int islot) {
        constexpr int a = decltype(at)::value;
        constexpr int na = a ? A1 : A0, NM = na * B0 * 8;
        constexpr int reads = a ? 4 * (B0 + A0) : 4 * A1, loads = a ? 2 * A1 : 2 * (A0 + B0);
        LIN_PHASE_HEAD((RING - 1) * LOADS);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
#pragma unroll
            for (int q = 0; q < reads; ++q)
                if (q >= reads * m / NM && q < reads * (m + 1) / NM) {
                    if (!a) read(TA1{}, S0{}, q, rslot);
                    else if (q < 4 * B0) read(TB0{}, rset, q, rslot);
                    else read(TA0{}, S0{}, q - 4 * B0, rslot);
                }
#pragma unroll
            for (int l = 0; l < loads; ++l)
                if (l >= loads * m / NM && l < loads * (m + 1) / NM) {
                    if (a) issue(TA1{}, l, istage, islot);
                    else if (l < 2 * A0) issue(TA0{}, l, istage, islot);
                    else issue(TB0{}, l - 2 * A0, istage, islot);
                }
            mfma(a, na, B0, 0, fb[decltype(bset)::value], m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int slot = 0;
    auto stage = [&](int st, auto par) {
        constexpr int P = decltype(par)::value;           // B0 of this stage is in set P
        using Own = std::integral_constant<int, P>;
        using Other = std::integral_constant<int, P ^ 1>;
        if (RING == 2) slot = P;                          // known when the code is generated
        const int next = RING == 2 ? P ^ 1 : slot + 1 == RING ? 0 : slot + 1;
        if constexpr (B1 > 0) {
            phase(S0{}, S0{}, Own{}, TB1{}, Other{}, slot, TB0{}, st + RING, slot);
            phase(S0{}, S1{}, Other{}, TA1{}, S0{}, slot, TB1{}, st + RING, slot);
            phase(S1{}, S1{}, Other{}, TA0{}, S0{}, next, TA1{}, st + RING, slot);
            phase(S1{}, S0{}, Own{}, TB0{}, Other{}, next, TA0{}, st + 1 + RING, next);
        } else {
            phase_one_half(S0{}, Own{}, S0{}, slot, st + RING, slot);
            phase_one_half(S1{}, Own{}, Other{}, next, st + RING, slot);
        }
        slot = next;
    };
    int st = 0;
    for (; st + 1 < n_stages; st += 2) {
        stage(st, S0{});
        stage(st + 1, S1{});
    }
    if (st < n_stages) stage(st, S0{});

    // ---- output.  The padding loads have landed and every wavefront is done with the operands: LDS (16 KiB per wavefront)
    // turns 32 tokens at a time into rows; 16-byte piece c of row r sits at c ^ (r & 15).  Element e of lane (g, n) of
    // accumulator q of block (i, j) is feature 32i + 16(q/2) + 4g + e, token 32j + 16(q%2) + n.
    LIN_PHASE_HEAD(0);
    asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");  // sixteen wait states between the last MFMA and the first read of its results
#undef LIN_PHASE_HEAD
    const int f_wave = n0 + wn * 32 * NI, t_wave = t0 + wt * 32 * NJ;
    char *const out = reinterpret_cast<char *>(smem) + wave * 16384;
    const bool final_rows = p.splits == 1;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        __builtin_amdgcn_sched_barrier(0);
        lin_wavefront_lds_order();  // the reads of the strip that the same LDS held before
        // The strip's results and the lane's index become values that the compiler cannot have read before: copies of all accumulators, or
        // places of all strips, made in front of the first one, would not fit the registers, and what is stored away for
        // that is stored next to the last MFMAs, which the compiler does not know to wait for.
        int strip_lane = lane;
        asm volatile("" : "+v"(strip_lane));
        strip_lane &= 63;  // known to the compiler again: rows and pieces without signed divisions
        const int n = strip_lane & 15, g = strip_lane >> 4;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) asm volatile("" : "+a"(acc[i][j][q]));
        if (final_rows) {
            constexpr int PIECES = 4 * NI;                // of a token's row of this wavefront, bf16
            char *const buf = out + (j & 1) * 8192;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<lu32x2 *>(buf + (q % 2 * 16 + n) * 256 + ((i * 4 + q / 2 * 2 + g / 2) ^ n) * 16 + g % 2 * 8) =
                        __builtin_bit_cast(lu32x2, __builtin_convertvector(acc[i][j][q], lbf16x4));
            lin_wavefront_lds_order();
#pragma unroll
            for (int u = 0; u < PIECES / 2; ++u) {
                const int row = (u * 64 + strip_lane) / PIECES, c = (u * 64 + strip_lane) % PIECES;
                const lu32x4 v = *reinterpret_cast<const lu32x4 *>(buf + row * 256 + (c ^ (row & 15)) * 16);
                const int t = t_wave + j * 32 + row, f = f_wave + c * 8;
                if (t < p.T && f < p.N) *reinterpret_cast<lu32x4_at8 *>(p.y + (int64_t)t * p.y_stride + f) = v;
            }
        } else {
            constexpr int PIECES = 8 * NI;                // the same, fp32
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<lf32x4 *>(out + (q % 2 * 16 + n) * 512 + ((i * 8 + q / 2 * 4 + g) ^ n) * 16) = acc[i][j][q];
            lin_wavefront_lds_order();
#pragma unroll
            for (int u = 0; u < PIECES / 2; ++u) {
                const int row = (u * 64 + strip_lane) / PIECES, c = (u * 64 + strip_lane) % PIECES;
                const lf32x4 v = *reinterpret_cast<const lf32x4 *>(out + row * 512 + (c ^ (row & 15)) * 16);
                const int t = t_wave + j * 32 + row, f = f_wave + c * 4;
                if (t < p.T && f < p.N) *reinterpret_cast<lf32x4 *>(p.part + ((int64_t)wi.split * p.T + t) * p.N + f) = v;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// A few tokens: a workgroup owns F features, so many that the layer is one workgroup per compute unit, and its wavefronts
// share the k range among themselves and add up in LDS: no partial tiles in memory and no second kernel.  A wavefront takes
// every eighth (fourth) stage of 64 k, so that the workgroup reads runs of 1 KiB of each row, brings weight rows and token rows to a
// ring of its own by direct loads and needs no barrier in the loop.  (Operands loaded straight into registers touch sixteen rows
// at once, which the vector-memory path of a compute unit serves at half the rate.)
// Bound by fetching the weights; every compute unit also pulls all token rows, out of L2, which tells beyond 16 tokens on a
// long k range: mixed like that a unit pulls 50 to 65 GB/s.  us a call (weights from memory), cut along k as before and
// now: 8 x 4096 x 4096 11.1 and 7.0 (4.9 at 6.8 TB/s), 8 x 6144 x 4096 13.3 and 9.3 (7.4), 8 x 4096 x 14336 23.5 and 19.6 (17.3),
// 16 x 4096 x 14336 24.1 and 22.3, 16 x 12288 x 4096 20.5 and 16.7 (14.8), 8 x 20480 x 7168 48.4 and 44.5 (43.2),
// 8 x 28672 x 4096 36.9 and 36.0 (34.5), 32 x 6144 x 4096 15.0 and 11.4.
// ---------------------------------------------------------------------------------------
constexpr int kThinTokens = 32;
template <int FROM, typename F>
__device__ __forceinline__ void lin_count_down(F &&f) {  // f(FROM), ..., f(0), as constants
    f(std::integral_constant<int, FROM>{});
    if constexpr (FROM > 0) lin_count_down<FROM - 1>(f);
}
template <int F, int XR, int WAVES, int RING>
__global__ __launch_bounds__(64 * WAVES, 1) void linear_thin_kernel(LinearParams p) {
    constexpr int KS = kLinStageK;
    constexpr int ROWS = F + XR;             // of a stage: weights, then tokens
    constexpr int STAGE = ROWS * KS;
    constexpr int W_LOADS = F / 8, X_LOADS = XR / 8, LOADS = W_LOADS + X_LOADS;
    constexpr int TILES = (F + 15) / 16;     // MFMA tiles of 16 features; the last may be half used
    constexpr int NJ = (XR + 15) / 16;       // MFMA tiles of 16 tokens
    constexpr int STRIDE = F + 4;            // floats between the tokens of a wavefront's sums
    static_assert(WAVES * RING * STAGE * 2 <= 160 * 1024 && NJ * 16 * STRIDE * 4 <= RING * STAGE * 2, "LDS of a compute unit; the sums fit the ring");
    static_assert(RING * LOADS < 64, "the vector-memory counter holds 63 loads");
    __shared__ __attribute__((aligned(16))) uint16_t smem[WAVES * RING * STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * F;
    auto row_key = [](int row) { return (row >> 1) & 7; };
    int off[LOADS];  // rows past the matrix re-read its last row
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int row = (i < W_LOADS ? i : i - W_LOADS) * 8 + lane / 8;
        const int source = i < W_LOADS ? min(n0 + row, p.N - 1) - n0 : min(row, p.T - 1);
        off[i] = (source * p.K + ((lane % 8) ^ row_key(row)) * 8) * 2;
    }
    const uint16_t *const w_base = p.w + (int64_t)n0 * p.K;
    uint16_t *const ring = smem + wave * RING * STAGE;
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(lin_lds_ptr)(ring);
    const int n_stages = p.K / KS;
    // Workgroups start at different places of the k range: lin_first_stage says why.  The places are kStagger stages apart, and the
    // features of a workgroup must not be a multiple of that: with 3 and 96 features of 4096 k, workgroup b's rows lie b x 3 x 2^18
    // bytes in and its first stage b x 3 x 2^7, so that the bits that pick the memory channel cancel (us a call with 3 and 5:
    // 8 x 24576 x 4096 42.3 and 31.2, 8 x 10240 x 8192 28.6 and 26.0; 5 everywhere moves that to 80 features: 8 x 20480 x 8192
    // 51.8 and 59.4).
    constexpr int kStagger = F % 3 == 0 ? 5 : 3;
    static_assert(F % kStagger != 0, "the start places would fall on few memory channels");
    const int first = __builtin_amdgcn_readfirstlane((int)blockIdx.x * kStagger % n_stages);
    const int mine = (n_stages - wave + WAVES - 1) / WAVES;  // stages wave, wave + 8, ... counted from `first`
    auto issue = [&](int i, int slot) {
        int at = first + wave + i * WAVES;
        if (at >= n_stages) at -= n_stages;
        const uint32_t dst = ring_addr + (uint32_t)(slot * STAGE * 2);
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            if (l < W_LOADS) lin_dma_load_16_stream(w_base + at * KS, off[l], dst + (uint32_t)l * 1024);
            else lin_dma_load_16(p.x + at * KS, off[l], dst + (uint32_t)l * 1024);
        }
    };
    // operands of v_mfma_f32_16x16x32_bf16: lane (g, n) holds row n, k 8g .. 8g+7; tokens and features past the rows
    // there are shadow earlier ones, and their results are not used
    const int n = lane & 15, g = lane >> 4;
    int a_rd[TILES][2], b_rd[NJ][2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int a = 0; a < TILES; ++a) {
            const int row = a * 16 + (a * 16 + 16 > F ? n & 7 : n);
            a_rd[a][s] = row * KS + ((4 * s + g) ^ row_key(row)) * 8;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int row = min(j * 16 + n, XR - 1);
            b_rd[j][s] = (F + row) * KS + ((4 * s + g) ^ row_key(row)) * 8;
        }
    }
    lf32x4 acc[TILES][NJ];
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[a][j] = lf32x4{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int slot) {
        asm volatile("" ::: "memory");
        const uint16_t *sp = ring + slot * STAGE;
        lbf16x8 fa[TILES][2], fb[NJ][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) fb[j][s] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + b_rd[j][s]));
#pragma unroll
            for (int a = 0; a < TILES; ++a) fa[a][s] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + a_rd[a][s]));
        }
        LIN_WAIT_LDS();  // in registers: the slot may be filled again
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int a = 0; a < TILES; ++a)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a][s], fb[j][s], acc[a][j], 0, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < RING; ++i)
        if (i < mine) issue(i, i);
    int slot = 0, i = 0;
    for (; i + RING < mine; ++i) {
        LIN_WAIT_VMCNT_AND_LDS((RING - 1) * LOADS);
        consume(slot);
        issue(i + RING, slot);
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
    lin_count_down<RING - 1>([&](auto left) {  // the last stages: nothing more to issue
        if (i + decltype(left)::value < mine) {
            LIN_WAIT_VMCNT_AND_LDS(decltype(left)::value * LOADS);
            consume(slot);
            slot = slot + 1 == RING ? 0 : slot + 1;
            ++i;
        }
    });
    // sums of this wavefront where its ring was: lane (g, n) holds token n, features 16a + 4g ..
    float *const sums = reinterpret_cast<float *>(ring);
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (a * 16 + 4 * g < F) *reinterpret_cast<lf32x4 *>(sums + (j * 16 + n) * STRIDE + a * 16 + 4 * g) = acc[a][j];
    __syncthreads();
    for (int e = (int)threadIdx.x; e < p.T * (F / 2); e += 64 * WAVES) {
        const int t = e / (F / 2), f = e % (F / 2) * 2;
        if (n0 + f >= p.N) continue;
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float *part = reinterpret_cast<const float *>(smem + w * RING * STAGE) + t * STRIDE + f;
            s0 += part[0];
            s1 += part[1];
        }
        typedef __attribute__((ext_vector_type(2))) float lf32x2;
        typedef __attribute__((ext_vector_type(2))) __bf16 lbf16x2;
        *reinterpret_cast<uint32_t *>(p.y + (int64_t)t * p.N + n0 + f) = __builtin_bit_cast(uint32_t, __builtin_convertvector(lf32x2{s0, s1}, lbf16x2));
    }
}

// ---------------------------------------------------------------------------------------
// 17 to 96 tokens, where cutting k costs partial tiles and a second kernel: as in linear_thin_kernel a workgroup per compute unit
// owns F features and the whole k range, but the token rows are too many for a ring per wavefront.  Four wavefronts share stages
// of 128 k (F weight rows and XR token rows of two lines each); wavefront w works on k 32w .. 32w + 31 of every stage
// with all results in registers (F / 16 x XR / 16 tiles), and the four sums meet in LDS at the end.
// Bound by what a compute unit pulls: its weights from memory and all token rows out of L2, together at about 65 GB/s.  us a
// call, cut along k and so: 77 x 20480 x 7168 59.9 and 53.6 (43.2 at 6.8 TB/s), 77 x 14848 x 3712 28.6 and 24.5 (16.2),
// 77 x 7168 x 3584 18.5 and 17.4 (7.6), 77 x 8192 x 2048 13.6 and 11.2, 77 x 14336 x 8192 49.0 and 46.3, 96 x 12288 x 2048 17.2 and 15.1;
// with fewer tokens fewer token rows: 36 x 20480 x 7168 53.6 and 45.5, 45 x 7168 x 3584 17.0 and 13.4, 63 x 15360 x 2944 24.0 and 19.8.
// ---------------------------------------------------------------------------------------
constexpr int kMidStageK = 128;
template <int F, int XR>
struct MidShape {
    static constexpr int kStageBytes = (F + XR) * kMidStageK * 2;
    static constexpr int kRing = std::min(6, 160 * 1024 / kStageBytes);
};
template <int F, int XR>
__global__ __launch_bounds__(256, 1) void linear_mid_kernel(LinearParams p) {
    constexpr int KS = kMidStageK, RING = MidShape<F, XR>::kRing, STAGE = (F + XR) * KS;
    constexpr int NI = F / 16, NJ = XR / 16;
    constexpr int LOADS = (F + XR) / 16;      // 1 KiB loads (four rows) of a wavefront per stage
    static_assert(RING >= 2 && F % 16 == 0 && XR % 16 == 0 && (RING - 1) * LOADS < 64, "");
    __shared__ __attribute__((aligned(16))) uint16_t smem[RING * STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * F;
    // load l of wavefront w moves rows 4 (4 l + w) ..; the sixteen pieces of a row are XOR-swizzled with the row's number modulo 16
    int off[LOADS];
#pragma unroll
    for (int l = 0; l < LOADS; ++l) {
        const int row = 4 * (4 * l + wave) + lane / 16, piece = (lane % 16) ^ (row & 15);
        // F is a multiple of 16: a load is all weights or all tokens.  Rows past the matrix re-read its last row.
        const int source = 16 * l < F ? min(n0 + row, p.N - 1) - n0 : min(row - F, p.T - 1);
        off[l] = (source * p.K + piece * 8) * 2;
    }
    const uint16_t *const w_base = p.w + (int64_t)n0 * p.K;
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lin_lds_ptr)(smem);
    const int n_stages = p.K / KS;
    const int first = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 3 % n_stages);
    auto issue = [&](int stage, int slot) {
        int at = first + stage;
        if (at >= n_stages) at -= n_stages;
        const uint32_t dst = smem_addr + (uint32_t)(slot * STAGE * 2 + wave * 1024);
#pragma unroll
        for (int l = 0; l < LOADS; ++l) {
            if (16 * l < F) lin_dma_load_16_stream(w_base + at * KS, off[l], dst + (uint32_t)l * 4096);
            else lin_dma_load_16(p.x + at * KS, off[l], dst + (uint32_t)l * 4096);
        }
    };
    const int n = lane & 15, g = lane >> 4;
    const int rd = n * KS + ((4 * wave + g) ^ n) * 8;  // row n of a block of sixteen, this wavefront's k
    lf32x4 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = lf32x4{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int slot) {
        const uint16_t *sp = smem + slot * STAGE + rd;
        lbf16x8 fa[NI], fb[NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) fa[i] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + i * 16 * KS));
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[j] = __builtin_bit_cast(lbf16x8, *reinterpret_cast<const lu32x4 *>(sp + (F + j * 16) * KS));
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int st = 0; st < RING - 1; ++st)
        if (st < n_stages) issue(st, st);
    int slot = 0, st = 0;
    for (; st + RING - 1 < n_stages; ++st) {
        // stage st has landed, and behind the barrier everyone's part of it, and everyone has stage st-1 in registers
        LIN_WAIT_VMCNT_AND_LDS((RING - 2) * LOADS);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(st + RING - 1, slot == 0 ? RING - 1 : slot - 1);
        consume(slot);
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
    for (; st < n_stages; ++st) {
        LIN_WAIT_VMCNT_AND_LDS(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        consume(slot);
        slot = slot + 1 == RING ? 0 : slot + 1;
    }
    // the four sums, as many token tiles at a time as LDS holds: lane (g, n) of tile (i, j) has token 16j + n, features 16i + 4g ..
    constexpr int STRIDE = F + 4, PER_WAVE = 16 * STRIDE;  // floats of a token tile
    constexpr int TILES = std::min(NJ, RING * STAGE * 2 / (4 * PER_WAVE * 4));
    static_assert(TILES >= 1, "LDS holds a token tile of every wavefront");
    float *const sums = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int j0 = 0; j0 < NJ; j0 += TILES) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TILES; ++j)
            if (j0 + j < NJ)
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    *reinterpret_cast<lf32x4 *>(sums + (wave * TILES + j) * PER_WAVE + n * STRIDE + i * 16 + 4 * g) = acc[i][j0 + j < NJ ? j0 + j : 0];
        __syncthreads();
        const int tokens = min(TILES * 16, p.T - j0 * 16);
        for (int e = (int)threadIdx.x; e < tokens * (F / 4); e += 256) {
            const int t = e / (F / 4), f = e % (F / 4) * 4;
            if (n0 + f >= p.N) continue;
            lf32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) sum += *reinterpret_cast<const lf32x4 *>(sums + (w * TILES + t / 16) * PER_WAVE + t % 16 * STRIDE + f);
            *reinterpret_cast<lu32x2 *>(p.y + (int64_t)(j0 * 16 + t) * p.N + n0 + f) = __builtin_bit_cast(lu32x2, __builtin_convertvector(sum, lbf16x4));
        }
    }
}

// Adds the split-K pieces of every output element in piece order and rounds once to bf16.  Rows of N (a multiple of 4), in y `y_stride` apart.
__global__ __launch_bounds__(256) void linear_reduce_kernel(const float *part, uint16_t *y, int64_t elems, int splits, int32_t N, int32_t y_stride) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= elems) return;
    lf32x4 sum = *reinterpret_cast<const lf32x4 *>(part + i);
    // four pieces are fetched before any is added (one memory latency per four pieces instead of one per piece;
    // indices past the last piece are clamped to it and not added); the additions keep the piece order
    for (int s = 1; s < splits; s += 4) {
        lf32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const lf32x4 *>(part + (int64_t)min(s + j, splits - 1) * elems + i);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (s + j < splits) sum += v[j];
    }
    int64_t at = i;
    if (N != y_stride) {  // features of a wider row: so few that 32 bits hold their number
        const uint32_t row = (uint32_t)i / (uint32_t)N;
        at = (int64_t)row * y_stride + ((uint32_t)i - row * (uint32_t)N);
    }
    *reinterpret_cast<lu32x2 *>(y + at) = __builtin_bit_cast(lu32x2, __builtin_convertvector(sum, lbf16x4));
}

}  // namespace

// Tile shapes of linear_phased_kernel (its template arguments), with the microseconds of one 64-k stage when every compute unit runs one, for
// batches of several token tiles and of one (weights straight from memory, with the non-temporal hint).
struct PhasedShape {
    int a0, a1, b0, b1, ring;  // LDS: ring x 128 x (features + tokens) bytes, 112 to 160 KiB
    double stage_us, stage_us_one_tile;
    constexpr int32_t features() const { return 64 * (a0 + a1); }
    constexpr int32_t tokens() const { return 64 * (b0 + b1); }
};
constexpr PhasedShape kPhasedShapes[] = {
    {2, 2, 2, 2, 2, 0.654, 0.619}, {2, 2, 2, 1, 2, 0.538, 0.588}, {2, 1, 2, 2, 2, 0.547, 0.545}, {2, 1, 2, 1, 3, 0.502, 0.573},
    {2, 2, 1, 1, 3, 0.530, 0.597}, {1, 1, 2, 2, 3, 0.487, 0.502}, {2, 1, 1, 1, 4, 0.465, 0.552}, {1, 1, 2, 1, 4, 0.413, 0.476},
    {1, 1, 1, 1, 5, 0.377, 0.414}, {2, 2, 1, 0, 4, 0.494, 0.630}, {2, 1, 1, 0, 5, 0.403, 0.526}, {1, 1, 1, 0, 6, 0.292, 0.346},
};
constexpr size_t kNumPhasedShapes = sizeof(kPhasedShapes) / sizeof(kPhasedShapes[0]);

// More than 64 tokens.  Cost of a tiling in microseconds, fitted to 3,600 timings of the kernels with the 32 x 32 x 16 instruction (the 13
// layer shapes of four models, 15 token counts from 40 to 2048, every tile shape and piece count that could compete; met within 7 % rms).
// The present kernels take 0.94 of it, within 6.5 % rms of that (2,809 timings, 260 layers of 65 to 2048 tokens, tilings up to a quarter dearer
// than the chosen one), and the chosen tiling is 1.4 % slower than the best of those on average, 13.6 % at most (554 x 4608 x 7168).
// The largest of
//   rounds of workgroups (one per compute unit) x (stages per piece x stage time + the tile's way out, 8.2 us for 256 x 256),
//   the padded product at 2.26 PFLOP/s, and the weights at 8.05 TB/s,
// plus 0.53 of the other two (none hides the others entirely), 4.3 us per launch, and for pieces of k their fp32 partial
// tiles, written and read back at 6.2 TB/s, and 1.2 us for the second kernel.
// `limit`: a cost from which on no plan is wanted; `cost` is then at least that.
static LinearPlan plan_phased(int32_t T, int32_t N, int32_t K, size_t workspace_bytes, double *cost = nullptr, double limit = 1.0e12) {
    const int64_t k_stages = K / kLinStageK;
    const int64_t per_split_bytes = (int64_t)T * N * 4;
    const double memory_us = 2.0 * N * K / 8.05e6;
    LinearPlan best{};
    double best_cost = -1.0;
    if (cost) *cost = limit;
    for (const PhasedShape &sh : kPhasedShapes) {
        const int64_t n_tiles = (N + sh.features() - 1) / sh.features();
        const int64_t t_tiles = (T + sh.tokens() - 1) / sh.tokens();
        const int64_t tiles = n_tiles * t_tiles;
        const double stage_us = t_tiles == 1 ? sh.stage_us_one_tile : sh.stage_us;
        const double out_us = 8.2 * sh.features() * sh.tokens() / 65536.0;
        const double product_us = 2.0 * (double)tiles * sh.features() * sh.tokens() * K / 2.26e9;
        if (4.3 + product_us >= limit) continue;
        for (int64_t s = 1; s <= 16 && (s == 1 || (s * 4 <= k_stages && tiles * s <= 1024)); ++s) {
            if (s > 1 && (size_t)(s * per_split_bytes) > workspace_bytes) break;
            const int64_t stages = (k_stages + s - 1) / s;
            const int64_t pieces = (k_stages + stages - 1) / stages;
            if (pieces != s) continue;  // the same stages per piece in fewer pieces has been looked at
            const double rounds = (double)((tiles * s + 255) / 256);
            const double compute_us = rounds * ((double)stages * stage_us + out_us);
            const double longest = std::max(compute_us, std::max(product_us, memory_us));
            double c = 4.3 + longest + 0.53 * (compute_us + product_us + memory_us - longest);
            if (s > 1) c += 1.2 + 2.0 * (double)s * (double)per_split_bytes / 6.2e6;
            if (best_cost < 0.0 || c < best_cost) {
                best_cost = c;
                best.feature_tile = sh.features();
                best.token_tile = sh.tokens();
                best.n_tiles = (int32_t)n_tiles;
                best.t_tiles = (int32_t)t_tiles;
                best.splits = (int32_t)s;
                best.k_per_split = s == 1 ? K : (int32_t)(stages * kLinStageK);
            }
        }
    }
    if (cost && best_cost >= 0.0) *cost = std::min(best_cost, limit);
    return best;
}

// Up to 64 tokens otherwise: 128 or 256 features x 64 tokens of linear_kernel, cut along k so that a small batch streams the weights
// through every compute unit.  Cost in microseconds, fitted to 1,900 timings (16 layer shapes, 1 to 64 tokens, 1 to 16
// pieces; 6 % rms, the chosen tiling 1 % slower than the best one): as above with the weights at 9.9 TB/s in a maximum that
// is approached from above by 0.61 of the smaller term, 0.13 us per stage for a full 64 tokens, 3.6 us for the second kernel
// and 3.7 TB/s for the partial tiles.  (128 features win nearly everywhere: 8 x 4096 x 4096 in 8 pieces 11.4 us, 256
// features x 32 tokens in 16 pieces, the tile this range had besides, 14.9.)
static LinearPlan plan_small(int32_t T, int32_t N, int32_t K, size_t workspace_bytes) {
    const int64_t k_stages = K / kLinStageK;
    const int64_t per_split_bytes = (int64_t)T * N * 4;
    const double memory_us = 2.0 * N * K / 9.94e6;
    LinearPlan best{};
    double best_cost = -1.0;
    for (const int32_t features : {128, 256}) {
        const int64_t n_tiles = (N + features - 1) / features;
        const double stage_us = (features == 128 ? 0.256 : 0.468) + 0.128 * T / 64.0;
        for (int64_t s = 1; s <= 16 && (s == 1 || (s * 4 <= k_stages && n_tiles * s <= 1024)); ++s) {
            if (s > 1 && (size_t)(s * per_split_bytes) > workspace_bytes) break;
            const int64_t stages = (k_stages + s - 1) / s;
            if ((k_stages + stages - 1) / stages != s) continue;  // the same stages per piece in fewer pieces has been looked at
            const double compute_us = (double)((n_tiles * s + 255) / 256) * ((double)stages * stage_us + 2.03 * features / 256.0);
            double c = 1.5 + std::max(compute_us, memory_us) + 0.61 * std::min(compute_us, memory_us);
            if (s > 1) c += 3.6 + 2.0 * (double)s * (double)per_split_bytes / 3.7e6;
            if (best_cost < 0.0 || c < best_cost) {
                best_cost = c;
                best.feature_tile = features;
                best.token_tile = kLinSmallTokens;
                best.n_tiles = (int32_t)n_tiles;
                best.t_tiles = 1;
                best.splits = (int32_t)s;
                best.k_per_split = s == 1 ? K : (int32_t)(stages * kLinStageK);
            }
        }
    }
    return best;
}

// Features of a workgroup of linear_thin_kernel: as few as give a workgroup per compute unit at most; 0: not for this layer.
// Beyond 16 tokens the token rows that every workgroup pulls grow with T x K (us cut along k and thin: 24 x 4096 x 4096 12.2 and
// 8.6, 20 x 2560 x 8192 14.2 and 12.7, 24 x 4608 x 7168 17.8 and 16.2, 32 x 4608 x 7168 17.7 and 17.9, 24 x 4096 x 14336 24.8 and
// 25.5, 32 x 4096 x 14336 25.5 and 28.7).  Few features leave too many compute units idle (16 x 1024 x 8192 11.0 and 10.2,
// 32 x 1024 x 8192 11.6 and 13.7; 16 x 1536 x 4096 10.1 and 6.4).
// Where features are few next to the compute units and k is long, a workgroup's own K (F + 0.8 T) elements are what the layer
// waits for (beyond 16 tokens as many token rows as it loads, 24 or 32): at the same 50 GB/s a layer cut along k streams N / 190 as
// many at once and pays 7.6 us for its second kernel (16 x 1536 x 49152 29.8 and 59.7, 8 x 1664 x 49152 30.6 and 48.2,
// 12 x 1664 x 17152 15.8 and 20.6, 16 x 4224 x 49152 71.2 and 86.2, 17 x 1536 x 10240 13.1 and 15.7; on the other side of the line
// 16 x 1536 x 8192 11.9 and 10.7, 16 x 4096 x 16384 25.6 and 22.5, 8 x 8192 x 28672 73.2 and 68.7, 17 x 7168 x 10240 28.2 and 27.0).
// Of 3,170 layers of 1536 to 32,768 features and k up to 65,536 45 are 3 to 10 % slower so than cut, and 20 that are cut would be
// 3 to 11 % faster thin; without the line 383 were slower, by up to a factor of two.
// Beyond 8192 features the line at 3072 k is where this kernel was first looked at, not where it stops to gain (8 x 9216 x 2048 11.7
// cut along k and 7.9 thin, 8 x 12288 x 1024 9.3 and 6.0, 16 x 24576 x 2048 18.7 and 17.0, 8 x 8320 x 192 5.4 and 5.3).
static int32_t thin_features(int32_t T, int32_t N, int32_t K) {
    if (T > kThinTokens || N < 1536 || (T > 16 && (int64_t)T * K > 200000)) return 0;
    for (const int f : {16, 24, 32, 48, 64, 80, 96, 112, 128}) {
        if (N > f * 256) continue;
        const int32_t rows = T > 16 ? (T + 7) / 8 * 8 : std::max(T, 4);
        if ((double)K * (190.0 * (f + 0.8 * rows) - N) >= (T > 16 ? 3.8e7 : 3.6e7)) return 0;
        return f <= 32 || (T <= 16 && K >= 3072) ? f : 0;
    }
    return 0;
}

// Features of a workgroup of linear_mid_kernel, or 0: not for this layer.  The token rows that every workgroup pulls grow with k and
// are paid for by its features, and the features have to fill the compute units (us cut along k and so: 77 x 6144 x 4096, 192
// workgroups, 18.0 and 18.7; 77 x 8192 x 7168 27.7 and 31.9; 77 x 7168 x 10240 37.1 and 46.5; 77 x 14848 x 14848 81.6 and 85.7).
// Beyond 80 tokens the line lies lower (85 x 14336 x 8192 49.3 and 52.1, 85 x 7168 x 3584 19.1 and 18.7), and beyond 96 next to
// nothing is left (128 x 6144 x 4096 20.1 and 24.0); 112 features leave two or three stages in LDS (77 x 28672 x 4096 42.8 and 43.4).
// 64 features with 96 token rows lose on their way in and out what they gain in the loop until k is long enough (81 x 14848 x 512 7.1
// and 7.4, 81 x 13824 x 1024 10.0 and 10.4, 96 x 16384 x 1024 10.8 and 10.8, 81 x 13824 x 2048 17.4 and 15.9).
static int32_t mid_features(int32_t T, int32_t N, int32_t K) {
    if (T <= kLinSmallTokens || T > 96 || K % kMidStageK != 0) return 0;
    for (const int f : {32, 48, 64, 80})
        if (N <= f * 256) return N >= f * 208 && K + 1024 <= (T <= 80 ? 144 : 96) * f && (T <= 80 || f != 64 || K > 1024) ? f : 0;
    return 0;
}

// The same for 17 to 64 tokens where linear_thin_kernel does not take them.  Cut along k pays 4 us for its second kernel, this for the token rows, K
// of them per workgroup, so the line falls with the tokens and rises where k is short.  us a call, cut and so: 20 x 14336 x 8192 41.6 and 37.0,
// 20 x 12288 x 2048 13.9 and 10.9, 32 x 20480 x 7168 52.2 and 45.4, 32 x 8192 x 7168 23.2 and 22.5, 32 x 14848 x 14848 72.4 and 70.4; 48 of them
// 74.1 and 77.0, 48 x 4096 x 4096 14.5 and 11.4, 48 x 6144 x 4096 16.6 and 14.6, 48 x 14336 x 8192 44.1 and 40.1, 48 x 8192 x 7168 24.3 and 24.5,
// 48 x 7168 x 10240 32.1 and 34.3, 33 x 4608 x 7168 18.0 and 20.5; 64 x 8192 x 2048 12.8 and 10.1, 64 x 6144 x 4096 18.0 and 16.6, 64 x 20480 x 7168
// 55.3 and 49.4, 64 x 10240 x 8192 35.6 and 40.2.  16 features with 64 token rows (64 x 4096 x 4096 15.8 and 12.8) and 112 features (48 x 28672 x
// 4096 38.1 and 38.2) are left as they were.  Of 160 drawn layers that run so none is slower, 1.165 x faster on average.
static int32_t few_features(int32_t T, int32_t N, int32_t K) {
    if (T <= 16 || T > kLinSmallTokens || K % kMidStageK != 0) return 0;
    const int64_t k_per_feature = T <= 32 ? 260 : T <= 48 ? 215 : 180, on_short_ranges = T <= 48 ? 330 : 215;
    if (256 * ((int64_t)K + 1024) > N * (K <= 4096 ? std::max(k_per_feature, on_short_ranges) : k_per_feature)) return 0;
    for (const int f : {16, 32, 48, 64, 80, 96})
        if (N <= f * 256) return N >= f * 160 && (f > 16 || T <= 48) ? f : 0;
    return 0;
}

LinearPlan plan_linear(int32_t T, int32_t N, int32_t K, size_t workspace_bytes) {
    if (const int32_t f = mid_features(T, N, K)) return LinearPlan{f, T <= 80 ? 80 : 96, (N + f - 1) / f, 1, 1, K};
    if (const int32_t f = thin_features(T, N, K)) return LinearPlan{f, kThinTokens, (N + f - 1) / f, 1, 1, K};
    if (const int32_t f = few_features(T, N, K)) return LinearPlan{f, T <= 48 ? 48 : 64, (N + f - 1) / f, 1, 1, K};
    return T > kLinSmallTokens ? plan_phased(T, N, K, workspace_bytes) : plan_small(T, N, K, workspace_bytes);
}

// More tiles than compute units: the features of the full rounds of one shape as they are, and the others, whose round would be partly
// filled, with the tiling that suits them, in a launch of their own; taken where the two costs together are below the one.
// us a call, one tiling and two: 2048 x 14336 x 8192 (448 tiles of 256 x 256) 346 and 323, 1156 x 14336 x 8192 (375 of 192 x 256) 256
// and 217, 562 x 24192 x 3840 117 and 99, 1284 x 28672 x 4096 267 and 243, 576 x 28672 x 4096, estimated 2 % dearer, 128 and 126.  260
// drawn layers that run so are 1.066 x faster on average, and one is slower (375 x 16640 x 9344, a full round and 256 features, 128.0 and 131.4).
// Up to 96 tokens one token tile covers the batch.
LinearParts plan_linear_parts(int32_t T, int32_t N, int32_t K, size_t workspace_bytes) {
    LinearParts best{N, {plan_linear(T, N, K, workspace_bytes), LinearPlan{}}};
    if (T <= 96 || (int64_t)best.part[0].n_tiles * best.part[0].t_tiles <= 128) return best;
    double bar;
    plan_phased(T, N, K, workspace_bytes, &bar);
    const double feature_us = 2.0 * T * (double)K / 2.26e9, k_stages = K / kLinStageK;
    for (const PhasedShape &sh : kPhasedShapes) {
        const int64_t n_tiles = (N + sh.features() - 1) / sh.features(), t_tiles = (T + sh.tokens() - 1) / sh.tokens();
        const int64_t rounds = n_tiles * t_tiles / 256;
        if (rounds == 0 || t_tiles == 1) continue;
        const int32_t whole = (int32_t)(rounds * 256 / t_tiles), first = whole * sh.features();
        if (whole == 0 || first >= N) continue;
        const double compute_us = (double)rounds * (k_stages * sh.stage_us + 8.2 * sh.features() * sh.tokens() / 65536.0);
        const double product_us = 2.0 * whole * (double)t_tiles * sh.features() * sh.tokens() * K / 2.26e9, memory_us = 2.0 * first * K / 8.05e6;
        const double longest = std::max(compute_us, std::max(product_us, memory_us));
        const double first_us = 4.3 + longest + 0.53 * (compute_us + product_us + memory_us - longest);
        if (first_us + 1.53 * (N - first) * feature_us >= bar) continue;  // (the least that the rest can cost)
        double rest_us;
        const LinearPlan rest = plan_phased(T, N - first, K, workspace_bytes, &rest_us, bar - first_us);
        if (rest.n_tiles == 0 || first_us + rest_us >= bar) continue;  // (none below the limit, whatever the two sums round to)
        bar = first_us + rest_us;
        best = LinearParts{first, {LinearPlan{sh.features(), sh.tokens(), whole, (int32_t)t_tiles, 1, K}, rest}};
    }
    return best;
}

// Launches the shape of the table that the plan names; false if it names none of them.
template <size_t I>
static bool launch_phased_shape(const LinearPlan &pl, const LinearParams &p, dim3 grid, hipStream_t st) {
    constexpr PhasedShape sh = kPhasedShapes[I];
    if (pl.feature_tile != sh.features() || pl.token_tile != sh.tokens()) return false;
    if constexpr (sh.b1 > 0) {  // a 64-token tile never covers these batches alone
        if (pl.t_tiles == 1) {
            hipLaunchKernelGGL((linear_phased_kernel<sh.a0, sh.a1, sh.b0, sh.b1, sh.ring, true>), grid, dim3(256), 0, st, p);
            return true;
        }
    }
    hipLaunchKernelGGL((linear_phased_kernel<sh.a0, sh.a1, sh.b0, sh.b1, sh.ring, false>), grid, dim3(256), 0, st, p);
    return true;
}
template <size_t... I>
static bool launch_phased(const LinearPlan &pl, const LinearParams &p, dim3 grid, hipStream_t st, std::index_sequence<I...>) {
    return (launch_phased_shape<I>(pl, p, grid, st) || ...);
}

static int launch_part(const LinearPlan &pl, const void *x, const void *w, void *y, int32_t T, int32_t N, int32_t K, int32_t y_stride,
                       void *workspace, void *stream) {
    LinearParams p;
    p.x = static_cast<const uint16_t *>(x);
    p.w = static_cast<const uint16_t *>(w);
    p.y = static_cast<uint16_t *>(y);
    p.part = static_cast<float *>(workspace);
    p.T = T; p.N = N; p.K = K; p.y_stride = y_stride;
    p.n_tiles = pl.n_tiles; p.t_tiles = pl.t_tiles; p.splits = pl.splits; p.k_per_split = pl.k_per_split;
    const int64_t items = (int64_t)pl.n_tiles * pl.t_tiles * pl.splits;
    const int64_t blocks = (items + kLinXcds - 1) / kLinXcds * kLinXcds;
    if (blocks > 0x7FFFFFFF) return (int)hipErrorInvalidValue;  // more workgroups than a grid holds
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)blocks);
    if (pl.token_tile == kThinTokens) {
        if (T > kThinTokens || pl.splits != 1) return (int)hipErrorInvalidConfiguration;
        auto launch = [&](auto f) {
            constexpr int F = decltype(f)::value;
            auto with = [&](auto xr) {
                constexpr int XR = decltype(xr)::value, WAVES = F <= 64 ? 8 : 4, kStage = (F + XR) * 128 * WAVES;  // bytes, of all wavefronts
                constexpr int RING = std::min(6, 160 * 1024 / kStage);
                hipLaunchKernelGGL((linear_thin_kernel<F, XR, WAVES, RING>), dim3((unsigned)pl.n_tiles), dim3(64 * WAVES), 0, st, p);
            };
            if (T <= 8) with(std::integral_constant<int, 8>{});
            else if (T <= 16) with(std::integral_constant<int, 16>{});
            else if constexpr (F <= 32) {
                if (T <= 24) with(std::integral_constant<int, 24>{});
                else with(std::integral_constant<int, 32>{});
            }
        };
        if (T > 16 && pl.feature_tile > 32) return (int)hipErrorInvalidConfiguration;
        if (pl.feature_tile == 16) launch(std::integral_constant<int, 16>{});
        else if (pl.feature_tile == 24) launch(std::integral_constant<int, 24>{});
        else if (pl.feature_tile == 32) launch(std::integral_constant<int, 32>{});
        else if (pl.feature_tile == 48) launch(std::integral_constant<int, 48>{});
        else if (pl.feature_tile == 64) launch(std::integral_constant<int, 64>{});
        else if (pl.feature_tile == 80) launch(std::integral_constant<int, 80>{});
        else if (pl.feature_tile == 96) launch(std::integral_constant<int, 96>{});
        else if (pl.feature_tile == 112) launch(std::integral_constant<int, 112>{});
        else if (pl.feature_tile == 128) launch(std::integral_constant<int, 128>{});
        else return (int)hipErrorInvalidConfiguration;
        return (int)hipGetLastError();
    }
    if (pl.token_tile == 48 || pl.token_tile == 80 || pl.token_tile == 96 || (pl.token_tile == 64 && pl.feature_tile < 128)) {
        bool known = false;
        auto with = [&](auto f, auto xr) {
            if (pl.feature_tile != decltype(f)::value || pl.token_tile != decltype(xr)::value || T > decltype(xr)::value) return;
            hipLaunchKernelGGL((linear_mid_kernel<decltype(f)::value, decltype(xr)::value>), dim3((unsigned)pl.n_tiles), dim3(256), 0, st, p);
            known = true;
        };
        auto few_rows = [&](auto f) {
            with(f, std::integral_constant<int, 48>{});
            with(f, std::integral_constant<int, 64>{});
        };
        auto rows = [&](auto f) {
            few_rows(f);
            with(f, std::integral_constant<int, 80>{});
            with(f, std::integral_constant<int, 96>{});
        };
        with(std::integral_constant<int, 16>{}, std::integral_constant<int, 48>{});
        few_rows(std::integral_constant<int, 96>{});
        rows(std::integral_constant<int, 32>{});
        rows(std::integral_constant<int, 48>{});
        rows(std::integral_constant<int, 64>{});
        rows(std::integral_constant<int, 80>{});
        return known ? (int)hipGetLastError() : (int)hipErrorInvalidConfiguration;
    }
    if (T > kLinSmallTokens) {
        if (!launch_phased(pl, p, grid, st, std::make_index_sequence<kNumPhasedShapes>{})) return (int)hipErrorInvalidConfiguration;
    } else if (pl.feature_tile == 128) {  // LDS: 6 x 24 KiB, 3 x 40 KiB
        hipLaunchKernelGGL((linear_kernel<64, 2, 6, 128>), grid, dim3(kLinThreads), 0, st, p);
    } else if (pl.feature_tile == 256) {
        hipLaunchKernelGGL((linear_kernel<64, 1, 3, 256>), grid, dim3(kLinThreads), 0, st, p);
    } else {
        return (int)hipErrorInvalidConfiguration;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.splits == 1) return (int)e;
    const int64_t elems = (int64_t)T * N;
    hipLaunchKernelGGL(linear_reduce_kernel, dim3((unsigned)((elems / 4 + 255) / 256)), dim3(256), 0, st, p.part, p.y, elems, pl.splits, N, y_stride);
    return (int)hipGetLastError();
}

int launch_linear(const LinearPlan &pl, const void *x, const void *w, void *y, int32_t T, int32_t N, int32_t K, void *workspace, void *stream) {
    return launch_part(pl, x, w, y, T, N, K, N, workspace, stream);
}

int launch_linear_parts(const LinearParts &parts, const void *x, const void *w, void *y, int32_t T, int32_t N, int32_t K, void *workspace, void *stream) {
    const int32_t first = parts.first_features;
    const int e = launch_part(parts.part[0], x, w, y, T, first, K, N, workspace, stream);
    if (e != (int)hipSuccess || first >= N) return e;
    // the workspace is free again when the first part's launches have ended, in the order of the stream
    return launch_part(parts.part[1], x, static_cast<const uint16_t *>(w) + (int64_t)first * K, static_cast<uint16_t *>(y) + first, T, N - first, K, N, workspace, stream);
}

}  // namespace sarathi
