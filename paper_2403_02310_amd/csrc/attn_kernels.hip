// gfx950 kernels of libsarathi: KV append, hybrid-batch attention over the paged cache,
// and the split-KV merge.
//
// Attention kernel (16-column wave tile).  A work item is 16 query COLUMNS (col = row*G +
// head_in_group, all sharing one KV head) against a key range; a workgroup of four wavefronts owns
// it, each wavefront walks a quarter of the keys in tiles of 32 (two pages), and the four results
// are merged in LDS (a decode has four memory streams from its first cycle and ends four times
// sooner than on one wavefront).  Both contractions run on v_mfma_f32_16x16x32_bf16 in the
// TRANSPOSED form so that the score accumulators already are the operand of the second one:
//
//   S^T[key, col] = sum_c K[key, c] * Q[col, c]      A = K tile (16 keys x 32 ch), B = Q^T
//   O^T[c,  col] += sum_key V^T[c, key] * P^T[key, col]   A = V^T tile (16 ch x 32 keys), B = P^T
//
// Operand layout of the instruction (64 lanes; g = lane/16, n = lane%16): A lane holds row n,
// contraction indices 8g..8g+7; B lane holds column n, contraction indices 8g..8g+7; the
// accumulator lane holds column n, rows 4g..4g+3.  With the K rows of the two score MFMAs of a
// tile assigned as  row 4g'+i of MFMA b  <->  key 8g'+4b+i,  lane (g, n) ends up with the eight
// scores of column n for keys 8g..8g+7 of the tile: exactly the B operand (P^T) of the second
// contraction, and V^T for those eight keys is one 16-byte run of the channel-major V page.
// The softmax is per-lane work plus two cross-lane steps (lanes n, n+16, n+32, n+48); there are no barriers in the key loop.
// K and V reach the operands through LDS: direct global -> LDS loads of whole pages into a ring that each wavefront has for
// itself.  Loaded straight into operands, sixteen neighbouring lanes touch sixteen K rows (or 32-byte V^T rows) at once, and
// the vector-memory path of a compute unit handles such a load at half the rate of one that reads 1 KiB front to back: 57
// against 90 to 106 GB/s for one compute unit out of its caches, 36 against 52 from memory while 64 of them stream.  That path
// is what decodes share with the chunk tiles of the same launch.  Straight into operands, and through LDS: 512 tokens behind
// 1871 next to 64 decodes, 32 and 8 heads, 124.1 and 107.6 us a call; 256 decodes 224.0 and 216.7; 512 decodes of 64 channels, 58
// and 2 heads, 173 and 123.  (The first two with the streaming hint, the last one without.  Next to chunk
// tiles neither gains alone: 124.6 us with neither, 121.7 with the hint, 124.9 through LDS, 110.8 with both on another part.)
//
// Chunk-tile path (prefill chunks).  A workgroup of four wavefronts owns 128 columns of one
// sequence (32 per wave) and walks the key range in 32-key tiles staged once per workgroup in
// LDS (rings of four K tiles and four V tiles filled by direct global -> LDS loads, K three tiles
// ahead of the step and V two; one barrier per tile), so K/V are fetched from L2/HBM once per 128
// columns instead of once per 16.  The contractions use v_mfma_f32_32x32x16_bf16, again in
// transposed form with the K rows of a tile permuted (MFMA row 16u+8a+4h+b <-> key 16u+8h+4a+b)
// so that accumulator lane (h, n) holds, for column n, keys 8h..8h+7 of page u in registers
// 8u..8u+7: the B operand of the second contraction without any data movement.  K rows are
// XOR-swizzled in LDS and the two 16-byte halves of a V^T row are swapped on every other group
// of eight channels, which makes both the staging writes and the operand reads bank-conflict free.
//
// Both paths share one launch: a block runs chunk tiles or wave tiles, one of them or, in long launches, many from a queue, so the
// memory-bound decodes fill the machine next to the MFMA-bound chunk tiles (the paper's reason
// for hybrid batches, section 4.1).
//
// The running maximum is only raised when a tile exceeds it by more than 2^8 (the softmax is
// invariant to the reference point as long as sum and output use the same one), which removes
// the accumulator rescale from almost every tile.
//
// Split-KV.  A tile whose key range was cut into pieces has every piece write its partial
// (reference maximum, sum, unnormalised output) triple; a second, small kernel merges the
// pieces of each tile in index order, so the result is bitwise reproducible.  (Merging inside
// the attention kernel by the last piece to finish was built twice and dropped on its timings.
// With device-scope release/acquire fences every block writes back and invalidates a whole L2 of
// this multi-die part: several times slower.  Without fences, the partial rows themselves written and
// read with device-scope accesses, whole 512-byte rows at a time, and a piece that finds the others
// done merging without publishing: correct, and still slower than the second kernel in every case
// measured (a 512-token chunk alone 57 us against 40 + 13, chunks of 256 tokens 1,866 us per prompt
// against 1,717), because such accesses bypass the L2 that serves the second kernel's reads, and
// ONE block per tile reads what 16 blocks of the merge kernel read in parallel.)
//
// Masking is by select: keys beyond a column's position (causal mask inside a chunk, section
// 4.1 of the paper) or beyond the item's key range get score -inf; V of slots at or beyond
// ctx_len is zeroed so that stale cache contents (possibly NaN) cannot reach an accumulator.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace sarathi {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

struct AttnParams {
    const uint16_t *q;
    const uint16_t *k_cache;
    const uint16_t *v_cache;
    uint16_t *out;
    const int32_t *block_table;
    const TileDesc *tiles;
    const uint32_t *units;
    float *part_ml;
    float *part_o;
    int64_t num_pages;
    int32_t max_blocks;
    int32_t num_q_heads;
    int32_t num_kv_heads;
    int32_t group;
    int32_t num_tile_units;  // units [0, num_tile_units) are 128-column chunk tiles (one block each)
    int32_t num_units;       // the rest are 16-column wave tiles (one block each as well)
    float scale_log2;        // sm_scale * log2(e): the softmax runs in base 2
    int32_t *sched;          // scheduling words (see internal.h)
    int32_t window;          // sliding window: a query at position p sees keys p-window+1 .. p; 0 = all keys up to p
};

// Arguments of a launch that carries its plan along and reads it where the arguments are: what the allocation-free call does with a
// small plan, instead of a launch of its own that puts it into memory (64 tokens next to three decodes, 4 heads and one, 14.2 -> 11.0 us a
// pass, the host's time for two launches).  Instantiations of their own, and two sizes: 4 KiB of arguments keep the host 0.5 us longer.
constexpr size_t kSmallPlanArgBytes = 960;
template <size_t BYTES>
struct AttnArgs {
    AttnParams base;
    uint32_t units_off;  // bytes from the plan's start to its work units
    uint32_t plan[BYTES / 4];
};
static_assert(sizeof(AttnArgs<kPlanArgBytes>) <= 4096, "kernel arguments are limited to 4 KiB");
__device__ __forceinline__ AttnParams attn_params(const AttnParams &p) { return p; }
template <size_t BYTES>
__device__ __forceinline__ AttnParams attn_params(const AttnArgs<BYTES> &a) {
    AttnParams p = a.base;
    const uintptr_t plan = (uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttnArgs<BYTES>, plan);
    p.tiles = reinterpret_cast<const TileDesc *>(plan);
    p.units = reinterpret_cast<const uint32_t *>(plan + a.units_off);
    return p;
}

// What one work unit (tile, split) covers.
struct UnitRange {
    int32_t key_begin;
    int32_t key_end;   // exclusive
    int32_t part_row;  // first partial row of this split, or -1: write `out` directly
};
__device__ __forceinline__ UnitRange unit_range(const TileDesc &t, int split) {
    UnitRange r;
    r.key_begin = t.key_lo + split * t.keys_per_split;
    r.key_end = min(t.n_keys, r.key_begin + t.keys_per_split);
    r.part_row = t.n_splits > 1 ? t.part_row0 + split * t.n_cols : -1;
    return r;
}

// Read-only int32 data fetched with scalar loads (wave-uniform indices): the block table and the plan.
typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;

__device__ __forceinline__ uint32_t load_unit(const AttnParams &p, int i) {
    return (uint32_t)((const_i32_ptr)p.units)[__builtin_amdgcn_readfirstlane(i)];
}
__device__ __forceinline__ TileDesc load_tile_desc(const AttnParams &p, uint32_t unit) {
    const const_i32_ptr t = (const_i32_ptr)(p.tiles + (unit & ((1u << kUnitTileBits) - 1)));
    return TileDesc{t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], t[9], t[10], t[11]};
}

// Queues of work items.  An item is a unit for one KV head, number unit * Hkv + head; list x of a queue holds the items that
// are x modulo 8, in order, behind one counter.  A block's home list is its index modulo 8 and thereby its XCD: items whose
// K/V meet in one L2 stay together.  Whoever finds a list empty goes on with the next, so that no XCD waits for another:
// with every compute unit streaming, the XCDs differ by up to 10 % in speed, and with the items dealt out evenly the slowest
// decides (1024 decodes and two chunks: XCDs ended between 1459 and 1632 us).  The counters are relaxed atomics: they hand out
// indices into the read-only plan.  They start at zero; the first `taken` items are the blocks' first ones.
constexpr int kNoItem = 0x7FFFFFFF;
constexpr int kOneEach = 0, kQueued = 1, kRoles = 2;  // how a launch of both kinds of tile hands them out
struct Queue {
    int32_t *counters;
    int n_items, taken, list;
    __device__ __forceinline__ int bump() const {
        return __hip_atomic_fetch_add(counters + list * kSchedStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the item at count `got` of the list, or kNoItem
    __device__ __forceinline__ int item(int got) const {
        const int i = queue_item(taken, list, got);
        return i < n_items ? i : kNoItem;
    }
    // Moves to the list that has most left; false if all are empty.  All counters are read at once: going round by
    // fetch-and-add would cost a block eight round trips to memory at its end.
    __device__ __forceinline__ bool move_on() {
        int counts[kSchedLists], most = 0;
#pragma unroll
        for (int x = 0; x < kSchedLists; ++x)
            counts[x] = __hip_atomic_load(counters + x * kSchedStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int x = 0; x < kSchedLists; ++x) {
            const int left = n_items - queue_item(taken, x, counts[x]);
            if (left > most) most = left, list = x;
        }
        return most > 0;
    }
    // the item at count `got`, or where the list is at its end one of another list, or kNoItem
    __device__ __forceinline__ int take(int got) {
        int i = item(got);
        while (i == kNoItem && move_on()) i = item(bump());
        return i;
    }
};

// The thread's index, as a value the compiler cannot follow: the per-lane offsets made from it are then formed anew for every item
// a block takes instead of being kept in registers across items (28 more registers, and 15 spilled).
__device__ __forceinline__ int thread_of_item() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

constexpr float kNegSentinel = -1.0e30f;  // finite "no key seen yet" running maximum
constexpr float kRescaleSlack = 8.0f;     // raise the softmax reference only when exceeded by 2^8
typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ bf16x8 load_bf16x8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// One direct global -> LDS load moves 16 bytes per lane (1 KiB per wavefront): lane l fetches base + byte_off(l) and the
// wavefront's data lands at LDS byte address lds_addr + 16 l.
// Written as inline assembly on purpose: the compiler's wait-count bookkeeping treats the builtin form as a flat access
// that may return out of order with LDS reads, and from then on turns every wait for an LDS operand into a full drain of
// the LDS queue (in the chunk loop one pipeline bubble per four MFMAs).  The loads issued here are waited for by hand
// (SARATHI_WAIT_VMCNT), they are the only vector-memory accesses of the key loops.
// A whole page of one KV head (N loads of 1 KiB) behind ONE write of the LDS base register: the instruction's immediate
// offset is added to the global address and to the LDS address alike, so load j uses offset 1024 j and a lane offset that
// has 1024 j taken off (rel_off[j] = byte offset inside the page minus 1024 j, which is never negative: load j fetches the
// page's j-th KiB).  STREAM: with the non-temporal hint (K/V read once, far more than the caches hold).
template <int N, bool STREAM = false>
__device__ __forceinline__ void dma_load_page(const uint16_t *base, const int (&rel_off)[N], uint32_t lds_addr) {
    static_assert(N == 2 || N == 4, "pages of 2 KiB (d = 64) or 4 KiB (d = 128) per KV head");
    if constexpr (N == 4 && !STREAM) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %5\n\t"
                     "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                     "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
                     "global_load_lds_dwordx4 %4, %5 offset:3072"
                     :
                     : "s"(lds_addr), "v"(rel_off[0]), "v"(rel_off[1]), "v"(rel_off[2]), "v"(rel_off[3]), "s"(base)
                     : "memory");
    } else if constexpr (N == 4) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %5 nt\n\t"
                     "global_load_lds_dwordx4 %2, %5 offset:1024 nt\n\t"
                     "global_load_lds_dwordx4 %3, %5 offset:2048 nt\n\t"
                     "global_load_lds_dwordx4 %4, %5 offset:3072 nt"
                     :
                     : "s"(lds_addr), "v"(rel_off[0]), "v"(rel_off[1]), "v"(rel_off[2]), "v"(rel_off[3]), "s"(base)
                     : "memory");
    } else if constexpr (!STREAM) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %3\n\t"
                     "global_load_lds_dwordx4 %2, %3 offset:1024"
                     :
                     : "s"(lds_addr), "v"(rel_off[0]), "v"(rel_off[1]), "s"(base)
                     : "memory");
    } else {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "global_load_lds_dwordx4 %1, %3 nt\n\t"
                     "global_load_lds_dwordx4 %2, %3 offset:1024 nt"
                     :
                     : "s"(lds_addr), "v"(rel_off[0]), "v"(rel_off[1]), "s"(base)
                     : "memory");
    }
}
typedef void __attribute__((address_space(3))) *lds_ptr;
__device__ __forceinline__ uint32_t lds_address(const uint16_t *p) {
    return (uint32_t)(uintptr_t)(lds_ptr)(p);
}
__device__ __forceinline__ bf16x8 lds_bf16x8(const uint16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima).
#define SARATHI_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)
// the same for the LDS (and scalar-load) counter at zero
#define SARATHI_WAIT_LDS() __builtin_amdgcn_s_waitcnt(0xC07F)

// K rows sit unpadded in LDS (a direct global->LDS load writes 1 KiB of consecutive bytes per
// wavefront); the 16-byte chunks of row r are XOR-swizzled with this key so that the 16 lanes
// of a b128 read, which walk 16 different rows at the same logical chunk, hit distinct banks.
template <int D>
__device__ __forceinline__ int k_swizzle(int r) {
    return D == 128 ? (r & 15) : ((r >> 1) & 7);
}
// LDS element offset of the 8-slot half `hh` of V^T row `d` of page `u`: the two halves of a
// row are swapped on every other group of eight channels (conflict-free reads).
template <int D>
__device__ __forceinline__ int v_lds_off(int u, int d, int hh) {
    return ((u * D + d) * 2 + (hh ^ ((d >> 3) & 1))) * 8;
}

// LDS of a wave-tile block: every wavefront has a ring of kRingTiles tiles of 32 keys of its own (K pages 0 and 1, V pages
// 0 and 1); at the end the same bytes hold its 16 columns x (D + 4) floats of unnormalised output (the pad spreads the
// columns over the banks) and 16 x (maximum, sum) for the merge.
template <int D>
struct WaveSmem {
    static constexpr int kPageElems = kPageSize * D;
    static constexpr int kTileElems = 4 * kPageElems;
    static constexpr int kRingTiles = D == 128 ? 1 : 2;
    static constexpr int kWaveElems = kRingTiles * kTileElems;
    static constexpr int kTotalElems = 4 * kWaveElems;
    static constexpr int kColStride = D + 4;
    static constexpr int kOutFloats = kWaveCols * kColStride;
    static_assert((kOutFloats + 2 * kWaveCols) * 4 <= kWaveElems * 2, "the merge data fits the wavefront's ring");
};

// What a wavefront needs to move its K/V pages from global memory to its ring.
template <int D>
struct WaveLoads {
    static constexpr int kLoads = kPageSize * D / 512;  // 1 KiB loads per page of one KV head
    const uint16_t *k_head;  // page 0 of this KV head
    const uint16_t *v_head;
    const_i32_ptr bt;      // this sequence's block-table row (scalar loads)
    int64_t page_stride;   // elements per page (all KV heads)
    int64_t last_page_id;  // num_pages - 1 (page ids are clamped: a corrupt table cannot fault)
    int32_t n_pages_seq;   // pages that hold positions < ctx_len
    uint32_t lds_addr;     // of this wavefront's ring
    int k_off[2][kLoads];  // this lane's byte offsets (see dma_load_page) for a tile's K pages 0 and 1
    int v_off[kLoads];
};

// The two block-table entries of a 32-key tile: wave-uniform, by scalar loads, which the vector-memory counter does not see.
struct TilePages {
    int32_t e0, e1;
};
template <int D>
__device__ __forceinline__ TilePages tile_pages(const WaveLoads<D> &ge, int tile) {
    // Pages at or beyond ceil(ctx_len/16) are never dereferenced: the index is clamped to the
    // sequence's last page and whatever is loaded for such keys is masked.
    return TilePages{ge.bt[min(tile * 2, ge.n_pages_seq - 1)], ge.bt[min(tile * 2 + 1, ge.n_pages_seq - 1)]};
}
template <int D>
__device__ __forceinline__ int64_t page_offset(const WaveLoads<D> &ge, int32_t entry) {
    return (entry < 0 ? 0 : (entry > ge.last_page_id ? ge.last_page_id : (int64_t)entry)) * ge.page_stride;
}
template <int D, bool STREAM>
__device__ __forceinline__ void issue_k(const WaveLoads<D> &ge, const TilePages &pages, int slot) {
    const uint32_t dst = ge.lds_addr + (uint32_t)(slot * WaveSmem<D>::kTileElems * 2);
    dma_load_page<WaveLoads<D>::kLoads, STREAM>(ge.k_head + page_offset(ge, pages.e0), ge.k_off[0], dst);
    dma_load_page<WaveLoads<D>::kLoads, STREAM>(ge.k_head + page_offset(ge, pages.e1), ge.k_off[1], dst + WaveSmem<D>::kPageElems * 2);
}
template <int D, bool STREAM>
__device__ __forceinline__ void issue_v(const WaveLoads<D> &ge, const TilePages &pages, int slot) {
    const uint32_t dst = ge.lds_addr + (uint32_t)((slot * WaveSmem<D>::kTileElems + 2 * WaveSmem<D>::kPageElems) * 2);
    dma_load_page<WaveLoads<D>::kLoads, STREAM>(ge.v_head + page_offset(ge, pages.e0), ge.v_off, dst);
    dma_load_page<WaveLoads<D>::kLoads, STREAM>(ge.v_head + page_offset(ge, pages.e1), ge.v_off, dst + WaveSmem<D>::kPageElems * 2);
}

template <int D>
struct SoftmaxState {
    f32x4 o[D / 16];  // O^T accumulators: channel 16t + 4g + i, column n
    float m;          // running maximum (base-2 scaled scores), identical in the 4 lanes of a column
    float l;          // this lane's share of the running sum (summed over g at the end)
};

// Scores of a tile from its K operands, masked, and their softmax weights as the B operand of the second contraction.
template <int D>
__device__ __forceinline__ bf16x8 tile_weights(const bf16x8 (&k)[2][D / 32], const bf16x8 (&qreg)[D / 32], SoftmaxState<D> &st,
                                               int tile, int g, int pos_eff, int min_pos_eff, int lo, int max_lo, float scale_log2) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[0][s], qreg[s], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[1][s], qreg[s], s1, 0, 0, 0);
    }
    const int key0 = tile * kTileKeys + g * 8;  // this lane's eight keys: key0 .. key0+7
    float t[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        t[j] = s0[j] * scale_log2;
        t[4 + j] = s1[j] * scale_log2;
    }
    if (tile * kTileKeys + (kTileKeys - 1) > min_pos_eff) {  // wave-uniform: some lane must mask
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (key0 + j <= pos_eff) ? t[j] : -INFINITY;
    }
    if (tile * kTileKeys < max_lo) {  // wave-uniform: some lane's sliding window starts inside or after this tile
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (key0 + j >= lo) ? t[j] : -INFINITY;
    }
    float tmax = fmaxf(fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3])), fmaxf(fmaxf(t[4], t[5]), fmaxf(t[6], t[7])));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    if (__any(tmax > st.m + kRescaleSlack)) {  // wave-uniform; rare after the first tiles
        const float m_new = fmaxf(st.m, tmax);
        const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
        st.l *= alpha;
        st.m = m_new;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) st.o[c] *= alpha;
    }
    f32x8 p;
    float psum = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        p[j] = __builtin_amdgcn_exp2f(t[j] - st.m);
        psum += p[j];
    }
    st.l += psum;
    return __builtin_convertvector(p, bf16x8);
}

// One wave-tile unit = one block.  The unit's key range is quartered (in multiples of 32 keys) among
// the block's four wavefronts, which run the same loop as independent split-KV pieces and then merge
// their (maximum, sum, unnormalised output) through LDS in wavefront order: the block writes the final
// rows, or one set of partial rows if the tile is split further across blocks.
//
// A wavefront's ring holds 16 KiB (one tile of 128 channels, two of 64): a tile's K operands are read into registers, its K
// pages' slots filled with those of the tile kRingTiles on, then the same with V, so 8 to 16 KiB of a wavefront are always
// on their way.  Two blocks to a compute unit reach the chip's rate so (6.7 TB/s; rings twice as deep are no faster: a unit
// needs 64 KiB in flight at 26 GB/s).  With 64 channels one tile instead of two is 1 to 6 % slower.
//
// claim() is called by the block's first thread while its last tiles are on their way: the next item's counter is read
// under the last loads, and not so early that a block sits on an item that another could have begun.  Returns what it returned.
template <int D, bool STREAM, typename Claim>
__device__ __forceinline__ int wave16_path(const AttnParams &p, const TileDesc &it, int split, int kvh, uint16_t *smem, Claim claim) {
    const int tid = thread_of_item();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;
    const int seq = it.seq;
    const int ctx = it.ctx_len;
    const int q_start = it.q_start;
    const int prefix = ctx - it.q_len;
    const int G = p.group;
    UnitRange ur = unit_range(it, split);
    {   // this wavefront's quarter of the unit (possibly empty: then it contributes weight zero)
        const int quarter = ((ur.key_end - ur.key_begin + 3) / 4 + kTileKeys - 1) / kTileKeys * kTileKeys;
        const int b = ur.key_begin + wave * quarter;   // a multiple of 32, as every piece start
        ur.key_end = min(ur.key_end, b + quarter);
        ur.key_begin = min(b, ur.key_end);
    }
    const bool piece_empty = ur.key_begin >= ur.key_end;

    // Lanes beyond the tile's valid columns shadow column 0 of the tile and store nothing.
    const bool col_valid = n < it.n_cols;
    const int col = it.col_begin + (col_valid ? n : 0);
    const int row = col / G;
    const int head = kvh * G + (col - row * G);
    const int pos_eff = min(prefix + row, ur.key_end - 1);                 // last key this column may see here
    const int min_pos_eff = min(prefix + it.col_begin / G, ur.key_end - 1);  // the same for the tile's first column
    // first key inside this column's sliding window, and the largest such key over the tile's columns
    const int lo = p.window > 0 ? max(0, prefix + row - p.window + 1) : 0;
    const int max_lo = p.window > 0 ? max(0, prefix + (it.col_begin + it.n_cols - 1) / G - p.window + 1) : 0;

    bf16x8 qreg[D / 32];
    {
        const uint16_t *qp = p.q + ((int64_t)(q_start + row) * p.num_q_heads + head) * D + g * 8;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) qreg[s] = load_bf16x8(qp + s * 32);
    }

    using WS = WaveSmem<D>;
    using WL = WaveLoads<D>;
    constexpr int kRing = WS::kRingTiles;
    constexpr int kPair = 2 * WL::kLoads;  // loads of a tile's K pages, and of its V pages
    uint16_t *const ring = smem + wave * WS::kWaveElems;
    WL ge;
    ge.k_head = p.k_cache + (int64_t)kvh * WS::kPageElems;
    ge.v_head = p.v_cache + (int64_t)kvh * WS::kPageElems;
    ge.bt = (const_i32_ptr)(p.block_table + (int64_t)seq * p.max_blocks);
    ge.page_stride = (int64_t)p.num_kv_heads * WS::kPageElems;
    ge.last_page_id = p.num_pages - 1;
    ge.n_pages_seq = (ctx + kPageSize - 1) / kPageSize;
    ge.lds_addr = lds_address(ring);
    // Page 1's K rows take part in the same reads as page 0's rows of the same slots: its swizzle key is moved by as many
    // chunks as four rows move it, which those reads leave out.
    constexpr int kPageKey = D == 128 ? 4 : 2;
    constexpr int kChunks = D / 8;  // 16-byte chunks of a K row
#pragma unroll
    for (int j = 0; j < WL::kLoads; ++j) {
        const int q = j * 64 + lane, slot = q / kChunks, d = q >> 1;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            ge.k_off[u][j] = slot * D * 2 + ((q % kChunks) ^ k_swizzle<D>(slot) ^ (u * kPageKey)) * 16 - j * 1024;
        ge.v_off[j] = (d * 2 + ((q & 1) ^ ((d >> 3) & 1))) * 16 - j * 1024;
    }
    // K operand: A-row n of MFMA b is page n/8, slot ((n/4)&1)*8 + 4b + n%4; contraction step s: chunk 4s + g of that row
    int k_rd[2][D / 32];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int s = 0; s < D / 32; ++s) {
            const int slot = ((n >> 2) & 1) * 8 + 4 * b + (n & 3);
            k_rd[b][s] = (n >> 3) * WS::kPageElems + slot * D + ((4 * s + g) ^ k_swizzle<D>(slot) ^ ((n >> 3) * kPageKey)) * 8;
        }
    // V operand of output tile c: A-row n is channel 16c + n, contraction indices 8g .. are slots 8*(g&1) .. of page g/2
    const int v_rd = 2 * WS::kPageElems + v_lds_off<D>(g >> 1, n, g & 1);

    SoftmaxState<D> st;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) st.o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.m = kNegSentinel;
    st.l = 0.f;

    const int tile_begin = ur.key_begin / kTileKeys;
    const int tile_end = piece_empty ? tile_begin : (ur.key_end + kTileKeys - 1) / kTileKeys;

    TilePages pages = tile_pages(ge, tile_begin);
    SARATHI_WAIT_VMCNT(0);  // the queries, so that from here on the counter counts the direct loads only
#pragma unroll
    for (int i = 0; i < kRing; ++i)
        if (tile_begin + i < tile_end) {
            issue_k<D, STREAM>(ge, pages, i);
            issue_v<D, STREAM>(ge, pages, i);
            pages = tile_pages(ge, tile_begin + i + 1);
        }
    // One tile.  `left`: tiles still in the ring or, if `more`, all of it: how many loads are younger than the tile's.
    auto step = [&](int tile, int slot, auto left, auto more) {
        constexpr int kYounger = 2 * decltype(left)::value - 1;
        constexpr bool kMore = decltype(more)::value;
        const uint16_t *t_lds = ring + slot * WS::kTileElems;
        SARATHI_WAIT_VMCNT(kYounger * kPair);
        asm volatile("" ::: "memory");
        bf16x8 k[2][D / 32];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int s = 0; s < D / 32; ++s) k[b][s] = lds_bf16x8(t_lds + k_rd[b][s]);
        SARATHI_WAIT_LDS();  // the operands are in registers: their slots may be filled again
        asm volatile("" ::: "memory");
        if (kMore) issue_k<D, STREAM>(ge, pages, slot);
        const bf16x8 pT = tile_weights<D>(k, qreg, st, tile, g, pos_eff, min_pos_eff, lo, max_lo, p.scale_log2);
        SARATHI_WAIT_VMCNT((kMore ? kYounger : kYounger - 1) * kPair);
        asm volatile("" ::: "memory");
        bf16x8 v[D / 16];
#pragma unroll
        for (int c = 0; c < D / 16; ++c) v[c] = lds_bf16x8(t_lds + v_rd + c * 16 * kPageSize);
        SARATHI_WAIT_LDS();
        asm volatile("" ::: "memory");
        if (kMore) {
            issue_v<D, STREAM>(ge, pages, slot);
            pages = tile_pages(ge, tile + kRing + 1);
        }
        if (tile * kTileKeys + kTileKeys > ctx) {  // wave-uniform: tile holds slots at or beyond ctx_len
            u32x4 keep;
            const int key0 = tile * kTileKeys + g * 8;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                keep[w] = ((key0 + 2 * w < ctx) ? 0x0000FFFFu : 0u) | ((key0 + 2 * w + 1 < ctx) ? 0xFFFF0000u : 0u);
#pragma unroll
            for (int c = 0; c < D / 16; ++c) v[c] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, v[c]) & keep);
        }
#pragma unroll
        for (int c = 0; c < D / 16; ++c) st.o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[c], pT, st.o[c], 0, 0, 0);
    };
    int tile = tile_begin, slot = 0;
    for (; tile + kRing + 1 < tile_end; ++tile) {
        step(tile, slot, std::integral_constant<int, kRing>{}, std::true_type{});
        slot = slot + 1 == kRing ? 0 : slot + 1;
    }
    int claimed = 0;
    if (tid == 0) claimed = claim();  // in front of the last tile's loads: results come back in order
    if (tile + kRing < tile_end) {
        step(tile, slot, std::integral_constant<int, kRing>{}, std::true_type{});
        ++tile;
        slot = slot + 1 == kRing ? 0 : slot + 1;
    }
    if (kRing == 2 && tile + 1 < tile_end) {
        step(tile, slot, std::integral_constant<int, 2>{}, std::false_type{});
        ++tile;
        slot ^= 1;
    }
    if (tile < tile_end) step(tile, slot, std::integral_constant<int, 1>{}, std::false_type{});

    float l = st.l + __shfl_xor(st.l, 16);
    l += __shfl_xor(l, 32);

    // Publish this wavefront's piece where its ring was: lane (n, g) holds channels 16c + 4g + i of column n.
    {
        float *o_w = reinterpret_cast<float *>(ring) + n * WS::kColStride + g * 4;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) *reinterpret_cast<f32x4 *>(o_w + c * 16) = st.o[c];
        if (g == 0) {
            float *ml = reinterpret_cast<float *>(ring) + WS::kOutFloats + n * 2;
            ml[0] = st.m;
            ml[1] = l;
        }
    }
    __syncthreads();
    // Merge: thread t owns column t / 16 and D / 16 consecutive channels of it.
    constexpr int CH = D / 16;
    const int mc = tid >> 4;
    const int ch0 = (tid & 15) * CH;
    if (mc >= it.n_cols) return claimed;
    float m_w[4], m_max = kNegSentinel;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        m_w[w] = reinterpret_cast<const float *>(smem + w * WS::kWaveElems)[WS::kOutFloats + mc * 2];
        m_max = fmaxf(m_max, m_w[w]);
    }
    float acc[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) acc[j] = 0.f;
    float l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float wt = __builtin_amdgcn_exp2f(m_w[w] - m_max);
        const float *merge = reinterpret_cast<const float *>(smem + w * WS::kWaveElems);
        l_tot += wt * merge[WS::kOutFloats + mc * 2 + 1];
        const float *o_w = merge + mc * WS::kColStride + ch0;
#pragma unroll
        for (int j = 0; j < CH; j += 4) {
            const f32x4 o4 = *reinterpret_cast<const f32x4 *>(o_w + j);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[j + i] += wt * o4[i];
        }
    }
    const int mcol = it.col_begin + mc;
    const int mrow = mcol / G;
    const int mhead = kvh * G + (mcol - mrow * G);
    const UnitRange whole = unit_range(it, split);
    if (whole.part_row < 0) {
        const float inv = 1.0f / l_tot;
        uint16_t *op = p.out + ((int64_t)(q_start + mrow) * p.num_q_heads + mhead) * D + ch0;
#pragma unroll
        for (int j = 0; j < CH; j += 4) {
            const f32x4 o = {acc[j] * inv, acc[j + 1] * inv, acc[j + 2] * inv, acc[j + 3] * inv};
            *reinterpret_cast<u32x2 *>(op + j) = __builtin_bit_cast(u32x2, __builtin_convertvector(o, bf16x4));
        }
        return claimed;
    }
    // Tile split across blocks: this block's (reference maximum, sum, unnormalised output).
    const int64_t prow = ((int64_t)(whole.part_row + mc) * p.num_kv_heads + kvh);
    float *po = p.part_o + prow * D + ch0;
#pragma unroll
    for (int j = 0; j < CH; j += 4) *reinterpret_cast<f32x4 *>(po + j) = f32x4{acc[j], acc[j + 1], acc[j + 2], acc[j + 3]};
    if ((tid & 15) == 0) {
        p.part_ml[prow * 2 + 0] = m_max;
        p.part_ml[prow * 2 + 1] = l_tot;
    }
    return claimed;
}

// ---------------------------------------------------------------------------------------
// Chunk-tile path: 4 waves x 32 columns, K/V tiles of 32 keys staged in LDS.
// ---------------------------------------------------------------------------------------
// LDS of the chunk-tile path: a ring of 4 K tiles and a ring of 4 V tiles (32 keys each).
// In the step that handles tile t the wave reads K(t+1) and V(t-1) while K(t+2), K(t+3), V(t+1)
// and V(t+2) are in flight from global memory straight into LDS (no staging registers).  Tile
// with index rel (relative to the unit's first tile) lives in slot rel % 4 of its ring.
constexpr int kRing = 4;

template <int D>
struct ChunkSmem {
    static constexpr int kTileElems = kTileKeys * D;  // one K tile or one V tile: 32 keys x D channels
    static constexpr int kVBase = kRing * kTileElems;
    static constexpr int kTotalElems = 2 * kRing * kTileElems;
};


constexpr int kCarry = 3;  // output-MFMA operands read one step ahead

// State a wave carries from one tile to the next in the software-pipelined chunk loop.
template <int D>
struct ChunkState {
    f32x16 oacc[D / 32];  // O^T accumulators: channel 32c + 8*(r/4) + 4h + r%4, column n
    // Two register sets used in turn by consecutive steps of the unrolled loop (a step reads one
    // and fills the other); steps outside that loop keep everything in set 0.
    f32x16 s[2];          // raw scores of the tile whose softmax is due (already masked)
    bf16x8 p[2][2];       // bf16 softmax weights of the previous tile (B operands of its output MFMAs)
    bf16x8 carry[kCarry]; // V operands of the next step's first output MFMAs, read at the end of this step
    float tmax;           // scaled maximum of the due scores over the column
    float m_ref;          // softmax reference, scaled base-2 units
    float l_run;          // this lane's share of the running sum
};

// One pipelined step.  Independent work of three tiles shares one basic block so that the
// matrix pipe and the vector ALU run side by side inside a single wavefront:
//   MFMA:  S^T(t+1) = K(t+1) Q^T    (HAS_NEXT)        O^T += V^T(t-1) P^T(t-1)      (HAS_PREV)
//   VALU:  P(t) = 2^(S(t)*scale - m_ref), row sums, bf16 packing; mask and maximum of S(t+1)
// k_chunk: this lane's (swizzled) K chunk offsets; K_OFF / V_OFF: element offsets of the ring
// slots read in this step (wave-uniform).
// Order of the MFMAs of a step: which kind slot i issues and its index within that kind.  A step
// with both kinds opens with three output MFMAs (their V operands were read at the end of the
// previous step, so the matrix pipe has work right after the barrier, before any read of this step
// returns), then all score MFMAs (one accumulator; the scores are complete a few slots before the
// end of the step, so that masking and the maximum of the next tile also run under MFMAs), then the
// remaining output MFMAs.
struct ChunkSlot {
    bool is_score;
    int sub;
};
constexpr ChunkSlot chunk_slot(int i, int n_s, int n_o) {
    const int lead = n_o < kCarry ? n_o : kCarry;
    if (i < lead) return ChunkSlot{false, i};
    if (i < lead + n_s) return ChunkSlot{true, i - lead};
    return ChunkSlot{false, i - n_s};
}
constexpr int chunk_last_score_slot(int n_s, int n_o) {
    return n_s == 0 ? -1 : (n_o < kCarry ? n_o : kCarry) + n_s - 1;
}

// PHASE >= 0: the tile's index inside the unit is PHASE modulo 4, which fixes the ring slots at
// compile time (K_OFF_RT / V_OFF_RT are ignored and the operand reads need no address
// arithmetic); PHASE < 0: slots given at run time.  The step reads register set PP and fills set
// PP ^ 1 (SWAP) or set PP again (the results are copied back).
// CARRY_IN: the operands of the first kCarry output MFMAs are in st.carry (read by the previous step);
// CARRY_OUT: this step reads them for the next step (whose previous tile, this step's current one,
// has been in LDS and visible since this step's barrier).
template <int D, bool HAS_PREV, bool HAS_NEXT, bool MASK_NEXT, bool CARRY_IN, bool CARRY_OUT, int PHASE = -1, int PP = 0,
          bool SWAP = false>
__device__ __forceinline__ void chunk_step(ChunkState<D> &st, const bf16x8 (&qreg)[D / 16], const uint16_t *smem,
                                           const int (&k_chunk)[D / 16], int v_rd, int K_OFF_RT, int V_OFF_RT, float scale,
                                           int next_key0, int pos_eff, int lo) {
    constexpr int TE_ = kTileKeys * D;
    static_assert(!CARRY_IN || HAS_PREV, "carried operands belong to output MFMAs");
    const int K_OFF = PHASE >= 0 ? ((PHASE + 1) & (kRing - 1)) * TE_ : K_OFF_RT;
    const int V_OFF = PHASE >= 0 ? ((PHASE + 3) & (kRing - 1)) * TE_ : V_OFF_RT;
    const int V_OFF_NEXT = (V_OFF + TE_) & (kRing * TE_ - 1);  // ring slot of the current tile
    constexpr int OUT = SWAP ? (PP ^ 1) : PP;
    constexpr int NS = D / 16;
    constexpr int NB = D / 32;
    constexpr int N_S = HAS_NEXT ? NS : 0;              // score MFMAs (one dependent chain through s_next)
    constexpr int N_O = HAS_PREV ? 2 * NB : 0;          // output MFMAs (NB accumulators, two pages each)
    constexpr int NM = N_S + N_O;
    constexpr int AHEAD = 3;                             // operand reads run this many MFMAs ahead
    auto is_score = [&](int i) { return chunk_slot(i, N_S, N_O).is_score; };
    auto sub_index = [&](int i) { return chunk_slot(i, N_S, N_O).sub; };

    // The step is laid out as NM slots fenced by scheduling barriers.  Slot i issues the LDS
    // read for MFMA i+AHEAD, then MFMA i, then its share of the vector-ALU work, which
    // executes while the matrix pipe is busy with MFMA i.
    auto operand = [&](int i) -> const uint16_t * {
        const int j = sub_index(i);
        if (is_score(i)) return smem + K_OFF + k_chunk[j < NS ? j : 0];
        // output MFMA j: page j / NB, channel block j % NB
        return smem + v_rd + (V_OFF + ((j / NB) * D + (j % NB) * 32) * 16);
    };
    static_assert(AHEAD == kCarry, "the operands carried between steps fill the read-ahead window");
    bf16x8 frag[AHEAD + 1];
    bf16x8 nxt[kCarry];
#pragma unroll
    for (int i = 0; i < AHEAD && i < NM; ++i) frag[i] = CARRY_IN ? st.carry[i] : lds_bf16x8(operand(i));

    f32x16 s_tmp;
    f32x16 &s_next = SWAP ? st.s[OUT] : s_tmp;
    const f32x16 &s_cur = st.s[PP];
    const bf16x8 p_old0 = st.p[PP][0], p_old1 = st.p[PP][1];

    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    uint32_t p_new[8];  // bf16 pairs of the current tile's weights: registers (2k, 2k+1)
    float e_even = 0.f;
    float psum = 0.f;
    float smax = -INFINITY;
    float neg_m = -st.m_ref;
    auto weight = [&](int r) {
        const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[r], scale, neg_m));
        psum += e;
        if (r & 1) {
            const bf16x2 pk = __builtin_convertvector(f32x2{e_even, e}, bf16x2);
            p_new[r >> 1] = __builtin_bit_cast(uint32_t, pk);
        } else {
            e_even = e;
        }
    };
    // mask + running maximum of register r of the next tile (key next_key0 + 16*(r/8) + r%8)
    auto next_max = [&](int r) {
        if (MASK_NEXT) {  // causal bound and, under a sliding window, the column's first visible key
            const int key = next_key0 + (r >> 3) * 16 + (r & 7);
            s_next[r] = (key <= pos_eff && key >= lo) ? s_next[r] : -INFINITY;
        }
        smax = fmaxf(smax, s_next[r]);
    };
    constexpr int LAST_SCORE = chunk_last_score_slot(N_S, N_O);  // slot of the last score MFMA
    constexpr int MAX_FROM = LAST_SCORE + 2;  // first slot in which the finished scores may be touched
    int w_done = 0, m_done = 0;         // compile-time after unrolling
    // Slot boundaries.  The arithmetic below has no side effects, so nothing but data flow
    // would keep it inside its slot; an empty asm that "touches" the values a slot produced and
    // one input of the next slot's arithmetic (the negated reference) pins both, and the
    // scheduling barrier keeps the machine scheduler from undoing the layout.  Neither emits
    // an instruction.
    asm volatile("" : "+v"(neg_m), "+v"(psum));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        bf16x8 &ahead = frag[(i + AHEAD) % (AHEAD + 1)];
        if (i + AHEAD < NM) ahead = lds_bf16x8(operand(i + AHEAD));
        else if (CARRY_OUT)  // operand j = i + AHEAD - NM of the next step: page j / NB, channel block j % NB of the current tile
            nxt[i + AHEAD - NM] = lds_bf16x8(smem + v_rd + (V_OFF_NEXT + (((i + AHEAD - NM) / NB) * D + ((i + AHEAD - NM) % NB) * 32) * 16));
        const bf16x8 a = frag[i % (AHEAD + 1)];
        const int j = sub_index(i);
        if (is_score(i)) {
            if (j == 0) {
                f32x16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[0], zero, 0, 0, 0);
            } else {
                s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[j < NS ? j : 0], s_next, 0, 0, 0);
            }
        } else {
            st.oacc[j % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, (j / NB) ? p_old1 : p_old0, st.oacc[j % NB], 0, 0, 0);
        }
        // vector-ALU share of this slot
        const int w_from = w_done;
        const int w_target = 16 * (i + 1) / (NM > 0 ? NM : 1);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (r >= w_from && r < w_target) weight(r);
        w_done = w_target;
        if (HAS_NEXT && i >= MAX_FROM) {
            const int m_target = 16 * (i + 1 - MAX_FROM) / (NM > MAX_FROM ? NM - MAX_FROM : 1);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (r >= m_done && r < m_target) next_max(r);
            m_done = m_target;
        }
        // pin: this slot's MFMA result and the weights made here.  The operand fetched ahead in
        // this slot is NOT pinned (that would make the slot wait for it); the scheduling barrier
        // alone keeps the read where it was issued.
        bf16x8 &older = frag[i % (AHEAD + 1)];
        if (is_score(i))
            asm volatile("" : "+v"(s_next), "+v"(older), "+v"(neg_m), "+v"(psum), "+v"(e_even));
        else if (i > LAST_SCORE)
            asm volatile("" : "+v"(st.oacc[j % NB]), "+v"(older), "+v"(neg_m), "+v"(psum), "+v"(e_even), "+v"(s_next), "+v"(smax));
        else
            asm volatile("" : "+v"(st.oacc[j % NB]), "+v"(older), "+v"(neg_m), "+v"(psum), "+v"(e_even));
#pragma unroll
        for (int r = 1; r < 16; r += 2)
            if (r >= w_from && r < w_target) asm volatile("" : "+v"(p_new[r >> 1]));
        __builtin_amdgcn_sched_barrier(0);
    }
    // whatever did not fit into the slots (steps without MFMAs, or too few of them)
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (r >= w_done) weight(r);
    if (HAS_NEXT) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (r >= m_done) next_max(r);
        // the other half-wave holds the other 16 keys of the column: one VALU half-swap, no LDS trip
        const auto halves = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, smax),
                                                             __builtin_bit_cast(uint32_t, smax), false, false);
        smax = fmaxf(__builtin_bit_cast(float, (uint32_t)halves[0]), __builtin_bit_cast(float, (uint32_t)halves[1]));
        st.tmax = smax * scale;  // scale > 0
        if (!SWAP) st.s[OUT] = s_tmp;
    }
    st.l_run += psum;
    if (CARRY_OUT) {
        static_assert(!CARRY_OUT || NM >= kCarry, "a step that reads ahead for the next one has at least kCarry slots");
#pragma unroll
        for (int j = 0; j < kCarry; ++j) st.carry[j] = nxt[j];
    }
    typedef __attribute__((ext_vector_type(4))) uint32_t pk4;
    st.p[OUT][0] = __builtin_bit_cast(bf16x8, pk4{p_new[0], p_new[1], p_new[2], p_new[3]});
    st.p[OUT][1] = __builtin_bit_cast(bf16x8, pk4{p_new[4], p_new[5], p_new[6], p_new[7]});
}

template <int D>
__device__ __forceinline__ void chunk_tile_path(const AttnParams &p, const TileDesc &it, int split, int kvh,
                                                uint16_t *smem) {
    constexpr int NS = D / 16;            // contraction steps of the score MFMAs
    constexpr int NB = D / 32;            // 32-channel blocks of the output
    constexpr int CPR = D / 8;            // 16-byte chunks per K row
    constexpr int PAGE_ELEMS = kPageSize * D;
    constexpr int LOADS_PER_PAGE = PAGE_ELEMS / 512;  // 1 KiB wavefront loads per page of one KV head
    using SM = ChunkSmem<D>;
    constexpr int TE = SM::kTileElems;
    const int tid = thread_of_item();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction; tell the compiler
    const int n = lane & 31;
    const int h = lane >> 5;
    const int seq = it.seq;
    const int ctx = it.ctx_len;
    const int q_start = it.q_start;
    const int prefix = ctx - it.q_len;
    const int G = p.group;
    const UnitRange ur = unit_range(it, split);

    // Columns of this wave; lanes (and whole waves) without a valid column shadow the tile's first column.
    const int wcol = wave * 32 + n;
    const bool col_valid = wcol < it.n_cols;
    const int col = it.col_begin + (col_valid ? wcol : 0);
    const int row = col / G;
    const int head = kvh * G + (col - row * G);
    const int pos_eff = min(prefix + row, ur.key_end - 1);
    const int wave_first_col = it.col_begin + ((wave * 32 < it.n_cols) ? wave * 32 : 0);
    const int min_pos_eff = min(prefix + wave_first_col / G, ur.key_end - 1);  // wave-uniform
    // Sliding window: first key this column sees, and the largest such key over the wave's valid
    // columns (wave-uniform; a wave without valid columns shadows the tile's first column).
    const int wave_last_col = it.col_begin + ((wave * 32 < it.n_cols) ? min(wave * 32 + 31, it.n_cols - 1) : 0);
    const int lo = p.window > 0 ? max(0, prefix + row - p.window + 1) : 0;
    const int max_lo = p.window > 0 ? max(0, prefix + wave_last_col / G - p.window + 1) : 0;

    bf16x8 qreg[NS];  // B operand of the score MFMAs: column n, channels 16s + 8h ..
    {
        const uint16_t *qp = p.q + ((int64_t)(q_start + row) * p.num_q_heads + head) * D + h * 8;
#pragma unroll
        for (int s = 0; s < NS; ++s) qreg[s] = load_bf16x8(qp + s * 16);
    }

    // Global -> LDS traffic of a tile: wave 0/1 move K page 0/1, wave 2/3 move V page 0/1, each
    // as LOADS_PER_PAGE direct loads of 1 KiB.  Lane l of load j fills physical 16-byte chunk
    // q = 64j + l of the page's LDS image and therefore fetches the logical chunk that lives there.
    // K pages run three tiles ahead of the step, V pages two (V is consumed two steps later than K).
    const bool moves_v = wave >= 2;
    const int my_page = wave & 1;
    int g_off[LOADS_PER_PAGE];  // this lane's byte offset inside the page of one KV head, per load, minus 1024 j
#pragma unroll
    for (int j = 0; j < LOADS_PER_PAGE; ++j) {
        const int q = j * 64 + lane;
        const int k_slot = q / CPR;
        const int k_elem = k_slot * D + ((q % CPR) ^ k_swizzle<D>(k_slot)) * 8;
        const int v_d = q >> 1;
        const int v_elem = (v_d * 2 + ((q & 1) ^ ((v_d >> 3) & 1))) * 8;
        g_off[j] = (moves_v ? v_elem : k_elem) * 2 - j * 1024;  // relative to the load's own KiB (see dma_load_page)
    }
    const const_i32_ptr bt = (const_i32_ptr)(p.block_table + (int64_t)seq * p.max_blocks);  // read-only: scalar loads
    const int n_pages_seq = (ctx + kPageSize - 1) / kPageSize;
    const int64_t page_stride = (int64_t)p.num_kv_heads * kPageSize * D;
    const uint16_t *cache_head = (moves_v ? p.v_cache : p.k_cache) + (int64_t)kvh * PAGE_ELEMS;
    const int64_t last_page_id = p.num_pages - 1;
    const int tile_begin = ur.key_begin / kTileKeys;
    const int tile_end = (ur.key_end + kTileKeys - 1) / kTileKeys;
    const int n_tiles = tile_end - tile_begin;
    const int my_lds_base = (moves_v ? SM::kVBase : 0) + my_page * PAGE_ELEMS;
    const uint32_t smem_addr = lds_address(smem);
    // page id of this wave's page of tile `tile` (a scalar load: issue it a step before it is needed)
    // The raw table entry and its clamp are separate so that the entry can be fetched a step
    // before it is needed and only then looked at (the clamp would otherwise wait for the load).
    auto page_raw = [&](int tile) -> int32_t { return bt[min(tile * 2 + my_page, n_pages_seq - 1)]; };
    auto page_clamp = [&](int32_t raw) -> int64_t {
        const int64_t pg = raw;
        return pg < 0 ? 0 : (pg > last_page_id ? last_page_id : pg);
    };
    auto page_of = [&](int tile) -> int64_t { return page_clamp(page_raw(tile)); };
    // this wave's page `pg` of tile `tile` -> ring slot (tile - tile_begin) % 4
    auto issue_page = [&](int tile, int64_t pg) {
        const uint16_t *src = cache_head + pg * page_stride;
        const uint32_t dst = smem_addr + (uint32_t)(my_lds_base + ((tile - tile_begin) & (kRing - 1)) * TE) * 2;
        dma_load_page<LOADS_PER_PAGE>(src, g_off, dst);
    };
    auto issue_tile = [&](int tile) { issue_page(tile, page_of(tile)); };
    const int my_ahead = moves_v ? 2 : 3;  // tiles this wave's loads run ahead of the step

    ChunkState<D> st;
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.oacc[c][r] = 0.f;
    st.m_ref = kNegSentinel;
    st.l_run = 0.f;
    st.tmax = kNegSentinel;

    // MFMA row n of the score tile is key  16u + 8h' + 4a + b  for n = 16u + 8a + 4h' + b.
    const int k_row = (n & 16) | ((n & 4) << 1) | ((n & 8) >> 1) | (n & 3);
    int k_chunk[NS];  // element offset of contraction step s inside this lane's K row (swizzled)
#pragma unroll
    for (int s = 0; s < NS; ++s) k_chunk[s] = k_row * D + ((s * 2 + h) ^ k_swizzle<D>(k_row)) * 8;
    const int v_rd = SM::kVBase + v_lds_off<D>(0, n, h);  // + slot*TE + (u*D + 32c)*16 elements
    const float scale = p.scale_log2;
    // first tile of the range in which some column of this wave needs masking (wave-uniform)
    const int mask_from = max(tile_begin, min(tile_end, (min_pos_eff + 1) / kTileKeys));
    // tiles below this index hold keys in front of some column's sliding window (wave-uniform; = tile_begin without one)
    const int mask_until = max(tile_begin, min(tile_end, (max_lo + kTileKeys - 1) / kTileKeys));

    // Prologue: the first tiles start loading; when they have landed the scores of tile 0 are
    // formed (as the "next" tile of an otherwise empty step).
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (i < my_ahead && i < n_tiles) issue_tile(tile_begin + i);
    SARATHI_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    {
#pragma unroll
        for (int r = 0; r < 16; ++r) st.s[0][r] = -INFINITY;  // "current" tile of the empty step: weights 0
        st.p[0][0] = st.p[0][1] = bf16x8{};
        const int key0 = tile_begin * kTileKeys + h * 8;
        if (tile_begin >= mask_from || tile_begin < mask_until)
            chunk_step<D, false, true, true, false, false>(st, qreg, smem, k_chunk, v_rd, 0, 0, scale, key0, pos_eff, lo);
        else
            chunk_step<D, false, true, false, false, false>(st, qreg, smem, k_chunk, v_rd, 0, 0, scale, key0, pos_eff, lo);
        st.l_run = 0.f;  // the empty step contributed exp2(-inf) = 0 terms only
    }

    int32_t pg_next = page_raw(tile_begin + my_ahead);  // table entry of the page the first step will fetch
    // Common head of a step for tile t, then the step proper.  Every loop below instantiates one
    // variant only, so its body stays a single basic block (plus the rare reference raise).
    // Every step but a unit's last fetches this wave's page of tile t + my_ahead; beyond the
    // unit's end that is a clamped, unused page landing in a free ring slot, which keeps the loop
    // body and the load counter the same for all steps.
    // pg_this: table entry of the page this step fetches; fetch_next: the step itself fetches the
    // entry of the step after it (single steps), or the caller brings entries in batches (the unrolled
    // group: while a scalar load is in flight every wait for an LDS read must wait for all of them,
    // so one batch per four steps costs a quarter of what one load per step did).
    auto step = [&](int tile, auto has_prev, auto has_next, auto mask_next, auto with_dma, auto phase, auto pp,
                    int32_t pg_this, auto fetch_next) {
        // Tile t+1 must have landed (only this wave's loads of one later tile may still be in
        // flight), and every wave must be done with the slots about to be overwritten (K of
        // tile t-1, V of tile t-2).
        if (decltype(with_dma)::value) SARATHI_WAIT_VMCNT(LOADS_PER_PAGE); else SARATHI_WAIT_VMCNT(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int rel = tile - tile_begin;
        if (decltype(with_dma)::value) {
            issue_page(tile + my_ahead, page_clamp(pg_this));
            if (decltype(fetch_next)::value) pg_next = page_raw(tile + my_ahead + 1);  // looked at in the next step only
        }
        // Raise the softmax reference of the columns whose due tile exceeds it by more than the slack
        // (rare).  Three things carry the old reference: the output accumulators (tiles up to t-2), the
        // running sum (up to t-1) and the bf16 weights of tile t-1, which still wait for their output
        // MFMAs in this step; all three are brought to the new one.  Columns that keep their
        // reference get alpha = 1 (both half-waves of a column see the same tmax and m_ref).
        if (__any(st.tmax > st.m_ref + kRescaleSlack)) {
            const float m_new = (st.tmax > st.m_ref + kRescaleSlack) ? st.tmax : st.m_ref;
            const float alpha = __builtin_amdgcn_exp2f(st.m_ref - m_new);
            st.l_run *= alpha;
            st.m_ref = m_new;
#pragma unroll
            for (int c = 0; c < NB; ++c) st.oacc[c] *= alpha;
            constexpr int kSet = decltype(pp)::value;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                st.p[kSet][u] = __builtin_convertvector(__builtin_convertvector(st.p[kSet][u], f32x8) * alpha, bf16x8);
        }
        const int next_key0 = (tile + 1) * kTileKeys + h * 8;
        constexpr int kPhase = decltype(phase)::value;
        // every step with a predecessor finds its first V operands carried over; every step with a successor reads them
        chunk_step<D, decltype(has_prev)::value, decltype(has_next)::value, decltype(mask_next)::value,
                   decltype(has_prev)::value, decltype(has_next)::value, kPhase, decltype(pp)::value, (kPhase >= 0)>(
            st, qreg, smem, k_chunk, v_rd, ((rel + 1) & (kRing - 1)) * TE, ((rel + 3) & (kRing - 1)) * TE, scale, next_key0,
            pos_eff, lo);
    };
    using T = std::true_type;
    using F = std::false_type;
    using DYN = std::integral_constant<int, -1>;  // ring slots taken from the tile index at run time
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    using P3 = std::integral_constant<int, 3>;
    if (n_tiles == 1) {
        step(tile_begin, F{}, F{}, F{}, F{}, DYN{}, P0{}, pg_next, F{});
    } else {
        // first tile: nothing to accumulate yet
        if (tile_begin + 1 >= mask_from || tile_begin + 1 < mask_until) step(tile_begin, F{}, T{}, T{}, T{}, DYN{}, P0{}, pg_next, T{});
        else step(tile_begin, F{}, T{}, F{}, T{}, DYN{}, P0{}, pg_next, T{});
        // steady state, unmasked tiles: groups of four steps with the ring slots and the register
        // sets compiled in (the group starts at tile index 1 modulo 4 and leaves the state in set 0),
        // then single steps up to the causal diagonal
        int tile = tile_begin + 1;
        // tiles in front of a sliding window's start (none without a window), then single steps up to the
        // tile index the unrolled group expects
        for (; tile + 1 < tile_end && tile + 1 < mask_until; ++tile) step(tile, T{}, T{}, T{}, T{}, DYN{}, P0{}, pg_next, T{});
        for (; tile + 1 < tile_end && tile + 1 < mask_from && ((tile - tile_begin) & 3) != 1; ++tile)
            step(tile, T{}, T{}, F{}, T{}, DYN{}, P0{}, pg_next, T{});
        if (tile + 4 < tile_end && tile + 4 < mask_from) {
            // table entries of the pages the group's steps fetch; the next group's come in one batch
            int32_t e0 = pg_next, e1 = page_raw(tile + my_ahead + 1), e2 = page_raw(tile + my_ahead + 2),
                    e3 = page_raw(tile + my_ahead + 3);
            for (; tile + 4 < tile_end && tile + 4 < mask_from; tile += 4) {
                const int32_t n0 = page_raw(tile + my_ahead + 4), n1 = page_raw(tile + my_ahead + 5),
                              n2 = page_raw(tile + my_ahead + 6), n3 = page_raw(tile + my_ahead + 7);
                step(tile, T{}, T{}, F{}, T{}, P1{}, P0{}, e0, F{});
                step(tile + 1, T{}, T{}, F{}, T{}, P2{}, P1{}, e1, F{});
                step(tile + 2, T{}, T{}, F{}, T{}, P3{}, P0{}, e2, F{});
                step(tile + 3, T{}, T{}, F{}, T{}, P0{}, P1{}, e3, F{});
                e0 = n0, e1 = n1, e2 = n2, e3 = n3;
            }
            pg_next = e0;
        }
        for (; tile + 1 < tile_end && tile + 1 < mask_from; ++tile) step(tile, T{}, T{}, F{}, T{}, DYN{}, P0{}, pg_next, T{});
        // the tiles on the causal diagonal
        for (; tile + 1 < tile_end; ++tile) step(tile, T{}, T{}, T{}, T{}, DYN{}, P0{}, pg_next, T{});
        // last tile: no further scores to form, nothing more to fetch (and no load left in flight after it)
        step(tile_end - 1, T{}, F{}, F{}, F{}, DYN{}, P0{}, pg_next, F{});
    }
    // Epilogue: the output MFMAs of the last tile.  Only here can a tile hold slots at or beyond
    // ctx_len (a unit never extends past the sequence), whose V bits must be zeroed: stale cache
    // contents times a zero weight would still poison the accumulator if they were NaN or Inf.
    {
        const int last = tile_end - 1;
        const uint16_t *v_last = smem + v_rd + ((last - tile_begin) & (kRing - 1)) * TE;
        const bool tail = last * kTileKeys + kTileKeys > ctx;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                u32x4 v = *reinterpret_cast<const u32x4 *>(v_last + (u * D + c * 32) * 16);
                if (tail) {
                    const int key0 = last * kTileKeys + u * kPageSize + h * 8;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        v[w] &= ((key0 + 2 * w < ctx) ? 0x0000FFFFu : 0u) | ((key0 + 2 * w + 1 < ctx) ? 0xFFFF0000u : 0u);
                }
                st.oacc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), st.p[0][u],
                                                                      st.oacc[c], 0, 0, 0);
            }
        }
    }
    f32x16 (&oacc)[NB] = st.oacc;
    const float l_run = st.l_run;
    const float m_ref = st.m_ref;

    const float l = l_run + __shfl_xor(l_run, 32);
    // accumulator register r of block c: channel 32c + 8*(r/4) + 4h + r%4
    uint16_t *op = p.out + ((int64_t)(q_start + row) * p.num_q_heads + head) * D + h * 4;
    if (ur.part_row < 0) {
        if (!col_valid) return;
        const float inv = 1.0f / l;
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 o = {oacc[c][q4 * 4 + 0], oacc[c][q4 * 4 + 1], oacc[c][q4 * 4 + 2], oacc[c][q4 * 4 + 3]};
                const bf16x4 o4 = __builtin_convertvector(o * inv, bf16x4);
                *reinterpret_cast<u32x2 *>(op + c * 32 + q4 * 8) = __builtin_bit_cast(u32x2, o4);
            }
        return;
    }
    // Split tile: publish this piece's (reference maximum, sum, unnormalised output).
    if (col_valid) {
        const int64_t prow = ((int64_t)(ur.part_row + wcol) * p.num_kv_heads + kvh);
        float *po = p.part_o + prow * D + h * 4;
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 o = {oacc[c][q4 * 4 + 0], oacc[c][q4 * 4 + 1], oacc[c][q4 * 4 + 2], oacc[c][q4 * 4 + 3]};
                *reinterpret_cast<f32x4 *>(po + c * 32 + q4 * 8) = o;
            }
        if (h == 0) {
            p.part_ml[prow * 2 + 0] = m_ref;
            p.part_ml[prow * 2 + 1] = l;
        }
    }
}

// Item `item` of the wave tiles.  An item's KV head is rotated by its sequence: with 8 heads item % 8 is also the XCD, the
// pages of one head lie 8 x 4 KiB apart, and an XCD that runs the same head of every sequence reads addresses of one residue
// only.  (1024 decodes + 2 chunks 1677 -> 1662 us, the long-context hybrid batch 978 -> 974, 256 decodes 224.7 -> 224.3.)  The
// column tiles of one sequence keep sharing an XCD, and chunk tiles, whose tiles share K/V in its L2, are not rotated.
template <int D, bool STREAM, typename Claim>
__device__ __forceinline__ int wave_item(const AttnParams &p, int item, uint16_t *smem, Claim claim) {
    const int blk = item / p.num_kv_heads, kvh = item - blk * p.num_kv_heads;
    const uint32_t u = load_unit(p, p.num_tile_units + blk);
    const TileDesc it = load_tile_desc(p, u);
    return wave16_path<D, STREAM>(p, it, (int)(u >> kUnitTileBits), (kvh + it.seq) % p.num_kv_heads, smem, claim);
}
template <int D>
__device__ __forceinline__ void chunk_item(const AttnParams &p, int item, uint16_t *smem) {
    const int blk = item / p.num_kv_heads, kvh = item - blk * p.num_kv_heads;  // consecutive items = the KV heads of one unit
    const uint32_t u = load_unit(p, blk);
    chunk_tile_path<D>(p, load_tile_desc(p, u), (int)(u >> kUnitTileBits), kvh, smem);
}

// Chunk tiles: one block per (unit, KV head); one wavefront per SIMD so that the pipelined
// loop has the registers it needs, the matrix pipe / vector ALU overlap comes from inside the wave.
template <int D, typename Args>
__global__ __launch_bounds__(256, 2) void attn_chunk_kernel(Args args) {
    const AttnParams p = attn_params(args);
    __shared__ __attribute__((aligned(16))) uint16_t smem[ChunkSmem<D>::kTotalElems];
    chunk_item<D>(p, (int)blockIdx.x, smem);
}

// Wave tiles (decodes, tiny chunks): one item per block or, QUEUED, the first gridDim.x items by the blocks in order and the
// others from the queue.
template <int D, bool STREAM, bool QUEUED, typename Args>
__global__ __launch_bounds__(256, 2) void attn_wave_kernel(Args args) {
    const AttnParams p = attn_params(args);
    __shared__ __attribute__((aligned(16))) uint16_t smem[WaveSmem<D>::kTotalElems];
    const int block = (int)blockIdx.x;
    if constexpr (!QUEUED) {
        wave_item<D, STREAM>(p, block, smem, [] { return 0; });
    } else {
        __shared__ int32_t next_item;
        Queue q{p.sched, (p.num_units - p.num_tile_units) * p.num_kv_heads, (int)gridDim.x, block % kSchedLists};
        for (int item = block; item != kNoItem;) {
            const int got = wave_item<D, STREAM>(p, item, smem, [&] { return q.bump(); });
            if (threadIdx.x == 0) next_item = q.take(got);
            __syncthreads();  // (and everyone is done with the ring's bytes; the next write is behind the next item's barrier)
            item = __builtin_amdgcn_readfirstlane(next_item);
        }
    }
}

// Both kinds of unit in ONE launch (saves the second stream's fork and join).
//
// kOneEach: a block per item, the chunk tiles in front.
// kQueued: the first blocks run a chunk tile each and the others begin with a wave tile; then all take wave tiles from the queue.
// kRoles: chunk blocks are compute-bound and wave blocks memory-bound, and they overlap only when they share a compute
// unit; two chunk blocks on one unit leave it without a memory stream.  So one block per compute unit (the first
// half of the grid, which the hardware spreads over the units before it gives any of them a second block) works off the chunk
// tiles and the other the wave tiles, each kind longest first, and a block whose queue is empty takes from the other one.
template <int D, int MODE, bool STREAM, typename Args>
__global__ __launch_bounds__(256, 2) void attn_hybrid_kernel(Args args) {
    const AttnParams p = attn_params(args);
    constexpr int kSmemElems = ChunkSmem<D>::kTotalElems > WaveSmem<D>::kTotalElems ? ChunkSmem<D>::kTotalElems : WaveSmem<D>::kTotalElems;
    __shared__ __attribute__((aligned(16))) uint16_t smem[kSmemElems];
    const int n_chunk = p.num_tile_units * p.num_kv_heads;
    const int block = (int)blockIdx.x;
    if constexpr (MODE == kOneEach) {
        if (block < n_chunk) chunk_item<D>(p, block, smem);
        else wave_item<D, STREAM>(p, block - n_chunk, smem, [] { return 0; });
    } else {
        __shared__ int32_t next_item;  // of the wave tiles; chunk tiles are numbered behind them
        const int n_wave = (p.num_units - p.num_tile_units) * p.num_kv_heads, blocks = (int)gridDim.x;
        const int chunk_blocks = MODE == kRoles ? blocks / 2 : n_chunk;
        Queue waves{p.sched, n_wave, min(n_wave, blocks - chunk_blocks), block % kSchedLists};
        Queue chunks{p.sched + kSchedLists * kSchedStride, n_chunk, min(n_chunk, chunk_blocks), block % kSchedLists};
        // the first thread's choice of the next item, after a wave tile whose claim returned `got` or after a chunk tile
        auto next = [&](bool after_wave, int got) -> int {
            if (MODE == kQueued) return waves.take(after_wave ? got : waves.bump());
            if (after_wave) {
                const int w = waves.item(got);
                if (w != kNoItem) return w;
            } else {
                const int c = chunks.item(chunks.bump());
                if (c != kNoItem) return n_wave + c;
            }
            for (;;) {  // the own list is at its end
                const bool more_waves = waves.move_on(), more_chunks = chunks.move_on();
                if (!more_waves && !more_chunks) return kNoItem;
                if (more_waves && (after_wave || !more_chunks)) {
                    const int w = waves.item(waves.bump());
                    if (w != kNoItem) return w;
                } else {
                    const int c = chunks.item(chunks.bump());
                    if (c != kNoItem) return n_wave + c;
                }
            }
        };
        int item;
        if (block < chunk_blocks && block < n_chunk) item = n_wave + block;
        else if (block >= chunk_blocks && block - chunk_blocks < n_wave) item = block - chunk_blocks;
        else {  // fewer items of the preferred kind than blocks that prefer it
            if (threadIdx.x == 0) next_item = next(block >= chunk_blocks, n_wave / kSchedLists + 1);
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(next_item);
            __syncthreads();
        }
        while (item != kNoItem) {
            const bool wave = item < n_wave;
            int got = 0;
            if (wave) got = wave_item<D, STREAM>(p, item, smem, [&] { return waves.bump(); });
            else chunk_item<D>(p, item - n_wave, smem);
            if (threadIdx.x == 0) next_item = next(wave, got);
            __syncthreads();  // (and everyone is done with the rings)
            item = __builtin_amdgcn_readfirstlane(next_item);
            __syncthreads();
        }
    }
}

// Per-call metadata, host -> device: a kernel that reads the pinned host buffer itself.  The runtime's copy
// goes through a copy kernel for a few kilobytes and through the DMA engine beyond that, and the DMA path
// leaves the stream idle for 10 us before and 13-23 us after the copy (kernel and copy trace of the
// decode-only batch, 13 KiB of metadata); a kernel of ours is followed by the next one at once.
__global__ __launch_bounds__(256) void upload_kernel(u32x4 *dst, const u32x4 *src, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// The same for callers that own no pinned buffer: the bytes travel in the kernel's arguments (the runtime copies
// the argument block when the launch is enqueued, so the source is free at once).  3,840 bytes per launch.
constexpr uint32_t kArgPieceWords = kUploadArgBytes / 4;
struct ArgPiece {
    uint32_t w[kArgPieceWords];
};
__global__ __launch_bounds__(256) void upload_args_kernel(u32x4 *dst, ArgPiece piece, uint32_t n16) {
    const uint32_t i = threadIdx.x;
    if (i < n16) dst[i] = u32x4{piece.w[4 * i], piece.w[4 * i + 1], piece.w[4 * i + 2], piece.w[4 * i + 3]};
}

__global__ void zero_words_kernel(uint32_t *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------------------
// Split-KV merge: out = sum_i w_i O_i / sum_i w_i l_i with w_i = 2^(m_i - max_i m_i), pieces
// taken in index order.  A block merges 8 columns of one split tile for one KV head: D/4
// threads per column, each owning four channels, so a piece's row is read as one coalesced
// run and the loop over pieces is unrolled to keep several loads in flight.
// ---------------------------------------------------------------------------------------
constexpr int kMergeCols = 8;  // columns per block of the merge kernel (must match the planner)

struct ReduceParams {
    const TileDesc *tiles;
    const uint32_t *reduce_units;  // (8-column group << kUnitTileBits) | tile index
    const float *part_ml;
    const float *part_o;
    uint16_t *out;
    int32_t num_q_heads;
    int32_t num_kv_heads;
    int32_t group;
};

// BATCH: pieces fetched at once.  Chunk tiles are cut into a few pieces of many rows and bound by their bytes: four (with
// eight, a batch of 56 tiles in two pieces took 25 us instead of 20).  Decodes that are cut to fill the chip have up to 32
// pieces of a few rows and are bound by latency: eight (32 pieces: 11.2 -> 6.8 us, 16 pieces 8.0 -> 6.5).  A launch has one
// size, by its finest cut: where both kinds are merged together eights and fours take the same time (14.2 and 14.5 us, 9.2
// and 8.1, 11.1 and 11.4, 8.3 and 8.5), and a launch per kind 2.5 to 3 us more.
template <int D, int BATCH>
__global__ __launch_bounds__(kMergeCols * D / 4) void splitkv_reduce_kernel(ReduceParams p) {
    constexpr int TPC = D / 4;  // threads per column
    const int kvh = blockIdx.x % p.num_kv_heads;
    const uint32_t u = p.reduce_units[blockIdx.x / p.num_kv_heads];
    const TileDesc it = p.tiles[u & ((1u << kUnitTileBits) - 1)];
    const int c = (int)(u >> kUnitTileBits) * kMergeCols + threadIdx.x / TPC;  // column inside the tile
    const int d4 = (threadIdx.x % TPC) * 4;
    if (c >= it.n_cols) return;
    const int col = it.col_begin + c;
    const int row = col / p.group;
    const int head = kvh * p.group + (col - row * p.group);
    const int64_t prow0 = ((int64_t)(it.part_row0 + c) * p.num_kv_heads + kvh);
    const int64_t split_stride = (int64_t)it.n_cols * p.num_kv_heads;
    const float *__restrict__ ml = p.part_ml;
    const float *__restrict__ po = p.part_o;
    // Loads first, arithmetic after: the pieces' rows were written by the attention launch and come from memory,
    // so a loop that loads, waits and accumulates piece by piece costs one memory latency per piece (and one more
    // per piece for the maxima).  BATCH pieces are fetched at once (indices beyond the last piece are clamped
    // to it: a valid, unused read), and the maxima of the later pieces as well; the sums still run in index order.
    const int n = it.n_splits;
    float m[BATCH], l[BATCH];
    f32x4 o[BATCH];
    auto fetch = [&](int base) {
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int64_t prow = prow0 + (int64_t)min(base + j, n - 1) * split_stride;
            const f32x2 v = *reinterpret_cast<const f32x2 *>(ml + prow * 2);
            m[j] = v[0];
            l[j] = v[1];
            o[j] = *reinterpret_cast<const f32x4 *>(po + prow * D + d4);
        }
    };
    fetch(0);
    float m_max = kNegSentinel;
#pragma unroll
    for (int j = 0; j < BATCH; ++j) m_max = fmaxf(m_max, m[j]);  // clamped entries repeat a valid piece
    for (int i = BATCH; i < n; i += BATCH) {
        float later[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) later[j] = ml[(prow0 + min(i + j, n - 1) * split_stride) * 2];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) m_max = fmaxf(m_max, later[j]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float lsum = 0.f;
    for (int base = 0;;) {
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            if (base + j < n) {
                const float w = __builtin_amdgcn_exp2f(m[j] - m_max);
                lsum += w * l[j];
                acc += o[j] * w;
            }
        }
        base += BATCH;
        if (base >= n) break;
        fetch(base);
    }
    const bf16x4 o4 = __builtin_convertvector(acc * (1.0f / lsum), bf16x4);
    uint16_t *op = p.out + ((int64_t)(it.q_start + row) * p.num_q_heads + head) * D + d4;
    *reinterpret_cast<u32x2 *>(op) = __builtin_bit_cast(u32x2, o4);
}

// ---------------------------------------------------------------------------------------
// KV append: byte copies into the paged pools.  A block fills the slots [lo, hi) of one cache
// page for one KV head (a page unit, built by the host: a decode has one, a chunk one per page
// it touches), one thread per channel.  K rows go over as 16-byte pieces (a page holds them
// slot-major, so the hi - lo rows are one contiguous run).  V pages are channel-major: thread c
// owns the 32-byte row of channel c, gathers the tokens' values of that channel (a wavefront
// reads 128 contiguous bytes per token) and, when the whole page is new, writes the row with
// two 16-byte stores (the block writes the 4 KiB page front to back); a partly filled page
// gets 2-byte stores into its new slots only, the others keep their bytes.
// ---------------------------------------------------------------------------------------
struct AppendParams {
    const uint16_t *k_new;
    const uint16_t *v_new;
    uint16_t *k_cache;
    uint16_t *v_cache;
    const int32_t *block_table;
    const AppendUnit *units;
    int64_t num_pages;
    int32_t max_blocks;
    int32_t num_kv_heads;
    // The first copy_blocks blocks move copy_n16 16-byte words from copy_src to copy_dst instead (the attention
    // metadata of the same iteration, pinned host memory -> workspace, riding in this launch).
    // The next zero_blocks clear zero_n16 words at zero_dst (scheduling words of the attention launch that follows).
    u32x4 *copy_dst;
    const u32x4 *copy_src;
    uint32_t copy_n16;
    uint32_t copy_blocks;
    u32x4 *zero_dst;
    uint32_t zero_n16;
    uint32_t zero_blocks;
};

// Small batches carry their records in the kernel's arguments, of two sizes, since the host copies them at each launch (64 tokens and 3 decodes
// in 384 bytes of records instead of 3584: 11.1 -> 10.6 us a pass; the argument block is on the device when the
// blocks start; a record in pinned host memory is a read across the host link at the head of every block's
// chain of dependent loads: record -> block-table entry -> stores).
constexpr int kInlineAppendUnits = 224, kFewAppendUnits = 24;
template <int UNITS>
struct AppendParamsInline {
    AppendParams base;
    AppendUnit units[UNITS];
};
static_assert(sizeof(AppendParamsInline<kInlineAppendUnits>) <= 4096, "kernel arguments are limited to 4 KiB");

template <int D>
__device__ __forceinline__ void kv_append_block(const AppendParams &p, const AppendUnit *units) {
    constexpr int kPieces = D / 8;  // 16-byte pieces of one K row
    if (blockIdx.x < p.copy_blocks) {
        const uint32_t i = blockIdx.x * D + threadIdx.x;
        if (i < p.copy_n16) p.copy_dst[i] = p.copy_src[i];
        return;
    }
    if (blockIdx.x < p.copy_blocks + p.zero_blocks) {
        const uint32_t i = (blockIdx.x - p.copy_blocks) * D + threadIdx.x;
        if (i < p.zero_n16) p.zero_dst[i] = u32x4{0, 0, 0, 0};
        return;
    }
    const unsigned blk = blockIdx.x - p.copy_blocks - p.zero_blocks;
    const int unit = (int)(blk / (unsigned)p.num_kv_heads);
    const int h = (int)(blk % (unsigned)p.num_kv_heads);
    const u32x4 rec = *reinterpret_cast<const u32x4 *>(units + unit);
    const int lo = (int)(rec[3] & 0xFFu), hi = (int)(rec[3] >> 8);
    const int n = hi - lo;
    const int64_t row_stride = (int64_t)p.num_kv_heads * D;
    const int64_t src = ((int64_t)(int)rec[2] * p.num_kv_heads + h) * D;
    const int tid = (int)threadIdx.x;
    // The block-table entry and the rows to move depend on the record only: all of these loads are issued
    // before the first is waited for (the table entry decides where the rows go, and whether they go at all).
    const int32_t *entry = p.block_table + (int64_t)(int)rec[0] * p.max_blocks + (int)rec[1];
    const int64_t page = *entry;

    // V: gather first (all loads in flight before any store)
    const uint16_t *vsrc = p.v_new + src + tid;
    uint16_t x[kPageSize];
#pragma unroll
    for (int i = 0; i < kPageSize; ++i) x[i] = (i < n) ? vsrc[i * row_stride] : (uint16_t)0;

    // K: n rows of D channels, destination contiguous
    constexpr int kRounds = (kPageSize * kPieces) / D;
    const uint16_t *ksrc = p.k_new + src;
    u32x4 krow[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int j = tid + r * D;
        const int i = j / kPieces, piece = j % kPieces;
        krow[r] = (i < n) ? *reinterpret_cast<const u32x4 *>(ksrc + i * row_stride + piece * 8) : u32x4{0, 0, 0, 0};
    }

    if (page < 0 || page >= p.num_pages) return;  // a corrupt table entry must not become a wild store
    const int64_t head_base = (page * p.num_kv_heads + h) * (int64_t)(kPageSize * D);
    uint16_t *kdst = p.k_cache + head_base + (int64_t)lo * D;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int j = tid + r * D;
        const int i = j / kPieces, piece = j % kPieces;
        if (i < n) *reinterpret_cast<u32x4 *>(kdst + i * D + piece * 8) = krow[r];
    }

    uint16_t *vdst = p.v_cache + head_base + (int64_t)tid * kPageSize;
    if (n == kPageSize) {
        u32x4 w0, w1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w0[e] = (uint32_t)x[2 * e] | ((uint32_t)x[2 * e + 1] << 16);
            w1[e] = (uint32_t)x[8 + 2 * e] | ((uint32_t)x[9 + 2 * e] << 16);
        }
        *reinterpret_cast<u32x4 *>(vdst) = w0;
        *reinterpret_cast<u32x4 *>(vdst + 8) = w1;
    } else {
#pragma unroll
        for (int i = 0; i < kPageSize; ++i)
            if (i < n) vdst[lo + i] = x[i];
    }
}

template <int D>
__global__ __launch_bounds__(D) void kv_append_kernel(AppendParams p) {
    kv_append_block<D>(p, p.units);
}
template <int D, int UNITS>
__global__ __launch_bounds__(D) void kv_append_inline_kernel(AppendParamsInline<UNITS> p) {
    kv_append_block<D>(p.base, p.units);
}

// ---------------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------------
int launch_kv_append(const sarathi_config &cfg, const AppendMeta &m, const void *k_new, const void *v_new,
                     void *k_cache, void *v_cache, int64_t num_pages, void *stream) {
    if (m.num_units == 0) return (int)hipSuccess;
    AppendParams p;
    p.k_new = static_cast<const uint16_t *>(k_new);
    p.v_new = static_cast<const uint16_t *>(v_new);
    p.k_cache = static_cast<uint16_t *>(k_cache);
    p.v_cache = static_cast<uint16_t *>(v_cache);
    p.block_table = m.block_table;
    p.units = m.units;
    p.num_pages = num_pages;
    p.max_blocks = m.max_blocks;
    p.num_kv_heads = cfg.num_kv_heads;
    p.copy_dst = static_cast<u32x4 *>(m.copy_dst);
    p.copy_src = static_cast<const u32x4 *>(m.copy_src);
    p.copy_n16 = (uint32_t)((m.copy_bytes + 15) / 16);
    p.copy_blocks = (p.copy_n16 + (uint32_t)cfg.head_dim - 1) / (uint32_t)cfg.head_dim;
    p.zero_dst = static_cast<u32x4 *>(m.zero_dst);
    p.zero_n16 = (uint32_t)((m.zero_bytes + 15) / 16);
    p.zero_blocks = (p.zero_n16 + (uint32_t)cfg.head_dim - 1) / (uint32_t)cfg.head_dim;
    const unsigned blocks = p.copy_blocks + p.zero_blocks + (unsigned)m.num_units * (unsigned)cfg.num_kv_heads;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (m.units_host && m.num_units <= kInlineAppendUnits) {
        auto launch = [&](auto units) {
            constexpr int U = decltype(units)::value;
            AppendParamsInline<U> pi;
            pi.base = p;
            std::memcpy(pi.units, m.units_host, sizeof(AppendUnit) * (size_t)m.num_units);
            if (cfg.head_dim == 128)
                hipLaunchKernelGGL((kv_append_inline_kernel<128, U>), dim3(blocks), dim3(128), 0, st, pi);
            else
                hipLaunchKernelGGL((kv_append_inline_kernel<64, U>), dim3(blocks), dim3(64), 0, st, pi);
        };
        if (m.num_units <= kFewAppendUnits) launch(std::integral_constant<int, kFewAppendUnits>{});
        else launch(std::integral_constant<int, kInlineAppendUnits>{});
        return (int)hipGetLastError();
    }
    if (cfg.head_dim == 128)
        hipLaunchKernelGGL(kv_append_kernel<128>, dim3(blocks), dim3(128), 0, st, p);
    else
        hipLaunchKernelGGL(kv_append_kernel<64>, dim3(blocks), dim3(64), 0, st, p);
    return (int)hipGetLastError();
}

int launch_upload(void *dst, const void *pinned_src, size_t bytes, void *stream) {
    const size_t n = (bytes + 15) / 16;
    if (n == 0) return (int)hipSuccess;
    hipLaunchKernelGGL(upload_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<u32x4 *>(dst), static_cast<const u32x4 *>(pinned_src), n);
    return (int)hipGetLastError();
}

int launch_upload_args(void *dst, const void *host_src, size_t bytes, void *stream) {
    static_assert(sizeof(ArgPiece) + 16 <= 4096, "kernel arguments are limited to 4 KiB");
    const char *src = static_cast<const char *>(host_src);
    char *d = static_cast<char *>(dst);
    for (size_t off = 0; off < bytes; off += sizeof(ArgPiece)) {
        const size_t n = bytes - off < sizeof(ArgPiece) ? bytes - off : sizeof(ArgPiece);
        ArgPiece piece;
        std::memcpy(piece.w, src + off, n);
        hipLaunchKernelGGL(upload_args_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream),
                           reinterpret_cast<u32x4 *>(d + off), piece, (uint32_t)((n + 15) / 16));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return (int)e;
    }
    return (int)hipSuccess;
}

// ---------------------------------------------------------------------------------------
// Scratch of the allocation-free entry point: one array in the device image of this library, so every GPU the
// library runs on holds its own copy until the process ends.  Host code never uses the array's name as an
// address: the device address is looked up once per device and used from then on.
// ---------------------------------------------------------------------------------------
constexpr size_t kStaticSchedBytes = (kSchedBytes + 255) / 256 * 256;
constexpr size_t kStaticScratchBytes = kStaticMetaBytes + kStaticSchedBytes + kStaticPartMlBytes + kStaticPartOBytes;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

int static_scratch(StaticScratch *out) {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static char *base_of_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    char *base;
    {
        std::lock_guard<std::mutex> guard(lock);
        if (!base_of_device[dev]) {
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return (int)e;
            if (!ptr) return (int)hipErrorInvalidSymbol;
            base_of_device[dev] = static_cast<char *>(ptr);
        }
        base = base_of_device[dev];
    }
    out->meta = base;
    out->sched = reinterpret_cast<int32_t *>(base + kStaticMetaBytes);
    out->part_ml = reinterpret_cast<float *>(base + kStaticMetaBytes + kStaticSchedBytes);
    out->part_o = reinterpret_cast<float *>(base + kStaticMetaBytes + kStaticSchedBytes + kStaticPartMlBytes);
    return (int)hipSuccess;
}

int launch_zero(void *ptr, size_t bytes, void *stream) {
    const size_t n = bytes / 4;
    if (n == 0) return (int)hipSuccess;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<uint32_t *>(ptr), n);
    return (int)hipGetLastError();
}

int launch_reduce(const sarathi_config &cfg, const AttnMeta &m, void *out, int32_t first, int32_t count, void *stream) {
    if (count <= 0) return (int)hipSuccess;
    static_assert(kMergeCols == kReduceCols, "planner and merge kernel must agree on columns per block");
    ReduceParams p;
    p.tiles = m.tiles;
    p.reduce_units = m.reduce_units + first;
    p.part_ml = m.part_ml;
    p.part_o = m.part_o;
    p.out = static_cast<uint16_t *>(out);
    p.num_q_heads = cfg.num_q_heads;
    p.num_kv_heads = cfg.num_kv_heads;
    p.group = cfg.num_q_heads / cfg.num_kv_heads;
    const unsigned blocks = (unsigned)count * (unsigned)cfg.num_kv_heads;
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto launch = [&](auto d, auto batch) {
        constexpr int D = decltype(d)::value;
        hipLaunchKernelGGL((splitkv_reduce_kernel<D, decltype(batch)::value>), dim3(blocks), dim3(kMergeCols * D / 4), 0, st, p);
    };
    auto pick_batch = [&](auto d) {
        if (m.most_pieces <= 4) launch(d, std::integral_constant<int, 4>{});
        else launch(d, std::integral_constant<int, 8>{});
    };
    if (cfg.head_dim == 128) pick_batch(std::integral_constant<int, 128>{});
    else pick_batch(std::integral_constant<int, 64>{});
    return (int)hipGetLastError();
}

int launch_attention(const sarathi_config &cfg, const AttnMeta &m, const void *q, const void *k_cache,
                     const void *v_cache, int64_t num_pages, float sm_scale, void *out, int which, void *stream) {
    if (m.num_units == 0) return (int)hipSuccess;
    AttnParams p;
    p.q = static_cast<const uint16_t *>(q);
    p.k_cache = static_cast<const uint16_t *>(k_cache);
    p.v_cache = static_cast<const uint16_t *>(v_cache);
    p.out = static_cast<uint16_t *>(out);
    p.block_table = m.block_table;
    p.tiles = m.tiles;
    p.units = m.units;
    p.part_ml = m.part_ml;
    p.part_o = m.part_o;
    p.num_pages = num_pages;
    p.max_blocks = m.max_blocks;
    p.num_q_heads = cfg.num_q_heads;
    p.num_kv_heads = cfg.num_kv_heads;
    p.group = cfg.num_q_heads / cfg.num_kv_heads;
    p.num_tile_units = m.num_tile_units;
    p.num_units = m.num_units;
    p.scale_log2 = sm_scale * 1.4426950408889634f;
    p.sched = m.sched;
    p.window = m.window;
    if (m.plan_bytes > 0 && (m.plan_bytes > kPlanArgBytes || m.queue_blocks > 0)) return (int)hipErrorInvalidConfiguration;
    // launch(arguments) of a launch of a block per item
    auto with_plan = [&](auto launch) {
        if (m.plan_bytes == 0) return launch(p);
        auto carry = [&](auto args) {
            args.base = p;
            args.units_off = (uint32_t)(reinterpret_cast<const char *>(m.units) - reinterpret_cast<const char *>(m.tiles));
            std::memcpy(args.plan, m.tiles, m.plan_bytes);
            launch(args);
        };
        if (m.plan_bytes <= kSmallPlanArgBytes) carry(AttnArgs<kSmallPlanArgBytes>{}); else carry(AttnArgs<kPlanArgBytes>{});
    };
    const bool stream_kv = m.stream_kv != 0;
    // unused LDS that lowers the blocks per compute unit; all it can take next to the blocks' own 64 KiB already leaves one
    const unsigned dyn_lds = (unsigned)std::min<int32_t>(m.lds_pad_bytes, 95 * 1024);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const unsigned chunk_blocks = (unsigned)m.num_tile_units * (unsigned)cfg.num_kv_heads;
    const unsigned wave_blocks = (unsigned)(m.num_units - m.num_tile_units) * (unsigned)cfg.num_kv_heads;
    const unsigned in_flight = m.queue_blocks > 0 ? (unsigned)m.queue_blocks : 0xFFFFFFFFu;
    auto with_stream = [&](auto launch) {
        if (stream_kv) launch(std::true_type{}); else launch(std::false_type{});
    };
    if (which == 4 || which == 5) {
        const dim3 grid(std::min(chunk_blocks + wave_blocks, in_flight));
        auto launch = [&](auto d, auto mode) {
            with_stream([&](auto hint) {
                auto go = [&](const auto &args) {
                    hipLaunchKernelGGL((attn_hybrid_kernel<decltype(d)::value, decltype(mode)::value, decltype(hint)::value, std::decay_t<decltype(args)>>), grid,
                                       dim3(256), dyn_lds, st, args);
                };
                if constexpr (decltype(mode)::value == kOneEach) with_plan(go); else go(p);
            });
        };
        auto pick_mode = [&](auto d) {
            if (which == 5) launch(d, std::integral_constant<int, kRoles>{});
            else if (m.queue_blocks > 0) launch(d, std::integral_constant<int, kQueued>{});
            else launch(d, std::integral_constant<int, kOneEach>{});
        };
        if (cfg.head_dim == 128) pick_mode(std::integral_constant<int, 128>{});
        else pick_mode(std::integral_constant<int, 64>{});
        return (int)hipGetLastError();
    }
    if (chunk_blocks && (which & 1)) {
        with_plan([&](const auto &args) {
            using Args = std::decay_t<decltype(args)>;
            if (cfg.head_dim == 128)
                hipLaunchKernelGGL((attn_chunk_kernel<128, Args>), dim3(chunk_blocks), dim3(256), dyn_lds, st, args);
            else
                hipLaunchKernelGGL((attn_chunk_kernel<64, Args>), dim3(chunk_blocks), dim3(256), dyn_lds, st, args);
        });
    }
    if (wave_blocks && (which & 2)) {
        const dim3 grid(std::min(wave_blocks, in_flight));
        auto launch = [&](auto d, auto queued) {
            with_stream([&](auto hint) {
                auto go = [&](const auto &args) {
                    hipLaunchKernelGGL((attn_wave_kernel<decltype(d)::value, decltype(hint)::value, decltype(queued)::value, std::decay_t<decltype(args)>>), grid,
                                       dim3(256), dyn_lds, st, args);
                };
                if constexpr (!decltype(queued)::value) with_plan(go); else go(p);
            });
        };
        auto pick_queued = [&](auto d) {
            if (m.queue_blocks > 0) launch(d, std::true_type{}); else launch(d, std::false_type{});
        };
        if (cfg.head_dim == 128) pick_queued(std::integral_constant<int, 128>{});
        else pick_queued(std::integral_constant<int, 64>{});
    }
    return (int)hipGetLastError();
}

}  // namespace sarathi
