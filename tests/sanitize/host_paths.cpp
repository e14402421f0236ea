// Host-only build of the library's CPU code (batch validation, planner, scheduler, the bookkeeping of the entry
// points) and of the fp64 checker, for AddressSanitizer / UndefinedBehaviorSanitizer.  No GPU and no HIP runtime:
// the few runtime calls api.cpp makes are replaced by host stand-ins below ("pinned" memory is malloc memory,
// events and streams are dummies), and the kernel launchers are replaced by functions that walk exactly the
// metadata a kernel would read and, for the append, move the rows on the host.  Every "device" buffer is a heap
// block of exactly the documented size, so a record or plan entry that points outside them is an ASan error.
//
// Built and run by tests/test_sanitizers.py (g++/gcc -fsanitize=address,undefined); exit code 0 = clean.
#include <hip/hip_runtime_api.h>

#include <cassert>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "internal.h"
#include "sarathi.h"

// ---- checker entry points (C, compiled separately with the same sanitizers) ----
extern "C" int oracle_hybrid_attention_window(const uint16_t *q, const uint16_t *k_seq, const uint16_t *v_seq,
                                              const int64_t *kv_start, const int32_t *q_start, const int32_t *q_len,
                                              const int32_t *ctx_len, int num_seqs, int num_tokens, int num_q_heads,
                                              int num_kv_heads, int d, double sm_scale, int window, const int32_t *tokens,
                                              int n_rows, double *out, int num_threads);
extern "C" int oracle_softmax_weights(const uint16_t *q, const uint16_t *k_seq, const int64_t *kv_start, const int32_t *q_start,
                                      const int32_t *q_len, const int32_t *ctx_len, int num_seqs, int num_q_heads,
                                      int num_kv_heads, int d, double sm_scale, int token, int head, double *w);
extern "C" int oracle_linear(const uint16_t *x, const uint16_t *w, int T, int N, int K, const int32_t *rows, int n_rows,
                             const int32_t *cols, int n_cols, double *out, int num_threads);

#define CHECK(cond)                                                                   \
    do {                                                                              \
        if (!(cond)) {                                                                \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(3);                                                             \
        }                                                                             \
    } while (0)

// ---- stand-ins for the HIP runtime calls of api.cpp ----
extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "host stand-in"; }
}

// ---- stand-ins for the kernel launchers: read what the kernels would read ----
namespace sarathi {

static int g_num_seqs = 0;          // shape of the call in flight, for the walkers below
static int64_t g_num_tokens = 0;
static uint64_t g_sink = 0;
static int32_t g_lds_pad_bytes = 0; // of the last attention launch
static int g_which = 0;             // and its kind
static int32_t g_queue_blocks = 0;
static int g_queued_launches = 0;
static size_t g_plan_bytes = 0;     // of the plan in the last attention launch's arguments

int launch_kv_append(const sarathi_config &cfg, const AppendMeta &m, const void *k_new, const void *v_new, void *k_cache,
                     void *v_cache, int64_t num_pages, void *) {
    const int D = cfg.head_dim, H = cfg.num_kv_heads;
    const uint16_t *kn = static_cast<const uint16_t *>(k_new), *vn = static_cast<const uint16_t *>(v_new);
    uint16_t *kc = static_cast<uint16_t *>(k_cache), *vc = static_cast<uint16_t *>(v_cache);
    if (m.copy_bytes) std::memcpy(m.copy_dst, m.copy_src, (m.copy_bytes + 15) / 16 * 16);
    CHECK(m.zero_bytes % 16 == 0 && reinterpret_cast<uintptr_t>(m.zero_dst) % 16 == 0);
    if (m.zero_bytes) std::memset(m.zero_dst, 0, m.zero_bytes);
    for (int u = 0; u < m.num_units; ++u) {
        const AppendUnit &r = m.units[u];
        const int lo = r.lo_hi & 0xFF, hi = r.lo_hi >> 8;
        CHECK(r.seq >= 0 && r.seq < g_num_seqs && r.page_idx >= 0 && r.page_idx < m.max_blocks);
        CHECK(0 <= lo && lo < hi && hi <= kPageSize && r.row0 >= 0 && r.row0 + (hi - lo) <= g_num_tokens);
        const int64_t page = m.block_table[(int64_t)r.seq * m.max_blocks + r.page_idx];
        CHECK(page >= 0 && page < num_pages);
        for (int h = 0; h < H; ++h)
            for (int i = lo; i < hi; ++i)
                for (int c = 0; c < D; ++c) {
                    const int64_t src = ((int64_t)(r.row0 + i - lo) * H + h) * D + c;
                    kc[((page * H + h) * kPageSize + i) * D + c] = kn[src];
                    vc[((page * H + h) * D + c) * kPageSize + i] = vn[src];
                }
    }
    return 0;
}

int launch_upload(void *dst, const void *src, size_t bytes, void *) {
    std::memcpy(dst, src, (bytes + 15) / 16 * 16);
    return 0;
}
int launch_upload_args(void *dst, const void *src, size_t bytes, void *) {
    CHECK(bytes % 16 == 0);
    std::memcpy(dst, src, bytes);
    return 0;
}
int launch_zero(void *p, size_t bytes, void *) {
    std::memset(p, 0, bytes);
    return 0;
}

static std::vector<char> g_static;
int static_scratch(StaticScratch *out) {
    const size_t sched = (kSchedBytes + 255) / 256 * 256;
    if (g_static.empty()) g_static.resize(kStaticMetaBytes + sched + kStaticPartMlBytes + kStaticPartOBytes);
    char *base = g_static.data();
    out->meta = base;
    out->sched = reinterpret_cast<int32_t *>(base + kStaticMetaBytes);
    out->part_ml = reinterpret_cast<float *>(base + kStaticMetaBytes + sched);
    out->part_o = reinterpret_cast<float *>(base + kStaticMetaBytes + sched + kStaticPartMlBytes);
    return 0;
}

// The blocks of a queued launch, advanced one item at a time in an order drawn at random: each takes its first item by its index and
// the others as the kernels do (own list first, then the one with most left, and with roles the other kind).  Every item has
// to be run exactly once.
static std::mt19937_64 g_order(7);
static void play_queues(const AttnMeta &m, int H, int which) {
    for (int w = 0; w < kSchedWords; ++w) CHECK(m.sched[w] == 0);
    const bool one_launch = which == 4 || which == 5, roles = which == 5;
    const int n_wave = (m.num_units - m.num_tile_units) * H, n_chunk = one_launch ? m.num_tile_units * H : 0;
    const int blocks = std::min(n_wave + n_chunk, m.queue_blocks);
    const int chunk_blocks = roles ? blocks / 2 : n_chunk;
    CHECK(chunk_blocks <= blocks);
    struct Queue {
        int32_t *counters;
        int n, taken;
        int bump(int list) { return counters[list * kSchedStride]++; }
        int item(int list, int got) { const int i = queue_item(taken, list, got); return i < n ? i : -1; }
        bool move_on(int &list) {
            int most = 0;
            for (int x = 0; x < kSchedLists; ++x) {
                const int left = n - queue_item(taken, x, counters[x * kSchedStride]);
                if (left > most) most = left, list = x;
            }
            return most > 0;
        }
    } waves{m.sched, n_wave, std::min(n_wave, blocks - chunk_blocks)}, chunks{m.sched + kSchedLists * kSchedStride, n_chunk, std::min(n_chunk, chunk_blocks)};
    std::vector<int> runs((size_t)(n_wave + n_chunk), 0);
    struct Block { int index, wave_list, chunk_list, item; };   // item -2: none yet
    std::vector<Block> busy;
    for (int b = 0; b < blocks; ++b) {
        int item = -2;
        if (b < chunk_blocks && b < n_chunk) item = n_wave + b;
        else if (b >= chunk_blocks && b - chunk_blocks < n_wave) item = b - chunk_blocks;
        busy.push_back(Block{b, b % kSchedLists, b % kSchedLists, item});
    }
    while (!busy.empty()) {
        const size_t at = (size_t)(g_order() % busy.size());
        Block &b = busy[at];
        if (b.item >= 0) CHECK(++runs[(size_t)b.item] == 1);
        const bool after_wave = b.item == -2 ? b.index >= chunk_blocks : b.item < n_wave;
        int next = -1;
        if (!roles || after_wave) {
            if (b.item != -2) next = waves.item(b.wave_list, waves.bump(b.wave_list));
        } else {
            next = chunks.item(b.chunk_list, chunks.bump(b.chunk_list));
            if (next >= 0) next += n_wave;
        }
        while (next < 0) {
            const bool more_waves = waves.move_on(b.wave_list), more_chunks = roles && chunks.move_on(b.chunk_list);
            if (!more_waves && !more_chunks) break;
            if (more_waves && (after_wave || !more_chunks)) {
                next = waves.item(b.wave_list, waves.bump(b.wave_list));
            } else {
                next = chunks.item(b.chunk_list, chunks.bump(b.chunk_list));
                if (next >= 0) next += n_wave;
            }
        }
        if (next >= 0) b.item = next;
        else { busy[at] = busy.back(); busy.pop_back(); }
    }
    for (int n : runs) CHECK(n == 1);
    for (int w = 0; w < kSchedWords; ++w) m.sched[w] ^= 0x5A5A5A5A;   // nobody may count on what a launch leaves
    g_queued_launches++;
}

// Every (column, key) pair of the batch must be covered by exactly one work unit, every unit must stay inside
// its sequence, and every partial row / counter a unit or merge item names must lie inside its buffer (touched
// here so that ASan sees an overrun).
int launch_attention(const sarathi_config &cfg, const AttnMeta &given, const void *, const void *, const void *, int64_t,
                     float, void *, int which, void *) {
    const int H = cfg.num_kv_heads, D = cfg.head_dim;
    // A plan in the launch's arguments: the kernels see so many bytes and nothing behind them.
    AttnMeta m = given;
    std::vector<char> arguments(m.plan_bytes);
    g_plan_bytes = m.plan_bytes;
    if (m.plan_bytes > 0) {
        CHECK(m.plan_bytes <= kPlanArgBytes && m.queue_blocks == 0 && m.num_reduce_units == 0);
        const size_t units = (size_t)(reinterpret_cast<const char *>(m.units) - reinterpret_cast<const char *>(m.tiles));
        std::memcpy(arguments.data(), m.tiles, m.plan_bytes);
        m.tiles = reinterpret_cast<const TileDesc *>(arguments.data());
        m.units = reinterpret_cast<const uint32_t *>(arguments.data() + units);
        CHECK(units + sizeof(uint32_t) * (size_t)m.num_units <= m.plan_bytes);
    }
    g_lds_pad_bytes = m.lds_pad_bytes;
    g_which = which;
    g_queue_blocks = m.queue_blocks;
    CHECK(which != 5 || m.queue_blocks > 0);
    CHECK(which != 4 || m.queue_blocks == 0 || m.queue_blocks >= m.num_tile_units * H);   // every chunk tile has a block of its own
    if (m.queue_blocks > 0 && which != 1) play_queues(m, H, which);
    for (int u = 0; u < m.num_units; ++u) {
        const uint32_t unit = m.units[u];
        const TileDesc &t = m.tiles[unit & ((1u << kUnitTileBits) - 1)];
        const int split = (int)(unit >> kUnitTileBits);
        CHECK(t.seq >= 0 && t.seq < g_num_seqs && split < t.n_splits);
        CHECK((u < m.num_tile_units) == (t.kind == kKindTile));
        CHECK(t.n_cols >= 1 && t.n_cols <= (t.kind == kKindTile ? kTileCols : kWaveCols));
        CHECK(t.n_keys >= 1 && t.n_keys <= t.ctx_len && t.key_lo >= 0 && t.key_lo % kTileKeys == 0 && t.key_lo < t.n_keys);
        CHECK(t.keys_per_split % kTileKeys == 0 && t.key_lo + (int64_t)split * t.keys_per_split < t.n_keys);
        CHECK((int64_t)t.q_start + t.q_len <= g_num_tokens);
        const int n_pages = (t.ctx_len + kPageSize - 1) / kPageSize;
        g_sink += (uint64_t)m.block_table[(int64_t)t.seq * m.max_blocks + n_pages - 1];  // last table entry the kernel may read
        if (t.n_splits > 1) {
            CHECK(t.part_row0 >= 0);
            const int64_t last_row = (int64_t)t.part_row0 + (int64_t)t.n_splits * t.n_cols - 1;
            m.part_o[(last_row * H + H - 1) * D + D - 1] = 0.f;
            m.part_ml[(last_row * H + H - 1) * 2 + 1] = 0.f;
        } else {
            CHECK(t.part_row0 == -1);
        }
    }
    for (int r = 0; r < m.num_reduce_units; ++r) {
        const uint32_t ru = m.reduce_units[r];
        const TileDesc &t = m.tiles[ru & ((1u << kUnitTileBits) - 1)];
        CHECK(t.n_splits > 1 && (int)(ru >> kUnitTileBits) * kReduceCols < t.n_cols);
    }
    return 0;
}
int launch_reduce(const sarathi_config &, const AttnMeta &m, void *, int32_t first, int32_t count, void *) {
    CHECK(first >= 0 && first + count <= m.num_reduce_units);
    return 0;
}

}  // namespace sarathi

// ---- drivers ----
static void drive_scheduler(std::mt19937_64 &rng) {
    auto rnd = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    for (int it = 0; it < 2000; ++it) {
        const int nd = rnd(0, 40), np = rnd(0, 4), nw = rnd(0, 6);
        std::vector<sarathi_request> dec(nd), pre(np), wait(nw);
        for (int i = 0; i < nd; ++i) { int p = rnd(1, 3000); dec[i] = sarathi_request{i, p, p, rnd(0, 50), 0}; }
        for (int i = 0; i < np; ++i) { int p = rnd(2, 9000); pre[i] = sarathi_request{100 + i, p, rnd(0, p - 1), 0, 0}; }
        for (int i = 0; i < nw; ++i) wait[i] = sarathi_request{200 + i, rnd(1, 9000), 0, 0, 0};
        const int cap = rnd(1, 60);
        std::vector<int64_t> id(cap);
        std::vector<int32_t> qs(cap), ql(cap), cl(cap);
        sarathi_batch b{};
        b.seq_id = id.data(); b.q_start = qs.data(); b.q_len = ql.data(); b.ctx_len = cl.data();
        const int budget = rnd(1, 2048), chunk = rnd(1, 4096);
        const sarathi_status st = sarathi_build_stall_free_batch(budget, chunk, nd ? dec.data() : nullptr, nd, np ? pre.data() : nullptr,
                                                                  np, nw ? wait.data() : nullptr, nw, rnd(0, 2000), 16, cap, &b);
        if (nd > cap) { CHECK(st == SARATHI_ECAPACITY); continue; }
        CHECK(st == SARATHI_OK && b.num_seqs <= cap && b.num_decodes == nd);
        int64_t run = 0;
        for (int i = 0; i < b.num_seqs; ++i) { CHECK(qs[i] == run && ql[i] >= 1 && cl[i] >= ql[i]); run += ql[i]; }
        CHECK(run == b.num_tokens);
    }
    sarathi_batch bad{};
    CHECK(sarathi_build_stall_free_batch(8, 8, nullptr, 0, nullptr, 0, nullptr, 0, 0, 16, 4, &bad) == SARATHI_EINVAL);
}

static void drive_attention_host_paths(std::mt19937_64 &rng) {
    auto rnd = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    const int shapes[][3] = {{8, 2, 128}, {4, 1, 64}, {14, 2, 128}, {3, 3, 64}};
    for (int it = 0; it < 60; ++it) {
        const int *sh = shapes[it % 4];
        sarathi_config cfg{sh[0], sh[1], sh[2], 16, 0, 4096, 64, 0};
        const int S = rnd(1, 24);
        std::vector<int32_t> qs(S), ql(S), cl(S);
        int64_t T = 0, pages_needed = 0;
        int max_blocks = 1;
        for (int s = 0; s < S; ++s) {
            const bool chunk = rnd(0, 3) == 0;
            ql[s] = chunk ? rnd(2, 300) : 1;
            cl[s] = ql[s] + rnd(0, it % 5 == 0 ? 9000 : 700);
            qs[s] = (int32_t)T;
            T += ql[s];
            pages_needed += (cl[s] + 15) / 16;
            max_blocks = std::max(max_blocks, (cl[s] + 15) / 16);
        }
        cfg.max_blocks_per_seq = max_blocks;
        sarathi_handle *h = nullptr;
        CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
        if (it % 3 == 1) CHECK(sarathi_set_option(h, "split_keys", 64) == SARATHI_OK && sarathi_set_option(h, "tile_split_keys", 64) == SARATHI_OK);
        if (it % 3 == 2) CHECK(sarathi_set_option(h, "window", rnd(1, 500)) == SARATHI_OK);
        if (it % 4 == 3) CHECK(sarathi_set_option(h, "resident_chunks", 1) == SARATHI_OK);
        const int64_t num_pages = pages_needed + 3;
        std::vector<int32_t> bt((size_t)S * max_blocks, -1);
        int64_t next = 0;
        for (int s = 0; s < S; ++s)
            for (int b = 0; b < (cl[s] + 15) / 16; ++b) bt[(size_t)s * max_blocks + b] = (int32_t)next++;
        const size_t row = (size_t)cfg.num_kv_heads * cfg.head_dim;
        std::vector<uint16_t> k_new((size_t)T * row, 1), v_new((size_t)T * row, 2);
        std::vector<uint16_t> kc((size_t)num_pages * row * 16), vc((size_t)num_pages * row * 16);
        std::vector<uint16_t> q((size_t)T * cfg.num_q_heads * cfg.head_dim), out(q.size());
        // the workspace is handed over 256-byte aligned and exactly as large as the library asks for
        const size_t ws_bytes = sarathi_workspace_bytes(h);
        void *ws = nullptr;
        CHECK(posix_memalign(&ws, 256, ws_bytes) == 0);
        std::memset(ws, 0xFF, ws_bytes);
        sarathi::g_num_seqs = S;
        sarathi::g_num_tokens = T;
        CHECK(sarathi_kv_append(h, k_new.data(), v_new.data(), kc.data(), vc.data(), bt.data(), qs.data(), ql.data(), cl.data(), S,
                                (int32_t)T, num_pages, ws, nullptr) == SARATHI_OK);
        for (int rep = 0; rep < 2; ++rep)   // the second call finds the plan the append brought still resident
            CHECK(sarathi_hybrid_attention(h, q.data(), kc.data(), vc.data(), bt.data(), qs.data(), ql.data(), cl.data(), S, (int32_t)T,
                                           num_pages, 0.1f, out.data(), ws, nullptr) == SARATHI_OK);
        CHECK(sarathi_hybrid_attention_noalloc(h, q.data(), kc.data(), vc.data(), bt.data(), qs.data(), ql.data(), cl.data(), S,
                                               (int32_t)T, num_pages, 0.1f, out.data(), nullptr) == SARATHI_OK);
        sarathi_plan_info info{};
        CHECK(sarathi_plan_hybrid_attention(h, qs.data(), ql.data(), cl.data(), S, (int32_t)T, &info, nullptr, 0) == SARATHI_OK);
        std::vector<sarathi_work_item> items((size_t)std::max(1, info.num_items));
        CHECK(sarathi_plan_hybrid_attention(h, qs.data(), ql.data(), cl.data(), S, (int32_t)T, &info, items.data(), info.num_items) == SARATHI_OK);
        // error paths: nothing may be touched
        ql[0] += 1;
        CHECK(sarathi_kv_append(h, k_new.data(), v_new.data(), kc.data(), vc.data(), bt.data(), qs.data(), ql.data(), cl.data(), S,
                                (int32_t)T, num_pages, ws, nullptr) != SARATHI_OK);
        ql[0] -= 1;
        CHECK(sarathi_hybrid_attention(h, q.data(), kc.data(), vc.data(), bt.data(), qs.data(), ql.data(), cl.data(), S, (int32_t)T,
                                       num_pages, 0.1f, out.data(), static_cast<char *>(ws) + 8, nullptr) == SARATHI_EWORKSPACE);
        CHECK(sarathi_destroy(h) == SARATHI_OK);
        std::free(ws);
    }
}

// Batches close to what the allocation-free entry point holds (96 KiB of metadata): one whose tiles fit whole is taken,
// however finely its keys would be cut elsewhere, and one whose tiles do not is refused.
static void drive_built_in_scratch_limits(std::mt19937_64 &rng) {
    auto rnd = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    const int shapes[][3] = {{71, 1, 64}, {64, 1, 128}, {20, 1, 128}, {64, 8, 128}};
    int taken = 0, refused = 0;
    for (int it = 0; it < 400; ++it) {
        const int *sh = shapes[it % 4];
        const int G = sh[0] / sh[1], target = rnd(1650, 1900), decodes = it % 3 ? 0 : rnd(1, 200);
        std::vector<int32_t> qs, ql, cl;
        int64_t T = 0, tiles = 0;
        auto add = [&](int q, int prefix) {
            qs.push_back((int32_t)T);
            ql.push_back(q);
            cl.push_back(prefix + q);
            const int64_t cols = (int64_t)q * G;
            tiles += cols >= 64 ? (cols + sarathi::kTileCols - 1) / sarathi::kTileCols : (cols + sarathi::kWaveCols - 1) / sarathi::kWaveCols;
            T += q;
        };
        for (int i = 0; i < decodes; ++i) add(1, rnd(100, 16000));
        while (tiles < target) add(std::max(1, std::min(rnd(40, 1600), (int)((target - tiles) * sarathi::kTileCols / G))), rnd(0, 2) ? rnd(0, 3000) : rnd(0, 16000));
        const int S = (int)ql.size();
        int max_blocks = 1;
        for (int32_t c : cl) max_blocks = std::max(max_blocks, (c + 15) / 16);
        const sarathi_config cfg{sh[0], sh[1], sh[2], 16, 0, (int32_t)T, S, max_blocks};
        sarathi_handle *h = nullptr;
        CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
        std::vector<int32_t> bt((size_t)S * max_blocks, 0);
        char dummy[16];
        sarathi::g_num_seqs = S;
        sarathi::g_num_tokens = T;
        const bool fits = sarathi::attn_meta_bytes((size_t)tiles, (size_t)tiles, 0) <= sarathi::kStaticMetaBytes;
        const sarathi_status st = sarathi_hybrid_attention_noalloc(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S,
                                                                   (int32_t)T, 1, 0.1f, dummy, nullptr);
        CHECK(st == (fits ? SARATHI_OK : SARATHI_ECAPACITY));
        (fits ? taken : refused)++;
        CHECK(sarathi_destroy(h) == SARATHI_OK);
    }
    CHECK(taken > 200 && refused > 5);
}

// Chunks and decodes that both want to be cut, with the 4096 partial rows that the built-in scratch holds at 8 x 128: the plan is
// one that was looked at, not both cuts doubled until they fit (twice the pieces at least).
static void drive_scarce_partial_rows() {
    struct Batch {
        int32_t hq, hkv, d, max_rows;
        std::vector<int32_t> q_len, ctx_len;
        int32_t longest_decode_piece;
    };
    const Batch batches[] = {{32, 8, 128, 4096, {512, 1, 1}, {4383, 9000, 3000}, 1024},
                             {32, 8, 128, 4096, {512, 1, 1, 1, 1}, {2383, 4000, 3000, 2000, 1000}, 1536},
                             {32, 8, 128, 4096, {512, 1, 1, 1}, {6000, 8000, 3000, 3000}, 2048},
                             {32, 1, 128, 32768, {512, 1, 1}, {4383, 4000, 9000}, 1024}};
    for (const Batch &b : batches) {
        const sarathi_config cfg{b.hq, b.hkv, b.d, 16, 0, 4096, 64, 1024};
        sarathi::WorkspaceLayout ws = sarathi::make_workspace_layout(cfg);
        ws.max_part_rows = b.max_rows;
        std::vector<int32_t> q_start;
        int32_t run = 0;
        for (int32_t q : b.q_len) { q_start.push_back(run); run += q; }
        sarathi::Plan plan;
        sarathi::plan_attention(cfg, sarathi::Options{}, ws, q_start.data(), b.q_len.data(), b.ctx_len.data(), (int32_t)b.q_len.size(), plan);
        CHECK(plan.num_part_rows <= b.max_rows);
        for (const sarathi::TileDesc &t : plan.tiles)
            if (t.kind == sarathi::kKindWave) CHECK(t.keys_per_split <= b.longest_decode_piece);
    }
}

// A launch of decodes alone runs one block per compute unit (padded LDS) unless it was cut into pieces of nearly one length.
static void drive_decode_blocks_per_unit() {
    struct Batch {
        std::vector<int32_t> ctx_len;
        bool cut, one_per_unit;
    };
    const Batch batches[] = {{std::vector<int32_t>(8, 4096), true, false},    // equal pieces
                             {std::vector<int32_t>(60, 300), false, true},    // whole decodes
                             {std::vector<int32_t>(120, 200), true, true}};   // every sixth 3600 keys and cut, the others whole
    for (const Batch &b : batches) {
        std::vector<int32_t> ctx = b.ctx_len;
        if (b.cut && b.one_per_unit)
            for (size_t i = 0; i < ctx.size(); i += 6) ctx[i] = 3600;
        const int32_t S = (int32_t)ctx.size();
        const sarathi_config cfg{16, 2, 128, 16, 0, S, S, 256};
        std::vector<int32_t> q_start((size_t)S), q_len((size_t)S, 1), bt((size_t)S * 256, 0);
        for (int32_t i = 0; i < S; ++i) q_start[(size_t)i] = i;
        sarathi_handle *h = nullptr;
        CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
        sarathi_plan_info info{};
        CHECK(sarathi_plan_hybrid_attention(h, q_start.data(), q_len.data(), ctx.data(), S, S, &info, nullptr, 0) == SARATHI_OK);
        CHECK((info.num_reduce_items > 0) == b.cut);
        char dummy[16];
        sarathi::g_num_seqs = S;
        sarathi::g_num_tokens = S;
        CHECK(sarathi_hybrid_attention_noalloc(h, dummy, dummy, dummy, bt.data(), q_start.data(), q_len.data(), ctx.data(), S, S, 1, 0.1f,
                                               dummy, nullptr) == SARATHI_OK);
        CHECK((sarathi::g_lds_pad_bytes > 0) == b.one_per_unit);
        CHECK(sarathi_destroy(h) == SARATHI_OK);
    }
}

// Allocation-free calls that the host bounds are not cut for the GPU's sake where the units take further launches.  The same batches
// are cut with a workspace; ones that the GPU bounds, and ones whose plan takes no more launches cut than whole, either way
// and alike.
static void drive_host_bound_cuts() {
    struct Batch {
        int32_t hq, hkv, d;
        std::vector<int32_t> q_len, ctx_len;
        bool cut;
    };
    Batch batches[] = {{4, 1, 64, {130}, {130}, false},
                       {32, 8, 128, std::vector<int32_t>(8, 1), {500, 1000, 1500, 2000, 2500, 3000, 3500, 4000}, true},
                       {64, 8, 128, {625, 1, 1}, {912, 3403, 3440}, true},
                       {64, 8, 128, {1}, {1200}, false},   // whole it takes one launch, cut four
                       {32, 8, 128, {1}, {1750}, true},
                       {8, 2, 128, {300, 1, 37, 1, 1, 200}, {1300, 555, 37, 1, 7000, 900}, true}};
    for (int32_t i = 0; i < 54; ++i) {
        batches[0].q_len.push_back(1);
        batches[0].ctx_len.push_back(125 + 69 * i);
    }
    for (const Batch &b : batches) {
        std::vector<int32_t> q_start;
        int32_t run = 0;
        for (int32_t q : b.q_len) { q_start.push_back(run); run += q; }
        const sarathi_config cfg{b.hq, b.hkv, b.d, 16, 0, 1024, 64, 512};
        const sarathi::WorkspaceLayout ws = sarathi::make_workspace_layout(cfg);
        sarathi::WorkspaceLayout in_arguments = ws;
        in_arguments.meta_per_launch = sarathi::kUploadArgBytes;
        sarathi::Plan plan, other;
        sarathi::plan_attention(cfg, sarathi::Options{}, ws, q_start.data(), b.q_len.data(), b.ctx_len.data(), (int32_t)b.q_len.size(), plan);
        sarathi::plan_attention(cfg, sarathi::Options{}, in_arguments, q_start.data(), b.q_len.data(), b.ctx_len.data(), (int32_t)b.q_len.size(), other);
        CHECK(plan.num_split_tiles > 0);
        CHECK((other.num_split_tiles > 0) == b.cut && (other.units == plan.units) == b.cut);
    }
}

// Launches that hand their items out from queues, forced and by the rule, in every way such a batch is launched: the words are zero
// when one starts (cleared by the append, by the attention call itself when it comes a second time, by the allocation-free
// call), the options that change between an append and its attention call included.
static void drive_queues() {
    struct Batch {
        int32_t hq, hkv, d, decodes, low, high;
        std::vector<int32_t> chunks;
        int32_t prefix;
        bool by_rule;
    };
    const Batch batches[] = {{4, 1, 64, 700, 1, 300, {}, 0, false},  {4, 2, 64, 20, 40, 900, {40, 90}, 300, false}, {4, 1, 64, 9, 30, 700, {400, 333}, 500, false},
                             {8, 2, 64, 400, 1, 200, {70, 130}, 40, false}, {8, 2, 64, 30, 100, 900, {4800}, 0, false}, {8, 8, 128, 400, 2048, 2048, {}, 0, true}};
    const int64_t forms[][4] = {{-1, -1, 2, 0}, {1, 0, 2, 0}, {1, -1, 2, 64}, {-1, 1, 2, 64}, {1, 1, 2, 32}, {1, -1, 0, 64}, {1, 1, 1, 64}, {0, 0, 2, 64}};
    int by_rule = 0;
    for (const Batch &b : batches)
        for (const auto &f : forms)
            for (const int one_per_unit : {0, 1}) {
                std::vector<int32_t> qs, ql, cl;
                int32_t T = 0, max_blocks = 1;
                auto add = [&](int32_t q, int32_t ctx) {
                    qs.push_back(T); ql.push_back(q); cl.push_back(ctx);
                    T += q;
                    max_blocks = std::max(max_blocks, (ctx + 15) / 16);
                };
                for (int32_t q : b.chunks) add(q, q + b.prefix);
                for (int32_t i = 0; i < b.decodes; ++i) add(1, b.low + (b.high > b.low ? i * 37 % (b.high - b.low) : 0));
                const int32_t S = (int32_t)ql.size();
                const sarathi_config cfg{b.hq, b.hkv, b.d, 16, 0, T, S, max_blocks};
                sarathi_handle *h = nullptr;
                CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
                const char *names[] = {"item_queue", "resident_chunks", "interleave"};
                for (int o = 0; o < 3; ++o) CHECK(sarathi_set_option(h, names[o], f[o]) == SARATHI_OK);
                CHECK(sarathi_set_option(h, "split_keys", f[3]) == SARATHI_OK && sarathi_set_option(h, "tile_split_keys", f[3]) == SARATHI_OK);
                if (one_per_unit) CHECK(sarathi_set_option(h, "lds_pad_kb", 96) == SARATHI_OK);
                std::vector<int32_t> bt((size_t)S * max_blocks, 0);
                const size_t row = (size_t)b.hkv * b.d;
                std::vector<uint16_t> fresh((size_t)T * row), pool(row * 16);   // every sequence's pages are one page: nothing is computed here
                char dummy[16];
                void *ws = nullptr;
                CHECK(posix_memalign(&ws, 256, sarathi_workspace_bytes(h)) == 0);
                std::memset(ws, 0xFF, sarathi_workspace_bytes(h));
                sarathi::g_num_seqs = S;
                sarathi::g_num_tokens = T;
                sarathi::g_queued_launches = 0;
                auto append = [&] {
                    CHECK(sarathi_kv_append(h, fresh.data(), fresh.data(), pool.data(), pool.data(), bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, ws,
                                            nullptr) == SARATHI_OK);
                };
                auto attend = [&] {
                    CHECK(sarathi_hybrid_attention(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, 0.1f, dummy, ws, nullptr) == SARATHI_OK);
                };
                append();
                attend();
                attend();
                if (b.by_rule && f[0] < 0 && sarathi::g_queued_launches > 0) by_rule++;
                const bool few_chunk_blocks = b.chunks.empty() || b.chunks[0] < 1000;
                if (f[0] == 1 && few_chunk_blocks) CHECK(sarathi::g_queued_launches == 2);
                append();
                append();
                attend();
                if (f[0] == 0) {   // queues that the append did not know of
                    append();
                    CHECK(sarathi_set_option(h, "item_queue", 1) == SARATHI_OK);
                    const int before = sarathi::g_queued_launches;
                    attend();
                    CHECK(sarathi::g_queued_launches == before + (few_chunk_blocks || !one_per_unit ? 1 : 0));
                    CHECK(!one_per_unit || !few_chunk_blocks || sarathi::g_queue_blocks == sarathi::kQueueBlocks / 2);
                }
                for (int rep = 0; rep < 2; ++rep) {
                    const sarathi_status st = sarathi_hybrid_attention_noalloc(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, 0.1f,
                                                                               dummy, nullptr);
                    CHECK(st == SARATHI_OK);
                    attend();
                }
                CHECK(sarathi_destroy(h) == SARATHI_OK);
                std::free(ws);
            }
    CHECK(by_rule > 0);
}

// Which launches of both kinds of tile take their roles at run time: those whose chunk blocks fill every slot next to decodes that take
// long to stream, or one of which is long; not those whose chunk blocks leave slots to the decodes from the start, short
// decodes, or column tiles that share keys.
static void drive_roles_by_rule() {
    struct Batch {
        int32_t hq, hkv, d;
        std::vector<int32_t> chunks, prefixes;
        int32_t decodes, keys;
        bool roles;
    };
    const Batch batches[] = {{64, 8, 128, {512, 512}, {911, 2840}, 1024, 2300, true}, {56, 8, 128, {1024, 512, 384}, {9475, 3210, 11117}, 128, 8700, true},
                             {64, 8, 128, {700, 700}, {800, 100}, 10, 12000, true},   {64, 8, 128, {1919}, {111}, 15, 3800, true},
                             {64, 8, 128, {285, 1984}, {431, 0}, 3, 3241, true},     {56, 8, 128, {1241}, {412}, 20, 3377, true},
                                  {64, 8, 128, {1119}, {1}, 1, 900, false},
                             {32, 8, 128, {1492}, {0}, 52, 4500, false},              {64, 8, 128, {1186}, {584}, 350, 200, false},
                             {58, 2, 64, {1833}, {0}, 678, 5000, false},              {32, 8, 128, {512}, {1871}, 64, 2100, false}};
    for (const Batch &b : batches) {
        std::vector<int32_t> qs, ql, cl;
        int32_t T = 0;
        for (size_t i = 0; i < b.chunks.size(); ++i) { qs.push_back(T); ql.push_back(b.chunks[i]); cl.push_back(b.chunks[i] + b.prefixes[i]); T += b.chunks[i]; }
        for (int32_t i = 0; i < b.decodes; ++i) { qs.push_back(T); ql.push_back(1); cl.push_back(b.keys); T += 1; }
        const int32_t S = (int32_t)ql.size(), blocks = 1024;
        const sarathi_config cfg{b.hq, b.hkv, b.d, 16, 0, T, S, blocks};
        sarathi_handle *h = nullptr;
        CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
        std::vector<int32_t> bt((size_t)S * blocks, 0);
        void *ws = nullptr;
        CHECK(posix_memalign(&ws, 256, sarathi_workspace_bytes(h)) == 0);
        char dummy[16];
        sarathi::g_num_seqs = S;
        sarathi::g_num_tokens = T;
        CHECK(sarathi_hybrid_attention(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, 0.1f, dummy, ws, nullptr) == SARATHI_OK);
        CHECK(sarathi::g_which == (b.roles ? 5 : 4));  // kinds of launch: internal.h
        CHECK(sarathi_destroy(h) == SARATHI_OK);
        std::free(ws);
    }
}

// Which launches of decodes alone hand their items out from queues by the rule: long ones, but not those of nearly one length whose
// third round would fill less than half of the slots.
static void drive_queue_by_rule() {
    struct Batch {
        int32_t decodes, low, high;
        bool queued;
    };
    const Batch batches[] = {{104, 4096, 4096, true}, {136, 4096, 4096, false}, {152, 3000, 4096, false}, {152, 1000, 6000, true},
                             {160, 4096, 4096, false}, {168, 4096, 4096, true}, {300, 4096, 4096, true}, {300, 200, 600, false}, {64, 500, 2000, false}};
    for (const Batch &b : batches) {
        const int32_t S = b.decodes, blocks = 400;
        const sarathi_config cfg{32, 8, 128, 16, 0, S, S, blocks};
        std::vector<int32_t> q_start((size_t)S), q_len((size_t)S, 1), ctx((size_t)S), bt((size_t)S * blocks, 0);
        for (int32_t i = 0; i < S; ++i) {
            q_start[(size_t)i] = i;
            ctx[(size_t)i] = b.low + (int32_t)((int64_t)(b.high - b.low) * i / std::max(1, S - 1));
        }
        sarathi_handle *h = nullptr;
        CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
        char dummy[16];
        sarathi::g_num_seqs = S;
        sarathi::g_num_tokens = S;
        CHECK(sarathi_hybrid_attention_noalloc(h, dummy, dummy, dummy, bt.data(), q_start.data(), q_len.data(), ctx.data(), S, S, 1, 0.1f, dummy,
                                               nullptr) == SARATHI_OK);
        CHECK((sarathi::g_queue_blocks > 0) == b.queued);
        CHECK(sarathi_destroy(h) == SARATHI_OK);
    }
}

// Which allocation-free calls carry their plan in the attention launch's arguments: those whose tiles fit, with nothing cut and no queue.
static void drive_plans_in_arguments() {
    struct Batch {
        int32_t chunk, decodes, keys;
        int64_t queue;
        size_t bytes;   // of tiles and units; 0: in memory
    };
    const Batch batches[] = {{0, 1, 40, -1, 52},      {0, 18, 40, -1, 936},    {0, 19, 40, -1, 988}, {0, 73, 40, -1, 3796}, {0, 74, 40, -1, 0},
                             {300, 60, 40, -1, 3640}, {300, 63, 40, -1, 3796}, {300, 64, 40, -1, 0}, {0, 18, 40, 1, 0},     {0, 2, 7000, -1, 0}};
    for (const Batch &b : batches)
        for (const int64_t interleave : {2, 1, 0}) {
            const int32_t S = b.decodes + (b.chunk > 0), T = b.decodes + b.chunk, blocks = 500;
            const sarathi_config cfg{8, 2, 128, 16, 0, T, S, blocks};
            std::vector<int32_t> qs, ql, cl, bt((size_t)S * blocks, 0);
            if (b.chunk > 0) { qs.push_back(0); ql.push_back(b.chunk); cl.push_back(b.chunk + 40); }
            for (int32_t i = 0; i < b.decodes; ++i) { qs.push_back(b.chunk + i); ql.push_back(1); cl.push_back(b.keys); }
            sarathi_handle *h = nullptr;
            CHECK(sarathi_create(&cfg, &h) == SARATHI_OK);
            CHECK(sarathi_set_option(h, "interleave", interleave) == SARATHI_OK && sarathi_set_option(h, "item_queue", b.queue) == SARATHI_OK);
            char dummy[16];
            void *ws = nullptr;
            CHECK(posix_memalign(&ws, 256, sarathi_workspace_bytes(h)) == 0);
            sarathi::g_num_seqs = S;
            sarathi::g_num_tokens = T;
            CHECK(sarathi_hybrid_attention_noalloc(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, 0.1f, dummy,
                                                   nullptr) == SARATHI_OK);
            CHECK(sarathi::g_plan_bytes == b.bytes);
            CHECK(sarathi_hybrid_attention(h, dummy, dummy, dummy, bt.data(), qs.data(), ql.data(), cl.data(), S, T, 1, 0.1f, dummy, ws, nullptr) == SARATHI_OK);
            CHECK(sarathi::g_plan_bytes == 0);
            CHECK(sarathi_destroy(h) == SARATHI_OK);
            std::free(ws);
        }
}

static void drive_checker() {
    // one chunk on a prefix and two decodes, GQA 4:2, d = 8; every buffer exactly as large as documented
    const int Hq = 4, Hkv = 2, d = 8;
    const int32_t q_start[3] = {0, 5, 6}, q_len[3] = {5, 1, 1}, ctx_len[3] = {9, 1, 13};
    const int64_t kv_start[3] = {0, 9, 10};
    const int T = 7, KV = 23;
    std::vector<uint16_t> q((size_t)T * Hq * d), k((size_t)KV * Hkv * d), v(k.size());
    for (size_t i = 0; i < q.size(); ++i) q[i] = (uint16_t)(0x3F80 + (i * 37 % 64));          // bf16 values near 1
    for (size_t i = 0; i < k.size(); ++i) { k[i] = (uint16_t)(0x3F00 + (i * 29 % 128)); v[i] = (uint16_t)(0xBF80 + (i * 13 % 96)); }
    std::vector<double> out((size_t)T * Hq * d);
    for (int window : {0, 1, 4})
        CHECK(oracle_hybrid_attention_window(q.data(), k.data(), v.data(), kv_start, q_start, q_len, ctx_len, 3, T, Hq, Hkv, d, 0.35,
                                             window, nullptr, T, out.data(), 2) == 0);
    const int32_t rows[2] = {6, 0};
    std::vector<double> two((size_t)2 * Hq * d);
    CHECK(oracle_hybrid_attention_window(q.data(), k.data(), v.data(), kv_start, q_start, q_len, ctx_len, 3, T, Hq, Hkv, d, 0.35, 0, rows,
                                         2, two.data(), 1) == 0);
    std::vector<double> w(13);
    CHECK(oracle_softmax_weights(q.data(), k.data(), kv_start, q_start, q_len, ctx_len, 3, Hq, Hkv, d, 0.35, 6, 3, w.data()) == 13);
    double sum = 0;
    for (double x : w) sum += x;
    CHECK(sum > 0.999999 && sum < 1.000001);
    const int32_t bad_rows[1] = {7};
    CHECK(oracle_hybrid_attention_window(q.data(), k.data(), v.data(), kv_start, q_start, q_len, ctx_len, 3, T, Hq, Hkv, d, 0.35, 0,
                                         bad_rows, 1, two.data(), 1) != 0);
    // linear layer: 3 x 5 by 4 x 5, all and a subset
    std::vector<uint16_t> x(15, 0x3F80), wt(20, 0x4000);
    std::vector<double> y(12);
    CHECK(oracle_linear(x.data(), wt.data(), 3, 4, 5, nullptr, 0, nullptr, 0, y.data(), 1) == 0 && y[11] == 10.0);
    const int32_t r[1] = {2}, c[2] = {3, 0};
    CHECK(oracle_linear(x.data(), wt.data(), 3, 4, 5, r, 1, c, 2, y.data(), 2) == 0 && y[1] == 10.0);
    const int32_t bad[1] = {4};
    CHECK(oracle_linear(x.data(), wt.data(), 3, 4, 5, nullptr, 0, bad, 1, y.data(), 1) != 0);
}

int main() {
    std::mt19937_64 rng(20240302);
    drive_scheduler(rng);
    drive_attention_host_paths(rng);
    drive_built_in_scratch_limits(rng);
    drive_scarce_partial_rows();
    drive_decode_blocks_per_unit();
    drive_host_bound_cuts();
    drive_queues();
    drive_roles_by_rule();
    drive_queue_by_rule();
    drive_plans_in_arguments();
    drive_checker();
    std::printf("host paths clean (sink %llu)\n", (unsigned long long)sarathi::g_sink);
    return 0;
}
