// Host side of sarathi_hybrid_attention: validation of the batch description, workspace
// layout, and the decomposition of one iteration's attention into independent work items.
//
// Decomposition.  For a KV head, the query side of sequence s is a list of COLUMNS,
// col = row*G + head_in_group (G = Hq/Hkv query heads share the KV head, paper section 2.2),
// so a decode has G columns and a chunk of c rows has c*G.  Columns are cut into tiles of 16
// (the N dimension of the 16x16x32 matrix-core instruction); a tile needs keys
// 0 .. position of its last row.  Long key ranges are cut into splits of about `split_keys`
// keys so that (a) a decode with a long context (paper section 3.3: decode cost grows with
// the accumulated context and differs across requests) does not become the tail of the
// launch and (b) there are enough units to fill 256 compute units.  Chunks with at least
// tile_min_cols columns use 128-column tiles instead (K/V staged once per tile in LDS).  The
// splits of a tile are merged in index order by a second, small kernel.
#include <algorithm>
#include <cstdio>
#include <utility>

#include "internal.h"

namespace sarathi {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

constexpr int32_t kMaxSplitUnits = 8192;
constexpr int32_t kMaxPartRows = 32768;
constexpr int32_t kMinWaveKeys = 1024;   // automatic choice: keys per wavefront of a wave-tile block before the tile is split
constexpr int32_t kMinTileSplitKeys = 1024;  // next to decodes
constexpr int32_t kChunkMinCols = 64;        // automatic choice: sequences with fewer columns run as wave tiles in any batch

WorkspaceLayout make_workspace_layout(const sarathi_config &cfg) {
    WorkspaceLayout w{};
    const int64_t G = cfg.num_q_heads / cfg.num_kv_heads;
    // wave tiles only exist for sequences below tile_min_cols columns; bounding every sequence by
    // 16-column tiles covers both kinds
    const int64_t max_tiles = ceil_div((int64_t)cfg.max_tokens * G, kWaveCols) + cfg.max_seqs;
    w.max_tiles = (int32_t)std::min<int64_t>(max_tiles, INT32_MAX / 64);
    w.max_units = (int32_t)std::min<int64_t>(max_tiles + kMaxSplitUnits, INT32_MAX / 64);
    w.max_part_rows = kMaxPartRows;
    // a split tile has at least 2 pieces of n_cols rows: sum over split tiles of ceil(n_cols/8) <= rows/16 + tiles
    w.max_reduce_units = (int32_t)std::min<int64_t>(kMaxPartRows / (2 * kReduceCols) + kMaxSplitUnits / 2, INT32_MAX / 64);
    const size_t attn_meta = sizeof(TileDesc) * (size_t)w.max_tiles +
                             sizeof(uint32_t) * ((size_t)w.max_units + (size_t)w.max_reduce_units) + 64;
    w.max_attn_meta = attn_meta;
    const size_t append_meta = sizeof(AppendUnit) * (size_t)max_append_units(cfg) + 64;
    size_t off = 0;
    w.meta = off;
    w.meta_bytes = align_up(align_up(append_meta, 256) + attn_meta, 256);  // an append may carry both
    off += w.meta_bytes;
    w.sched = off;     off = align_up(off + kSchedBytes, 256);
    w.part_ml = off;   off = align_up(off + sizeof(float) * 2 * (size_t)w.max_part_rows * cfg.num_kv_heads, 256);
    w.part_o = off;    off = align_up(off + sizeof(float) * (size_t)w.max_part_rows * cfg.num_kv_heads * cfg.head_dim, 256);
    w.total = off;
    return w;
}

sarathi_status validate_batch(const sarathi_config &cfg, const int32_t *q_start, const int32_t *q_len,
                              const int32_t *ctx_len, int32_t num_seqs, int32_t num_tokens,
                              int64_t num_pages, std::string &err) {
    char buf[160];
    if (num_seqs < 0 || num_tokens < 0) { err = "negative num_seqs or num_tokens"; return SARATHI_EINVAL; }
    if (num_seqs == 0) {
        if (num_tokens != 0) { err = "num_tokens != 0 with num_seqs == 0"; return SARATHI_EINVAL; }
        return SARATHI_OK;
    }
    if (!q_start || !q_len || !ctx_len) { err = "null length array"; return SARATHI_EINVAL; }
    if (num_seqs > cfg.max_seqs) { err = "num_seqs exceeds max_seqs"; return SARATHI_ECAPACITY; }
    if (num_tokens > cfg.max_tokens) { err = "num_tokens exceeds max_tokens"; return SARATHI_ECAPACITY; }
    if (num_pages < 1) { err = "num_pages < 1"; return SARATHI_EINVAL; }
    int64_t run = 0;
    for (int32_t s = 0; s < num_seqs; ++s) {
        if (q_len[s] < 1 || ctx_len[s] < q_len[s]) {
            snprintf(buf, sizeof buf, "sequence %d: need 1 <= q_len <= ctx_len (q_len %d, ctx_len %d)", s, q_len[s], ctx_len[s]);
            err = buf;
            return SARATHI_EINVAL;
        }
        if (q_start[s] != run) {
            snprintf(buf, sizeof buf, "sequence %d: q_start %d is not the prefix sum of q_len (%lld)", s, q_start[s], (long long)run);
            err = buf;
            return SARATHI_EINVAL;
        }
        if (ceil_div(ctx_len[s], cfg.page_size) > cfg.max_blocks_per_seq) {
            snprintf(buf, sizeof buf, "sequence %d: ctx_len %d needs more than max_blocks_per_seq pages", s, ctx_len[s]);
            err = buf;
            return SARATHI_ECAPACITY;
        }
        run += q_len[s];
    }
    if (run != num_tokens) { err = "sum of q_len != num_tokens"; return SARATHI_EINVAL; }
    return SARATHI_OK;
}

namespace {

inline int32_t steps_of_split(const TileDesc &t, int32_t split) {
    const int32_t b = t.key_lo + split * t.keys_per_split;
    const int32_t e = std::min(t.n_keys, b + t.keys_per_split);
    return (int32_t)ceil_div(e - b, kTileKeys);
}

// Chooses the split of every tile in [first, last) for `split_keys` (spans of up to `whole_keys` stay uncut), assigns partial rows and
// counters, and appends the units sorted longest first (counting sort on 32-key steps).
void emit_units(Plan &plan, size_t first, size_t last, int64_t split_keys, int64_t whole_keys, std::vector<uint32_t> &scratch,
                std::vector<int32_t> &bucket) {
    scratch.clear();
    int32_t max_steps = 0;
    for (size_t ti = first; ti < last; ++ti) {
        TileDesc &t = plan.tiles[ti];
        const int64_t span = t.n_keys - t.key_lo;  // keys the tile reads
        int32_t ns = (span <= std::max(split_keys + split_keys / 2, whole_keys)) ? 1 : (int32_t)ceil_div(span, split_keys);
        t.keys_per_split = (int32_t)(ceil_div(ceil_div(span, ns), kTileKeys) * kTileKeys);
        t.n_splits = (int32_t)ceil_div(span, t.keys_per_split);
        if (t.n_splits > 1) {
            t.part_row0 = plan.num_part_rows;
            plan.num_part_rows += t.n_splits * t.n_cols;
            plan.num_split_tiles++;
            plan.most_pieces = std::max(plan.most_pieces, t.n_splits);
            for (int32_t c0 = 0, grp = 0; c0 < t.n_cols; c0 += kReduceCols, ++grp)
                plan.reduce_units.push_back(pack_unit((uint32_t)ti, (uint32_t)grp));
        } else {
            t.part_row0 = -1;
        }
        for (int32_t i = 0; i < t.n_splits; ++i) {
            scratch.push_back(pack_unit((uint32_t)ti, (uint32_t)i));
            max_steps = std::max(max_steps, steps_of_split(t, i));
        }
    }
    auto steps = [&](uint32_t u) {
        return steps_of_split(plan.tiles[u & ((1u << kUnitTileBits) - 1)], (int32_t)(u >> kUnitTileBits));
    };
    bucket.assign((size_t)max_steps + 2, 0);
    for (uint32_t u : scratch) bucket[(size_t)(max_steps - steps(u)) + 1]++;
    for (size_t i = 1; i < bucket.size(); ++i) bucket[i] += bucket[i - 1];
    const size_t base = plan.units.size();
    plan.units.resize(base + scratch.size());
    for (uint32_t u : scratch) plan.units[base + (size_t)bucket[(size_t)(max_steps - steps(u))]++] = u;
}

// Column tiles of one sequence (more than 16 columns in a wave tile's sequence: many heads per KV head, or a few rows) read
// the same keys, from memory once if they run at about the same time behind the same L2.  Block % 8 picks the XCD and a
// unit is num_kv_heads blocks, so with 8 / gcd units between them they meet there: the wave units from `base` on are
// re-ordered in windows of that many sequence pieces, first the first column tile of each, then the second, and so on.
// (29 heads per KV head, two KV heads of 64 channels: 512 decodes of 256-4096 keys 189 -> 167 us, 200 of 1024-8192 keys
// 167 -> 137; 32 heads per KV head, two of 128 channels: 128 decodes 100 -> 87.)
void pair_column_tiles(Plan &plan, size_t base, int32_t num_kv_heads, std::vector<uint32_t> &scratch) {
    int64_t apart = 8;
    while (apart > 1 && (apart / 2) * num_kv_heads % 8 == 0) apart /= 2;
    if (apart == 1) return;  // neighbours meet anyway
    constexpr uint32_t kTileMask = (1u << kUnitTileBits) - 1;
    auto tile_of = [&](uint32_t u) -> const TileDesc & { return plan.tiles[u & kTileMask]; };
    bool several = false;
    for (size_t i = base; i < plan.units.size(); ++i) several |= tile_of(plan.units[i]).col_begin > 0;
    if (!several) return;
    scratch.assign(plan.units.begin() + (ptrdiff_t)base, plan.units.end());
    size_t out = base;
    std::vector<uint32_t> window;  // pieces of first column tiles
    auto flush = [&]() {
        bool any = !window.empty();
        for (uint32_t c = 0; any; ++c) {
            any = false;
            for (uint32_t u : window) {
                const uint32_t t = (u & kTileMask) + c, split = u >> kUnitTileBits;
                if (t >= plan.tiles.size() || plan.tiles[t].seq != tile_of(u).seq || plan.tiles[t].kind != kKindWave) continue;
                any = true;
                if ((int32_t)split < plan.tiles[t].n_splits) plan.units[out++] = pack_unit(t, split);
            }
        }
        window.clear();
    };
    for (uint32_t u : scratch)
        if (tile_of(u).col_begin == 0) {
            window.push_back(u);
            if ((int64_t)window.size() == apart) flush();
        }
    flush();
    for (uint32_t u : scratch) {  // pieces that the first column tile of their sequence does not have
        const TileDesc &t = tile_of(u);
        const TileDesc &first = plan.tiles[(u & kTileMask) - (uint32_t)(t.col_begin / kWaveCols)];
        if ((int32_t)(u >> kUnitTileBits) >= first.n_splits) plan.units[out++] = u;
    }
}

// What a choice of split_keys would need for tiles [first, last).
struct SplitCount {
    int64_t units = 0;         // pieces of the split tiles
    int64_t rows = 0;          // partial rows
    int64_t tiles = 0;         // split tiles
    int64_t reduce_units = 0;  // merge units
};
SplitCount count_splits(const Plan &plan, size_t first, size_t last, int64_t split_keys, int64_t whole_keys) {
    SplitCount c;
    for (size_t ti = first; ti < last; ++ti) {
        const TileDesc &t = plan.tiles[ti];
        const int64_t span = t.n_keys - t.key_lo;
        if (span <= std::max(split_keys + split_keys / 2, whole_keys)) continue;
        const int64_t ns = ceil_div(span, split_keys);
        c.units += ns;
        c.rows += ns * t.n_cols;
        c.tiles++;
        c.reduce_units += ceil_div(t.n_cols, kReduceCols);
    }
    return c;
}

// Estimated time of a launch of chunk tiles alone whose keys are cut at `split_keys`, merge included, in microseconds; a
// huge number if the cut does not fit the partial rows.  The launch is played through: units longest first over
// 256 / Hkv groups of compute units (the KV heads of a unit start next to each other) with two block slots each.  From
// measurements on this part: a block advances 32 keys in 0.62 us alone on its unit and in 0.92 us next to a second block
// (0.72 of that with 64 channels), costs 1.2 us besides, the launch 5 us; a cut launch pays 2 us + 0.4 of the time its partial
// rows take to merge for writing them, and the merge 5 us + 0.25 per piece + the rows twice at 5.5 TB/s.
// Against 340 timings (36 batches of 1 to 4 chunks of 17-8192 tokens behind 0-12,117 keys, ten cuts each) the cheapest
// cut by this estimate is 1 % slower than the best one.  The rules it replaces (0.42 of a block slot's share of the keys
// from 512 blocks on, else rounds of average pieces) were 8 % off: 2048 tokens of two prompts, 64 heads: 159 + 17 us cut
// into 1784 pieces, 140 us whole.
// The estimate is asked for up to sixteen cuts before the launch can be enqueued, so it is kept short: tiles of equal length are
// looked at together; a cut is not played through if all slots busy to the end, or its longest piece, already cost `limit`
// (the best cut so far); and where a KV head's units run on more than 32 groups, every m-th unit is played on an m-th of
// the groups (the longest of each m, so that a few long ones tell).  Planned, on the host, with every cut played in full, now,
// and with the older rules: 58 and 2 heads, 2000 tokens of three prompts 117, 21, 13 us; 71 heads and one, 8192 tokens 470,
// 109, 90; 64 and 8 heads, 8192 tokens 35, 21, 11; 600 random batches 12.0, 7.1, 5.6 on average.
struct ChunkBin {  // tiles of equal length
    int32_t steps, tiles;
    int64_t cols;
};
double chunk_launch_us(const sarathi_config &cfg, const std::vector<ChunkBin> &bins, int64_t split_keys, int64_t max_rows, double limit) {
    static thread_local std::vector<std::pair<int32_t, int32_t>> cuts;    // (steps of a piece, pieces) of the bins' tiles
    static thread_local std::vector<int32_t> count;                       // units by steps
    static thread_local std::vector<std::pair<double, double>> busy;      // heap: (when the group's first slot falls free, steps its other block then has left)
    const double scale = cfg.head_dim == 128 ? 1.0 : 0.72;
    const double alone = 0.62 * scale, shared = 0.92 * scale, fixed_steps = 1.2 / alone;
    const int32_t split_steps = (int32_t)std::min<int64_t>(split_keys / kTileKeys, INT32_MAX / 2);
    int32_t max_steps = 0, most = 1;
    int64_t rows = 0, units = 0, steps = 0;
    cuts.clear();
    for (const ChunkBin &b : bins) {
        int32_t piece = b.steps, n = 1;
        if (b.steps > split_steps + split_steps / 2) {
            n = (b.steps - 1) / split_steps + 1;
            piece = (b.steps - 1) / n + 1;
            n = (b.steps - 1) / piece + 1;
            rows += n * b.cols;
            most = std::max(most, n);
        }
        max_steps = std::max(max_steps, piece);
        units += (int64_t)n * b.tiles;
        steps += (int64_t)b.steps * b.tiles;
        cuts.emplace_back(piece, n);
    }
    if (rows > max_rows) return 1.0e12;
    double c = 5.0;
    if (most > 1) {
        const double move_us = 2.0 * (double)rows * cfg.num_kv_heads * (cfg.head_dim + 2) * 4.0 / 5.5e6;
        c += 2.0 + 0.4 * move_us + 5.0 + 0.25 * (double)most + move_us;
    }
    const int64_t all_groups = std::max(1, 256 / cfg.num_kv_heads);
    const double at_least = std::max(shared / 2.0 * ((double)steps + fixed_steps * (double)units) / (double)all_groups, alone * (max_steps + fixed_steps));
    if (c + at_least >= limit) return c + at_least;

    count.assign((size_t)max_steps + 1, 0);
    for (size_t i = 0; i < bins.size(); ++i) {
        const auto [piece, n] = cuts[i];
        count[(size_t)piece] += (n - 1) * bins[i].tiles;
        count[(size_t)(bins[i].steps - (n - 1) * piece)] += bins[i].tiles;
    }
    const int64_t every = std::max<int64_t>(1, std::min(all_groups / 32, units / 128));
    const size_t groups = (size_t)(all_groups / every);
    busy.clear();
    size_t started = 0;
    int64_t seen = every - 1;  // the longest unit of each m
    auto earlier = [](const std::pair<double, double> &x, const std::pair<double, double> &y) { return y < x; };  // of groups free at the same time the one with less left
    for (int32_t st = max_steps; st > 0; --st) {
        seen += count[(size_t)st];
        for (; seen >= every; seen -= every) {
            const double u = (double)st + fixed_steps;
            if (started < groups) {
                busy.emplace_back(0.0, u);                                // alone so far
            } else if (started < 2 * groups) {                            // second slots, next to the longest units first
                auto &g = busy[started - groups];
                const double both = std::min(u, g.second);
                g = {shared * both, std::max(u, g.second) - both};
                if (started + 1 == 2 * groups) std::make_heap(busy.begin(), busy.end(), earlier);
            } else {                                                      // the first group to fall free, moved down to its new place
                const double both = std::min(u, busy[0].second);
                const std::pair<double, double> g = {busy[0].first + shared * both, std::max(u, busy[0].second) - both};
                if (c + g.first >= limit) return c + g.first;
                size_t at = 0;
                for (size_t child; (child = 2 * at + 1) < groups; at = child) {
                    if (child + 1 < groups && busy[child + 1] < busy[child]) ++child;
                    if (!(busy[child] < g)) break;
                    busy[at] = busy[child];
                }
                busy[at] = g;
            }
            ++started;
        }
    }
    double end = 0.0;
    for (const auto &g : busy) end = std::max(end, g.first + alone * g.second);
    return c + end;
}

// Where the plan travels in kernel arguments: how many launches it takes, and for how many microseconds an iteration keeps the
// host.  From calls that the host bounded when it took 26 us for a few tiles, 38 for 59 tiles in 264 pieces (two launches for the plan and a
// merge).  Marshalled natively they keep it 12 to 14 us less, and a whole plan of one launch travels with the attention launch: the line is
// too high on both sides and has not been drawn anew.
struct ArgumentLaunches {
    int64_t launches;
    double host_us;
};
ArgumentLaunches argument_launches(const WorkspaceLayout &ws, size_t tiles, const SplitCount &chunk, const SplitCount &wave) {
    const int64_t units = (int64_t)tiles - chunk.tiles - wave.tiles + chunk.units + wave.units, reduce = chunk.reduce_units + wave.reduce_units;
    const int64_t launches = ceil_div((int64_t)attn_meta_bytes(tiles, (size_t)units, (size_t)reduce), (int64_t)ws.meta_per_launch);
    return {launches, 22.5 + 3.2 * (double)launches + 0.015 * (double)units + (reduce > 0 ? 3.5 : 0.0)};
}

// The cut of a batch's chunk tiles that chunk_launch_us finds cheapest within `max_rows` partial rows, in keys per piece (the longest
// tile's keys: whole).  Pieces of fewer than eight key steps are all prologue, and the search ends where finer cuts have cost
// more twice in a row.
struct ChunkCut {
    int64_t keys;          // per piece
    double us, whole_us;   // of the launch by the estimate, cut and whole
};
const std::vector<ChunkBin> &chunk_bins(const Plan &plan, size_t n_chunk_tiles, int64_t longest_span) {
    static thread_local std::vector<ChunkBin> by_steps, bins;
    by_steps.assign((size_t)ceil_div(longest_span, kTileKeys) + 1, ChunkBin{0, 0, 0});
    for (size_t ti = 0; ti < n_chunk_tiles; ++ti) {
        ChunkBin &b = by_steps[(size_t)((uint32_t)(plan.tiles[ti].n_keys - plan.tiles[ti].key_lo + kTileKeys - 1) / kTileKeys)];
        b.tiles++;
        b.cols += plan.tiles[ti].n_cols;
    }
    bins.clear();
    for (size_t st = 1; st < by_steps.size(); ++st)
        if (by_steps[st].tiles > 0) bins.push_back(ChunkBin{(int32_t)st, by_steps[st].tiles, by_steps[st].cols});
    return bins;
}
ChunkCut cheapest_chunk_cut(const sarathi_config &cfg, const Plan &plan, size_t n_chunk_tiles, int64_t chunk_keys, int64_t longest_span, int64_t max_rows) {
    ChunkCut cut{ceil_div(longest_span, kTileKeys) * kTileKeys, 0.0, 0.0};
    const std::vector<ChunkBin> &bins = chunk_bins(plan, n_chunk_tiles, longest_span);
    // Where whole tiles all run at once a cut has to promise 5 %: 578 tokens behind 10,320 of a 4096-key window and
    // 231 more, 64 heads, promise 0.5 % in 1008 pieces instead of 416 blocks and run 3.5 % slower (106.5 us a call
    // whole, 110.2 cut).  Beyond one round it may cost 2 % more: 1024, 512 and 384 tokens behind 10,801, 8,115 and
    // 2,739, 56 heads, are estimated alike whole and in halves and run 3 % faster in halves (840 blocks 504 us, 1288
    // blocks 477 + 15); of 9 timed batches of several rounds none is cut for the worse by this.
    const bool one_round = (int64_t)n_chunk_tiles * cfg.num_kv_heads <= 512;
    const double whole_us = chunk_launch_us(cfg, bins, cut.keys, max_rows, 1.0e12);
    cut.us = cut.whole_us = whole_us;
    double best = one_round ? whole_us : 1.02 * whole_us;
    // all slots busy to the end: no cut can gain what its merge costs
    const double full_us = (double)chunk_keys / kTileKeys * cfg.num_kv_heads * (cfg.head_dim == 128 ? 0.92 : 0.66) / 512.0;
    int worse = whole_us < full_us + 15.0 ? 2 : 0;
    for (int64_t n = 2; n <= 16 && longest_span / n >= 256 && worse < 2; ++n) {
        const int64_t keys = ceil_div(ceil_div(longest_span, n), kTileKeys) * kTileKeys;
        const double c = chunk_launch_us(cfg, bins, keys, max_rows, best);
        if (c < best) {
            best = c;
            worse = 0;
            if (!one_round || c < 0.95 * whole_us) {
                cut.keys = keys;
                cut.us = c;
            }
        } else {
            ++worse;
        }
    }
    return cut;
}

// Chunk tiles next to decodes: estimated microseconds of the launch and its merge with the chunks' keys cut at `split_keys`.  From
// timings of 290 batches (1 to 3 chunks of 64-1024 tokens behind 0-12,288 keys next to 1-600 decodes of up to 16,384 keys,
// five head shapes, seven cuts each; the estimate errs by 10 % rms):
//   the decodes take 2.3 + the larger of (their bytes at 6.5 TB/s, the longest block's at 68 GB/s) + a quarter of the
//   smaller + 0.15 of the chunks' work spread over the compute units (68 is what fits these launches; cheapest_wave_cut keeps
//   the 40 of its own fit, which chooses as well);
//   a chunk block takes 0.91 us per 32-key step next to a decode block and 0.55 once they have ended, between that and 0.67 and
//   0.76 where there are 256 to 512 chunk blocks, and 1.4 steps besides (0.69 of all that with 64 channels); beyond
//   512 blocks, or one per compute unit where blocks take roles, the launch is as long as the work dealt out evenly + 0.55 of
//   the longest block; decodes that wait for slots of chunk blocks add up to 0.38 of the chunks' time;
//   together: 7.1 + the longer of the two + 0.04 of the shorter + for a merge 2.5 + the partial rows twice at 3.4 TB/s.
struct HybridBatch {
    double wave_us;       // all decode keys at 6.5 TB/s
    double wave_block_us; // the longest decode block's
    int64_t wave_blocks;
    bool shared;          // most keys are read by several wave tiles
};
double hybrid_launch_us(const sarathi_config &cfg, const std::vector<ChunkBin> &bins, const HybridBatch &b, int64_t split_keys, int64_t max_rows) {
    const double scale = cfg.head_dim == 128 ? 1.0 : 0.69;
    const int32_t split_steps = (int32_t)std::min<int64_t>(split_keys / kTileKeys, INT32_MAX / 2);
    int64_t units = 0, steps = 0, longest = 0, rows = 0;
    for (const ChunkBin &t : bins) {
        int32_t piece = t.steps, n = 1;
        if (t.steps > split_steps + split_steps / 2) {
            n = (t.steps - 1) / split_steps + 1;
            piece = (t.steps - 1) / n + 1;
            n = (t.steps - 1) / piece + 1;
            rows += n * t.cols;
        }
        longest = std::max<int64_t>(longest, piece);
        units += (int64_t)n * t.tiles;
        steps += (int64_t)t.steps * t.tiles;
    }
    if (rows > max_rows) return 1.0e12;
    const int64_t blocks = units * cfg.num_kv_heads;
    const double work = ((double)steps + 1.37 * (double)units) * cfg.num_kv_heads, block_steps = (double)longest + 1.37;
    double decode_us = 2.3 + std::max(b.wave_us, b.wave_block_us) + 0.25 * std::min(b.wave_us, b.wave_block_us);
    decode_us += 0.15 * std::min(work / 256.0 * scale, decode_us);
    auto two_phases = [&](double x, double next_to_decodes, double after) {
        const double us = x * next_to_decodes * scale;
        return us <= decode_us ? us : decode_us + (us - decode_us) / next_to_decodes * after;
    };
    double chunk_us;
    const bool roles = roles_pay(blocks, b.wave_blocks, b.wave_us, b.wave_block_us * (68.0e3 / kNextToChunks), b.shared);
    if (roles) {
        chunk_us = std::max(two_phases(block_steps, 0.91, 0.76), two_phases(work / 256.0, 0.91, 0.38) + 0.55 * 0.76 * scale * block_steps);
    } else if (blocks <= 512) {
        const double second = std::max(0.0, (double)(blocks - 256) / 256.0);
        chunk_us = two_phases(block_steps, 0.91 - 0.24 * second, 0.55 + 0.21 * second);
        if (blocks + b.wave_blocks > 512) decode_us += 0.38 * second * std::min(chunk_us, decode_us);
    } else {
        chunk_us = std::max(two_phases(block_steps, 0.67, 0.76), (work / 512.0 + 0.55 * block_steps) * 0.76 * scale);
        decode_us += 0.38 * std::min(chunk_us, decode_us);
    }
    double us = 7.1 + std::max(chunk_us, decode_us) + 0.04 * std::min(chunk_us, decode_us);
    if (rows > 0) us += 2.5 + 2.0 * (double)rows * cfg.num_kv_heads * (cfg.head_dim + 2) * 4.0 / 3.4e6;
    return us;
}

// Few decodes.  Uncut, a batch's wave blocks (tiles x KV heads) leave compute units idle or finish with the longest
// decode streaming alone, and one block pulls 40 GB/s at most where the chip streams 6,550.  Up to 512 blocks (two per
// compute unit, all resident at once) the keys per piece therefore come from an estimate, in microseconds, of
//   decodes: the larger of (all keys at the chip's rate, the longest piece at a block's) + a quarter of the smaller
//            + 3, and 2 for every further 512 blocks;
//   with prefill chunks in the launch: the longer of decodes and chunks + 0.3 of the shorter (they share the units);
//   merge, if anything is cut: 5.3 + 0.25 per piece of the tile with the most + its partial rows twice at 4.5 TB/s.
// Against timings of 20 decode-only and 17 hybrid batches (1 to 64 decodes of 256 to 32,768 keys, seven pieces each):
// the chosen piece is within 5 % of the best one at the median and 1.9 x (decodes only) and 1.17 x (hybrid) faster than
// whole decodes on average; 8 decodes of 256-4096 keys: 53 -> 19 + 6 us.  A cut has to promise 5 %, and
// below 18 us (28 next to chunk tiles) nothing is cut: the merge is one launch more, 3 us a pass (us a pass, whole and cut: a decode of
// 3072 keys of 64 channels 20.0 and 13.8, of 2048, estimated at 16, 15.3 and 13.9, of 1536 13.0 and 14.0; of 1536 of 128 channels, 22.7, 16.5
// and 14.1, of 1024, 16.2, 12.9 and 13.7; next to 191 tokens two of 1293, 56 and 8 heads, 16.3 and 19.2).  From 18 to 28 us the host decides:
// it is done with an iteration whose decodes are cut after 12.8 us and 0.03 for each of their tiles, in an allocation-free call, where the
// cut also costs the launches that put the plan into memory, after 15.8 us and 0.09, and whole they take 0.85 and 0.8 of the estimate (us a
// pass, whole and cut: 4 heads and one of 64 channels, 168 decodes 21.9 and 18.3, 212 18.5 and 21.8, 348 18.5 and 24.3; allocation-free one
// decode of 32 and 8 heads estimated at 19.7 14.9 and 15.9, at 26.9 18.3 and 15.0; 50 tiles of 64 channels at 18.8 17.4 and 20.3.  The dearest of
// 330 drawn batches: 39 decodes of 32 and 8 heads at 23.8, allocation-free, stay whole, 20.6 and 18.3).
// Fitted when a block pulled 40 GB/s alone; now that its loads go through LDS it pulls about 55, and the estimate fitted to that
// chose no better (120 batches of few decodes 1.001 x, 110 hybrid ones 0.999 x).
// Where one decode holds half of the keys or more, a plan that cuts it finer and leaves all of up to half its length whole
// is tried first and taken if it promises the 5 %, as such batches always were (7000 and 3000 keys next to three short
// ones then end with the 3000-key block, at 42 us).  Where it does not the general search follows: 14,000, 7000 and 6500
// keys 54 + 6 us in pieces of 4096, 23 + 6 in pieces of 1024; 16,000 keys next to three times 4000 60 + 6 and 23 + 6.
struct WaveCut {
    int64_t keys;   // per piece
    int64_t whole;  // spans of up to this many keys stay uncut
    bool few;       // chosen by the estimate
    double us, as_is_us;  // of the launch and its merge by the estimate, cut so and by the rule for many decodes
};
WaveCut cheapest_wave_cut(const sarathi_config &cfg, const Plan &plan, size_t n_chunk_tiles, int64_t wave_keys, int64_t tile_split, int64_t wave_split,
                          int64_t max_rows, bool chunks_made_do, bool plan_in_arguments) {
    const int64_t n_wave_tiles = (int64_t)(plan.tiles.size() - n_chunk_tiles);
    const double key_us = cfg.head_dim * 4.0;  // bytes of a key and its value, one KV head
    double chunk_steps = 0.0;
    int64_t chunk_blocks = 0;
    bool chunk_cut = false;
    if (n_chunk_tiles > 0) {
        int64_t steps = 0, longest = 0, chunk_units = 0;
        for (size_t ti = 0; ti < n_chunk_tiles; ++ti) {
            const int64_t span = plan.tiles[ti].n_keys - plan.tiles[ti].key_lo;
            const int64_t ns = span <= tile_split + tile_split / 2 ? 1 : ceil_div(span, tile_split);
            const int64_t piece = ceil_div(ceil_div(span, ns), kTileKeys);
            steps += ceil_div(span, kTileKeys) + ns;
            longest = std::max(longest, piece + 1);
            chunk_units += ns;
            chunk_cut |= ns > 1;
        }
        chunk_blocks = chunk_units;
        chunk_steps = std::max((double)longest, (double)steps * cfg.num_kv_heads / 512.0);
    }
    const double stream_us = (double)wave_keys * cfg.num_kv_heads * key_us / 6.55e6;
    int64_t longest_wave = 0;
    for (size_t ti = n_chunk_tiles; ti < plan.tiles.size(); ++ti)
        longest_wave = std::max<int64_t>(longest_wave, plan.tiles[ti].n_keys - plan.tiles[ti].key_lo);
    const int64_t whole = 2 * longest_wave >= wave_keys ? longest_wave / 2 : 0;
    auto estimate = [&](int32_t keys, int64_t uncut) {
        int64_t longest = 0, pieces = 0, rows = 0, most = 1;
        for (size_t ti = n_chunk_tiles; ti < plan.tiles.size(); ++ti) {
            const int32_t span = plan.tiles[ti].n_keys - plan.tiles[ti].key_lo;
            if (span <= std::max<int64_t>(keys + keys / 2, uncut)) {
                longest = std::max<int64_t>(longest, span);
                pieces += 1;
            } else {
                const int32_t ns = (span - 1) / keys + 1;
                longest = std::max<int64_t>(longest, keys);
                pieces += ns;
                rows += ns * plan.tiles[ti].n_cols;
                most = std::max<int64_t>(most, ns);
            }
        }
        const double block_us = (double)longest * key_us / 40.0e3;
        const double decode_us = 3.0 + std::max(stream_us, block_us) + 0.25 * std::min(stream_us, block_us) +
                                 2.0 * (double)((pieces * cfg.num_kv_heads - 1) / 512);
        if (rows > max_rows && most > 1) return 1.0e12;
        // whole chunk tiles that were to be cut are the launch's tail: pieces that push a second block onto their units tell
        const int64_t blocks = (chunk_blocks + (chunks_made_do ? pieces : n_wave_tiles)) * cfg.num_kv_heads;
        const double chunk_us = n_chunk_tiles == 0 ? 0.0 : 4.0 + chunk_steps * (blocks <= 256 ? 0.62 : 0.9);
        double c = std::max(decode_us, chunk_us) + 0.3 * std::min(decode_us, chunk_us);
        if (most > 1) {
            c += 0.25 * (double)most + 2.0 * (double)rows * cfg.num_kv_heads * (cfg.head_dim + 2) * 4.0 / 4.5e6;
            if (!chunk_cut) c += 5.3;
        }
        return c;
    };
    const double as_is = estimate((int32_t)std::min<int64_t>(wave_split, INT32_MAX / 2), 0);
    WaveCut best{wave_split, 0, false, as_is, as_is};
    auto search = [&](int64_t uncut) {
        for (const int32_t keys : {4096, 3072, 2048, 1536, 1024, 768, 512, 384, 256}) {
            const double c = estimate(keys, uncut);
            if (c < std::min(0.95 * as_is, best.us)) best = WaveCut{keys, uncut, true, c, as_is};
        }
    };
    const double host_us = (plan_in_arguments ? 15.8 : 12.8) + (plan_in_arguments ? 0.09 : 0.03) * (double)n_wave_tiles;
    if (as_is >= 28.0 || (n_chunk_tiles == 0 && as_is >= 18.0 && host_us < (plan_in_arguments ? 0.8 : 0.85) * as_is)) {
        if (whole > 0) search(whole);
        if (!best.few) search(0);
    }
    return best;
}

// Whether a batch's short prefill chunks run as wave tiles like its decodes: eight times the blocks, each with an eighth of the columns and
// its keys quartered among its wavefronts, where 128-column tiles leave the chip idle and walk all keys in a row.  A chunk
// tile alone on its compute unit takes 0.52 us per 32 keys (0.33 with 64 channels); a wave block reads its keys, which its
// neighbours read as well, at 95 GB/s out of L2, at half of that next to a second block, and every tile costs the host 0.03 us.
// The line in keys is where cut chunk tiles take as long.  us a pass (append, attention), chunk tiles and wave tiles: 64 tokens
// behind 512, 32 and 8 heads, 18.6 and 11.1; 256 behind 512 22.1 and 18.5, behind 2048 27.3 and 36.2; 64 behind 2048 19.6 and 20.0; 64
// tokens of 64 channels, 4 heads and one, behind 512 14.7 and 9.6, behind 2048 14.2 and 16.2; 256 behind none, 56 and 8 heads, 14.4 and
// 18.5; 64 behind none, 58 and 2 heads of 64, 9.4 and 11.1.  Chunks of more than 1024 columns keep chunk tiles: with few KV heads they would
// gain as well (256 tokens behind 512, 16 and 2 heads, 21.5 and 12.6), but only as long as the batch holds little else.
bool chunks_as_wave_tiles(const sarathi_config &cfg, const Options &opt, const WorkspaceLayout &ws, const int32_t *q_len, const int32_t *ctx_len,
                          int32_t num_seqs) {
    if (opt.tile_split_keys > 0 || opt.resident_chunks == 1 || opt.interleave != 2) return false;  // asks for chunk tiles
    const int64_t G = cfg.num_q_heads / cfg.num_kv_heads;
    int64_t tiles = 0, chunk_tiles = 0, span = 0, other_span = 0, other_keys = 0;  // spans: of the chunks, of the others
    for (int32_t s = 0; s < num_seqs; ++s) {
        const int64_t n = ((int64_t)q_len[s] * G + kWaveCols - 1) / kWaveCols;
        const int64_t keys = opt.window > 0 ? std::min<int64_t>(ctx_len[s], opt.window + q_len[s]) : ctx_len[s];
        tiles += n;
        if (n > 64 || tiles * cfg.num_kv_heads > 512) return false;
        if ((int64_t)q_len[s] * G < kChunkMinCols) {
            other_span = std::max(other_span, keys);
            other_keys += n * keys;
            continue;
        }
        chunk_tiles += n;
        span = std::max(span, keys);
    }
    if (chunk_tiles == 0) return false;
    const bool alone = tiles * cfg.num_kv_heads <= 256;
    const double chunk_us = (double)span / kTileKeys * (cfg.head_dim == 128 ? 0.52 : 0.33);
    const double wave_us = (double)span * cfg.head_dim * 4.0 / (alone ? 95.0e3 : 47.5e3) + 0.03 * (double)chunk_tiles;
    // Decodes that run longer hide the chunks either way, and next to them two blocks to a compute unit take each other's rate (88
    // tokens behind 527 next to 14 decodes of up to 2655 keys, 56 and 8 heads, 30.5 and 35.1; 44 next to 8 of 2328 17.0 and 18.7).
    const double other_us = (double)other_span * cfg.head_dim * 4.0 / 55.0e3;
    // Decodes that stream for longer than the chunk tiles take hide those, and wave tiles take from their rate (us a pass: 121 tokens
    // behind 813 next to 167 decodes that stream 4.0 times as long, 4 heads and one of 64 channels, 47.5 and 53.6; 50 behind 552 next to
    // 6, 3.9 times, 32 and 8 heads, 47.2 and 57.9; of 190 drawn batches beyond 1.5 times 26 are more than 3 % slower as wave tiles, and the
    // average is 1.02 x faster; of 59 between 1.0 and 1.5 times 4, and 1.11 x).
    const double stream_us = (double)other_keys * cfg.num_kv_heads * cfg.head_dim * 4.0 / 6.5e6;
    if (stream_us > 1.5 * chunk_us) return false;
    // Decodes that are cut next to chunk tiles too (25 us at a block's rate) bring a merge along, with which those are cut at no further
    // launch, while wave tiles of long contexts are cut into eight times as many pieces (61 tokens behind 1395 next to 5 decodes of up to
    // 7618 keys, 32 and 8 heads, 25.4 and 36.6; 228 behind 893 next to 80 of up to 4965, 4 heads and one of 64 channels, 17.9 and 20.4; 52
    // behind 964 next to 14 of up to 2934, 32 and 8 heads, 33.1 and 24.5; behind 1445 next to two of up to 3716, which hardly stream, 19.5 and 16.6;
    // allocation-free, where the host pays for each piece, 65 behind 1 and 48 behind 1639 next to 34 of up to 10,291, 4 heads and one of 64, 20.6 and 27.0).
    if (span > 1100 && (double)other_span * cfg.head_dim * 4.0 / 40.0e3 >= 25.0 && (ws.meta_per_launch != 0 || stream_us > 0.15 * chunk_us)) return false;
    if (span > (alone ? 1792 : 896) || std::max(wave_us, std::min(other_us, alone ? 8.0 : 1.0e9)) + 1.0 >= chunk_us) return false;
    // a plan that travels in kernel arguments has to fit one launch so
    return ws.meta_per_launch == 0 || attn_meta_bytes((size_t)tiles, (size_t)tiles, 0) <= ws.meta_per_launch;
}

}  // namespace

void plan_attention(const sarathi_config &cfg, const Options &opt, const WorkspaceLayout &ws,
                    const int32_t *q_start, const int32_t *q_len, const int32_t *ctx_len, int32_t num_seqs,
                    Plan &plan) {
    plan.tiles.clear();
    plan.units.clear();
    plan.reduce_units.clear();
    plan.num_part_rows = 0;
    plan.num_tile_units = 0;
    plan.num_tile_reduce_units = 0;
    plan.num_split_tiles = 0;
    plan.most_pieces = 0;
    plan.shared_wave_keys = 0;
    const int32_t G = cfg.num_q_heads / cfg.num_kv_heads;
    int64_t min_cols = opt.tile_min_cols;
    if (min_cols <= 0) min_cols = chunks_as_wave_tiles(cfg, opt, ws, q_len, ctx_len, num_seqs) ? INT64_MAX : kChunkMinCols;

    // Tiles: chunk tiles first, then wave tiles (two passes keep each kind contiguous).
    int64_t keys_of_kind[2] = {0, 0};
    size_t n_chunk_tiles = 0;
    for (int pass = 0; pass < 2; ++pass) {
        const int32_t kind = pass == 0 ? kKindTile : kKindWave;
        for (int32_t s = 0; s < num_seqs; ++s) {
            const int64_t n_cols = (int64_t)q_len[s] * G;
            const bool chunk = n_cols >= min_cols;   // prefill chunk: 128-column LDS-staged tiles
            if (chunk != (kind == kKindTile)) continue;
            const int32_t prefix = ctx_len[s] - q_len[s];
            const int32_t width = chunk ? kTileCols : kWaveCols;
            for (int64_t c0 = 0; c0 < n_cols; c0 += width) {
                TileDesc t{};
                t.seq = s;
                t.col_begin = (int32_t)c0;
                t.n_cols = (int32_t)std::min<int64_t>(width, n_cols - c0);
                t.kind = kind;
                t.n_keys = prefix + (int32_t)((c0 + t.n_cols - 1) / G) + 1;  // keys .. position of the tile's last row
                if (opt.window > 0) {  // the first row's window starts the range (rounded down to a 32-key tile)
                    const int64_t first_key = (int64_t)prefix + c0 / G - opt.window + 1;
                    t.key_lo = first_key > 0 ? (int32_t)(first_key / kTileKeys * kTileKeys) : 0;
                }
                t.q_start = q_start[s];
                t.q_len = q_len[s];
                t.ctx_len = ctx_len[s];
                plan.tiles.push_back(t);
                keys_of_kind[kind] += t.n_keys - t.key_lo;
                if (!chunk && n_cols > kWaveCols) plan.shared_wave_keys += t.n_keys - t.key_lo;
            }
        }
        if (pass == 0) n_chunk_tiles = plan.tiles.size();
    }

    // Keys per split: the automatic choice aims at ~target units per KV head, never below a
    // floor, and both kinds are coarsened together until the partial buffers suffice.
    auto pick = [](int64_t forced, int64_t total, int64_t target, int64_t floor_keys) {
        int64_t k = forced > 0 ? forced : std::max<int64_t>(floor_keys, ceil_div(total, std::max<int64_t>(1, target)));
        return ceil_div(k, kTileKeys) * kTileKeys;
    };
    // A wave-tile unit is a BLOCK: its four wavefronts take a quarter of the unit's keys each and
    // merge their results in LDS, so a unit of up to 4 x 1024 keys (6144 with the 1.5x allowance
    // below) needs no partial rows and no merge kernel; "split_keys" counts keys per wavefront.
    // When the decodes of the batch take long to stream as a whole, one block may take longer too: a unit that
    // needs up to 0.4 of that time (a block streams about 25 GB/s next to a second one on its compute unit) is
    // dealt out first and is done well before the launch ends, and every cut avoided saves partial rows and,
    // for a batch without other cuts, the merge launch.
    const double wave_stream_us = (double)keys_of_kind[kKindWave] * cfg.num_kv_heads * cfg.head_dim * 4.0 / 5.0e6;
    const int64_t wave_floor = std::max<int64_t>(4 * kMinWaveKeys, (int64_t)(0.4 * wave_stream_us * 25000.0 / (cfg.head_dim * 4.0)));
    int64_t wave_split = pick(4 * opt.split_keys, keys_of_kind[kKindWave], std::max<int64_t>(1, opt.target_items / 4), wave_floor);
    // Chunk tiles: enough units per KV head to put two blocks on every compute unit (a block
    // alone on its unit cannot hide its per-step latencies), but never pieces below the floor.
    // Next to wave tiles the chunk blocks run in the shadow of the memory-bound ones, which keep
    // the other block slots busy: a chunk piece only has to finish within the time the decodes
    // take to stream (about 5 bytes/ps on this part; a chunk block advances 32 keys in roughly a
    // microsecond), and every split avoided saves partial rows that need merging.
    const int64_t tile_units_wanted = std::max<int64_t>(1, 768 / cfg.num_kv_heads);
    const bool has_wave_tiles = plan.tiles.size() > n_chunk_tiles;
    int64_t tile_floor = kMinTileSplitKeys;
    if (has_wave_tiles) {
        const double wave_us = wave_stream_us;
        tile_floor = std::max<int64_t>(2 * kMinTileSplitKeys, (int64_t)(wave_us / 1.2) * kTileKeys);
    }
    // Chunks alone, or next to decodes that hardly count (chunk blocks on at most half of the compute units, decodes that
    // stream for less than a quarter of the time the longest chunk block takes uncut; 512 tokens behind 1871 next to 4
    // decodes: 48 + 6 us with whole chunk tiles, 40 + 9 cut in two; next to 16 decodes, 0.4 of that time, 54 + 6 against
    // 58 + 10): the cheapest cut by playing the launch through.
    int64_t longest_span = 1;
    for (size_t ti = 0; ti < n_chunk_tiles; ++ti)
        longest_span = std::max<int64_t>(longest_span, plan.tiles[ti].n_keys - plan.tiles[ti].key_lo);
    const bool few_decodes = (int64_t)n_chunk_tiles * cfg.num_kv_heads <= 128 &&
                             wave_stream_us < 0.25 * 0.62 * (double)longest_span / kTileKeys;
    auto chunk_count = [&](int64_t keys) { return count_splits(plan, 0, n_chunk_tiles, keys, 0); };
    // Where the plan travels in kernel arguments, a cut that needs further launches for it and keeps the host longer than it
    // spares the GPU is not made: 130 tokens next to 54 decodes of 125-3863 keys, 4 heads and one, 34 us a call whole and 38
    // in 264 pieces.  A cut that fits the launches the uncut plan takes anyway is the same as with a workspace.
    auto host_pays = [&](double us, double whole_us, const SplitCount &chunk, const SplitCount &wave, const SplitCount &whole_chunk) {
        if (ws.meta_per_launch == 0) return true;
        const ArgumentLaunches cut = argument_launches(ws, plan.tiles.size(), chunk, wave);
        const ArgumentLaunches whole = argument_launches(ws, plan.tiles.size(), whole_chunk, SplitCount{});
        return cut.launches == whole.launches || cut.host_us <= us || cut.host_us < 0.95 * std::max(whole_us, whole.host_us);
    };
    int64_t longest_wave_span = 0;
    for (size_t ti = n_chunk_tiles; ti < plan.tiles.size(); ++ti)
        longest_wave_span = std::max<int64_t>(longest_wave_span, plan.tiles[ti].n_keys - plan.tiles[ti].key_lo);
    // What the rules below chose, or a cut that hybrid_launch_us finds 6 % cheaper.  (512 tokens behind 9000 next to 64 decodes,
    // 32 and 8 heads: 177 us in pieces of 3072 keys, 142 in halves.  Of 1500 drawn batches 161 are cut differently, at 0.876 x
    // the time on average; 14 of them are more than 3 % slower, at worst 201 tokens behind 4332 next to one decode, 32 and 32
    // heads, 44.7 and 52.4 us.  Were 10 % to be promised, 6 would be, and the average 0.879 x.)  Forced roles and separate
    // launches get the same cuts: 90 batches with such options are on average within 2 % with and without them.
    auto cheaper_next_to_decodes = [&](int64_t keys, int64_t max_rows) {
        const double key_us = cfg.head_dim * 4.0;
        const int64_t wave_block_keys = std::min(longest_wave_span, wave_split + wave_split / 2);
        HybridBatch b{(double)keys_of_kind[kKindWave] * cfg.num_kv_heads * key_us / 6.5e6, (double)wave_block_keys * key_us / 68.0e3,
                      (int64_t)(plan.tiles.size() - n_chunk_tiles) * cfg.num_kv_heads, 2 * plan.shared_wave_keys > keys_of_kind[kKindWave]};
        if (b.wave_blocks <= 512) b.wave_block_us = std::min(b.wave_block_us, std::max(b.wave_us, 10.0));  // few decodes are cut below
        const std::vector<ChunkBin> &bins = chunk_bins(plan, n_chunk_tiles, longest_span);
        const double as_is = hybrid_launch_us(cfg, bins, b, keys, max_rows);
        if (as_is < 32.0) return keys;  // drawn when the host took as long; it takes about half now, and shorter launches have not been looked at
        double best = 0.94 * as_is;
        int64_t best_keys = keys;
        for (int64_t n = 1; n <= 16 && (n == 1 || longest_span / n >= 256); ++n) {
            const int64_t k = ceil_div(ceil_div(longest_span, n), kTileKeys) * kTileKeys;
            const double us = hybrid_launch_us(cfg, bins, b, k, max_rows);
            if (us < best) best = us, best_keys = k;
        }
        if (best_keys != keys && !host_pays(best, as_is, chunk_count(best_keys), SplitCount{}, chunk_count(keys))) return keys;
        return best_keys;
    };
    auto cut_chunks = [&](int64_t max_rows) {
        if (opt.tile_split_keys <= 0 && n_chunk_tiles > 0 && (!has_wave_tiles || few_decodes)) {
            const ChunkCut cut = cheapest_chunk_cut(cfg, plan, n_chunk_tiles, keys_of_kind[kKindTile], longest_span, max_rows);
            int64_t keys = cut.keys;
            if (!host_pays(cut.us, cut.whole_us, chunk_count(cut.keys), SplitCount{}, SplitCount{}))
                keys = ceil_div(longest_span, kTileKeys) * kTileKeys;
            return has_wave_tiles ? cheaper_next_to_decodes(keys, max_rows) : keys;
        }
        int64_t keys = pick(opt.tile_split_keys, keys_of_kind[kKindTile], tile_units_wanted, tile_floor);
        while (opt.tile_split_keys <= 0 && chunk_count(keys).rows > max_rows) keys *= 2;
        if (opt.tile_split_keys <= 0 && n_chunk_tiles > 0 && has_wave_tiles) return cheaper_next_to_decodes(keys, max_rows);
        return keys;
    };
    int64_t tile_split = cut_chunks(ws.max_part_rows);
    int64_t wave_whole = 0;
    bool few_cut = false;
    if (opt.split_keys <= 0 && has_wave_tiles && (int64_t)(plan.tiles.size() - n_chunk_tiles) * cfg.num_kv_heads <= 512) {
        WaveCut w = cheapest_wave_cut(cfg, plan, n_chunk_tiles, keys_of_kind[kKindWave], tile_split, wave_split, ws.max_part_rows, false,
                                      ws.meta_per_launch != 0);
        auto wave_count = [&]() { return count_splits(plan, n_chunk_tiles, plan.tiles.size(), w.keys, w.whole); };
        const int64_t wave_rows = wave_count().rows;
        if (w.few && wave_rows + chunk_count(tile_split).rows > ws.max_part_rows) {
            // The partial rows do not suffice for both cuts.  The decodes need few and the chunks make do with the rest (512 tokens
            // behind 3871 next to 4000 and 3000 keys, 32 and 8 heads, 4096 rows: 87 us a call with whole chunk tiles, 97 with
            // halves and whole decodes, which next to chunk blocks stream at 25 GB/s); then the decodes are looked at again
            // (512 tokens behind 3871 next to 9000 and 3000 keys: 89 us, 136 with both cuts doubled until they fit).
            if (opt.tile_split_keys <= 0) tile_split = cut_chunks(ws.max_part_rows - wave_rows);
            w = cheapest_wave_cut(cfg, plan, n_chunk_tiles, keys_of_kind[kKindWave], tile_split, wave_split,
                                  std::max<int64_t>(0, ws.max_part_rows - chunk_count(tile_split).rows), true, ws.meta_per_launch != 0);
        }
        if (w.few && host_pays(w.us, w.as_is_us, chunk_count(tile_split), wave_count(), chunk_count(tile_split))) {
            wave_split = w.keys;
            wave_whole = w.whole;
            few_cut = true;
        }
    }
    for (;;) {
        const SplitCount chunk = count_splits(plan, 0, n_chunk_tiles, tile_split, 0);
        const SplitCount wave = count_splits(plan, n_chunk_tiles, plan.tiles.size(), wave_split, wave_whole);
        const int64_t n_split_units = chunk.units + wave.units, n_split_tiles = chunk.tiles + wave.tiles;
        const int64_t n_units = (int64_t)plan.tiles.size() - n_split_tiles + n_split_units;
        const int64_t max_splits_per_tile = (1 << (32 - kUnitTileBits)) - 1;
        bool fits = n_split_units <= kMaxSplitUnits && chunk.rows + wave.rows <= ws.max_part_rows && n_split_tiles <= kMaxSplitUnits / 2 &&
                    (int64_t)plan.tiles.size() + n_split_units <= ws.max_units;
        // a batch whose tiles fit whole is not refused for the pieces it would have been cut into
        if (n_split_tiles > 0 && attn_meta_bytes(plan.tiles.size(), (size_t)n_units, (size_t)(chunk.reduce_units + wave.reduce_units)) > ws.max_attn_meta)
            fits = false;
        for (const TileDesc &t : plan.tiles)
            if (ceil_div(t.n_keys - t.key_lo, t.kind == kKindTile ? tile_split : wave_split) > max_splits_per_tile) { fits = false; break; }
        if (fits) break;
        // partial rows: the kind that needs more of them makes do with less
        const bool rows_only = chunk.rows + wave.rows > ws.max_part_rows;
        if (!rows_only || wave.rows >= chunk.rows) wave_split *= 2;
        if (!rows_only || chunk.rows >= wave.rows) tile_split *= 2;
    }
    plan.split_keys = (int32_t)std::min<int64_t>(wave_split / 4, INT32_MAX);  // per wavefront
    plan.tile_split_keys = (int32_t)std::min<int64_t>(tile_split, INT32_MAX);

    static thread_local std::vector<uint32_t> scratch;
    static thread_local std::vector<int32_t> bucket;
    emit_units(plan, 0, n_chunk_tiles, tile_split, 0, scratch, bucket);
    plan.num_tile_units = (int32_t)plan.units.size();
    plan.num_tile_reduce_units = (int32_t)plan.reduce_units.size();
    plan.wave_keys = keys_of_kind[kKindWave];
    const size_t wave_base = plan.units.size();
    const int32_t split_chunk_tiles = plan.num_split_tiles;
    emit_units(plan, n_chunk_tiles, plan.tiles.size(), wave_split, wave_whole, scratch, bucket);
    plan.longest_wave_keys = 0;  // units are sorted longest first
    if (plan.units.size() > wave_base) {
        const uint32_t u = plan.units[wave_base];
        plan.longest_wave_keys = steps_of_split(plan.tiles[u & ((1u << kUnitTileBits) - 1)], (int32_t)(u >> kUnitTileBits)) * kTileKeys;
    }
    // Few decodes in pieces of nearly one length: the longest piece (the first unit), were all as long as it, would be at most
    // 1.35 times the keys there are.
    plan.even_decode_pieces = false;
    if (few_cut && plan.num_split_tiles > split_chunk_tiles) {
        const int64_t n_units = (int64_t)(plan.units.size() - wave_base);
        plan.even_decode_pieces = 20 * (int64_t)plan.longest_wave_keys * n_units <= 27 * keys_of_kind[kKindWave];
    }
    pair_column_tiles(plan, wave_base, cfg.num_kv_heads, scratch);
}

}  // namespace sarathi
