"""CPU tests: the C-ABI library loads without a GPU, exports every declared symbol, validates batch
descriptions before touching the device, and plans a work decomposition that covers every
(column, key) pair exactly once."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2403_02310_amd import binding, workloads as wl

from . import linear_tile_cases

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "sarathi.h")).read()
    declared = set(re.findall(r"\b(sarathi_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found"
    assert declared == set(binding.EXPORTED)
    for name in declared:
        assert getattr(binding.lib, name) is not None


def test_create_rejects_bad_shapes():
    for kw, status in [(dict(num_q_heads=6, num_kv_heads=4), binding.ESHAPE),
                       (dict(head_dim=96), binding.ESHAPE), (dict(page_size=32), binding.ESHAPE),
                       (dict(dtype=1), binding.ESHAPE), (dict(max_tokens=0), binding.EINVAL)]:
        args = dict(num_q_heads=8, num_kv_heads=2, head_dim=128, max_tokens=64, max_seqs=8, max_blocks_per_seq=8,
                    page_size=16, dtype=0)
        args.update(kw)
        with pytest.raises(binding.SarathiError) as e:
            binding.Handle(**args)
        assert e.value.status == status


def _call_attention(h, q_start, q_len, ctx_len, num_tokens=None, ws=256, ptr=1, num_pages=100, scale=0.1):
    qs, ql, cl = (np.ascontiguousarray(a, np.int32) for a in (q_start, q_len, ctx_len))
    i32p = ctypes.POINTER(ctypes.c_int32)
    n = int(ql.sum()) if num_tokens is None else num_tokens
    # non-null fake device pointers: validation must fail before anything is dereferenced or enqueued
    return binding.lib.sarathi_hybrid_attention(h._h, ptr, ptr, ptr, ptr, qs.ctypes.data_as(i32p), ql.ctypes.data_as(i32p),
                                                cl.ctypes.data_as(i32p), len(ql), n, num_pages, scale, ptr, ws, None)


def test_validation_errors_are_reported_without_a_gpu():
    h = binding.Handle(8, 2, 128, max_tokens=64, max_seqs=4, max_blocks_per_seq=4)
    assert _call_attention(h, [0], [0], [5]) == binding.EINVAL                 # q_len < 1
    assert _call_attention(h, [0], [6], [5]) == binding.EINVAL                 # q_len > ctx_len
    assert "q_len" in h.last_error()
    assert _call_attention(h, [1], [2], [5]) == binding.EINVAL                 # q_start not the prefix sum
    assert _call_attention(h, [0, 2], [2, 3], [5, 9], num_tokens=6) == binding.EINVAL   # sum q_len != num_tokens
    assert _call_attention(h, [0], [2], [65]) == binding.ECAPACITY             # more pages than max_blocks_per_seq
    assert _call_attention(h, [0], [65], [65]) == binding.ECAPACITY            # more tokens than max_tokens
    assert _call_attention(h, [0, 1, 2, 3, 4], [1] * 5, [3] * 5) == binding.ECAPACITY   # more seqs than max_seqs
    assert _call_attention(h, [0], [2], [5], num_pages=0) == binding.EINVAL
    assert _call_attention(h, [0], [2], [5], ptr=None) == binding.EINVAL       # null tensor
    assert _call_attention(h, [0], [2], [5], ws=None) == binding.EWORKSPACE
    assert _call_attention(h, [0], [2], [5], ws=264) == binding.EWORKSPACE      # not 256-byte aligned
    assert _call_attention(h, [0], [2], [5], scale=float("nan")) == binding.EINVAL
    assert _call_attention(h, [0], [2], [5], scale=-1.0) == binding.EINVAL
    assert _call_attention(h, [], [], [], num_tokens=0) == binding.OK          # empty batch: nothing to do
    with pytest.raises(binding.SarathiError):
        h.set_option("no_such_option", 1)


def _coverage_check(batch, **options):
    s = batch.shape
    h = binding.Handle(s.num_q_heads, s.num_kv_heads, s.head_dim, max_tokens=max(2048, batch.num_tokens),
                       max_seqs=max(128, batch.num_seqs), max_blocks_per_seq=batch.max_blocks_per_seq)
    for k, v in options.items():
        h.set_option(k, v)
    info, items = h.plan(batch.q_start, batch.q_len, batch.ctx_len)
    assert len(items) == info.num_items
    G = s.group
    covered = {}
    part_rows = set()
    for idx, it in enumerate(items):
        assert it.kind == (1 if idx < info.num_tile_items else 0)
        assert 1 <= it.n_cols <= (128 if it.kind == 1 else 16)
        assert it.key_begin % 32 == 0 and it.key_begin < it.key_end
        seq, prefix = it.seq, int(batch.ctx_len[it.seq] - batch.q_len[it.seq])
        assert it.col_begin + it.n_cols <= int(batch.q_len[seq]) * G
        last_row = (it.col_begin + it.n_cols - 1) // G
        assert it.key_end <= prefix + last_row + 1          # never past the tile's last visible key
        key = (seq, it.col_begin, it.n_cols)
        covered.setdefault(key, []).append((it.key_begin, it.key_end, it.part_row))
        if it.part_row >= 0:
            rows = set(range(it.part_row, it.part_row + it.n_cols))
            assert not (rows & part_rows), "partial rows overlap"
            part_rows |= rows
    assert len(part_rows) == info.num_part_rows
    # tiles partition every sequence's columns; their pieces partition keys 0 .. last visible key
    for seq in range(batch.num_seqs):
        cols = sorted((c0, nc) for (s_, c0, nc) in covered if s_ == seq)
        pos = 0
        for c0, nc in cols:
            assert c0 == pos
            pos += nc
        assert pos == int(batch.q_len[seq]) * G
    for (seq, c0, nc), pieces in covered.items():
        prefix = int(batch.ctx_len[seq] - batch.q_len[seq])
        pieces.sort()
        window = int(options.get("window", 0))
        first_visible = max(0, prefix + c0 // G - window + 1) if window else 0   # first key of the tile's first row
        assert pieces[0][0] == first_visible // 32 * 32 and pieces[-1][1] == prefix + (c0 + nc - 1) // G + 1
        for a, b in zip(pieces, pieces[1:]):
            assert a[1] == b[0]
        assert all((p[2] >= 0) == (len(pieces) > 1) for p in pieces)
    return info


@pytest.mark.parametrize("make", [wl.config1_tiny, wl.config2_mistral_hybrid, wl.config4_yi_long, wl.config5_llama70b])
def test_plan_covers_every_column_and_key_once(make):
    _coverage_check(make())


def test_plan_coverage_with_forced_options():
    b = wl.random_hybrid(3, wl.AttnShape(14, 2, 128), n_chunks=3, n_decodes=9, max_chunk=200, max_ctx=3000)
    _coverage_check(b, split_keys=32, tile_split_keys=32)
    _coverage_check(b, tile_min_cols=1)
    _coverage_check(b, tile_min_cols=1 << 20, split_keys=1 << 20)


@pytest.mark.parametrize("heads,q_len,ctx_len,window,chunk_tiles", [
    ((32, 8, 128), [64], [1792], 0, False), ((32, 8, 128), [64], [1793], 0, True),               # keys, a block per compute unit
    ((32, 8, 128), [128], [1000], 0, False), ((32, 8, 128), [129], [1000], 0, True),             # beyond 256 blocks fewer keys
    ((32, 8, 128), [256], [896], 0, False), ((32, 8, 128), [256], [897], 0, True), ((32, 8, 128), [257], [700], 0, True),  # 512 blocks
    ((32, 8, 128), [64], [96], 0, True), ((4, 1, 64), [64], [1500], 0, False), ((4, 1, 64), [64], [192], 0, True),
    ((32, 8, 128), [64] + [1] * 4, [576] + [500] * 4, 0, False), ((32, 8, 128), [64] + [1] * 4, [576] + [3000] * 4, 0, False),
    ((32, 8, 128), [64] + [1] * 4, [400] + [3000] * 4, 0, True), ((56, 8, 128), [88] + [1] * 14, [615] + [2655] * 14, 0, True),
    ((32, 8, 128), [64], [9000], 500, False), ((32, 8, 128), [16, 17], [400, 1000], 0, False), ((16, 2, 128), [15], [700], 0, False),
    ((16, 2, 128), [128], [700], 0, False), ((16, 2, 128), [129], [700], 0, True),                                        # columns
])
def test_short_chunks_of_small_batches_run_as_wave_tiles(heads, q_len, ctx_len, window, chunk_tiles):
    b = wl._make("short_chunks", wl.AttnShape(*heads), q_len, ctx_len, 5)
    assert (_coverage_check(b, window=window).num_tile_items > 0) == chunk_tiles
    assert _coverage_check(b, window=window, tile_min_cols=64).num_tile_items > 0
    for asks in ({"tile_split_keys": 64}, {"resident_chunks": 1}, {"interleave": 0}):
        assert _coverage_check(b, window=window, **asks).num_tile_items > 0


@pytest.mark.parametrize("heads,q_len,ctx_len,chunk_tiles", [
    ((32, 8, 128), [61] + [1] * 5, [1456] + [7618, 6000, 4000, 3000, 2802], True),       # decodes that are cut, 1456 keys
    ((32, 8, 128), [61] + [1] * 5, [1100] + [7618, 6000, 4000, 3000, 2802], False),      # up to 1100
    ((32, 8, 128), [61] + [1] * 5, [1456] + [1900] * 5, False),                          # decodes that stay whole
    ((32, 8, 128), [43] + [1] * 2, [1488] + [3716, 631], False),                         # and hardly stream
    ((4, 1, 64), [228] + [1] * 80, [1121] + [4965] + [1156] * 79, True),
    ((4, 1, 64), [121] + [1] * 167, [934] + [5862] * 167, True),                         # decodes stream four times as long as the chunk
    ((32, 8, 128), [49] + [1] * 11, [569] + [2151] * 11, True), ((32, 8, 128), [49] + [1] * 10, [569] + [2151] * 10, False),   # 1.6 and 1.5 times
])
def test_short_chunks_stay_chunk_tiles_next_to_long_decodes(heads, q_len, ctx_len, chunk_tiles):
    """Where the decodes hide the chunks, or are cut and merged anyway, as chunk tiles of long contexts then are."""
    b = wl._make("short_chunks", wl.AttnShape(*heads), q_len, ctx_len, 6)
    assert (_coverage_check(b).num_tile_items > 0) == chunk_tiles


@pytest.mark.parametrize("heads,n,keys,cut", [
    ((4, 1, 64), 60, 2500, True), ((4, 1, 64), 212, 2500, False), ((4, 1, 64), 348, 2200, False),   # the host's time for the pieces
    ((4, 1, 64), 348, 4200, True),                                                                   # estimated at 28 us and more
    ((16, 2, 128), 40, 1250, True), ((32, 8, 128), 1, 1300, True), ((32, 8, 128), 1, 1024, False),
])
def test_decodes_are_cut_where_the_host_is_done_sooner(heads, n, keys, cut):
    ctx_len = [keys] + [max(1, keys // 7)] * (n - 1)
    b = wl._make("few_decodes", wl.AttnShape(*heads), [1] * n, ctx_len, 7)
    assert (_coverage_check(b).num_reduce_items > 0) == cut


@pytest.mark.parametrize("window", [1, 33, 500, 4096])
def test_plan_coverage_under_a_sliding_window(window):
    """Pieces start at the 32-key tile that holds the first key of the tile's first row's window."""
    b = wl.random_hybrid(4, wl.AttnShape(14, 2, 128), n_chunks=3, n_decodes=9, max_chunk=200, max_ctx=3000)
    _coverage_check(b, window=window)
    _coverage_check(b, window=window, split_keys=32, tile_split_keys=64)
    _coverage_check(wl.config4_yi_long(), window=window)


def test_long_decodes_are_cut_only_where_their_block_would_be_the_tail():
    """A decode's keys go to one block of four wavefronts unless that block would outlast a good part of the time
    the batch's decodes take to stream: the 16,384-key decodes of the long-context recipe stay whole (no partial
    rows, no merge launch), the same decode next to a handful of short ones is cut, and so is a lone long decode."""
    info = _coverage_check(wl.config4_yi_long())
    assert info.num_reduce_items == 0 and info.num_part_rows == 0
    s = wl.AttnShape(56, 8, 128)
    few = wl._make("few", s, [1] * 6, [16384, 300, 900, 50, 1200, 700], 10)
    info = _coverage_check(few)
    assert info.num_reduce_items == 1 and info.num_part_rows > 0          # only the long one, in several pieces
    lone = wl._make("lone", s, [1], [100000], 11)
    info = _coverage_check(lone)
    assert info.num_reduce_items == 1 and info.num_items >= 8


def test_plan_stays_within_the_workspace_when_everything_is_long():
    s = wl.AttnShape(64, 8, 128)
    b = wl._make("long", s, [2048], [16384], 9)
    info = _coverage_check(b, tile_split_keys=32, split_keys=32)
    assert info.num_part_rows <= 32768


def test_linear_refuses_bad_shapes_without_a_gpu():
    """Shape checks come before any device call, so they can be exercised here."""
    for (T, N, K) in [(-1, 128, 64), (4, 0, 64), (4, 100, 64), (4, 128, 32), (4, 128, 96), (4, 128, (1 << 20) + 64)]:
        assert binding.lib.sarathi_linear(None, None, None, T, N, K, None, 0, None) == binding.ESHAPE
        assert binding.linear_workspace_bytes(T, N, K) == 0
    assert binding.lib.sarathi_linear(None, None, None, 0, 128, 64, None, 0, None) == 0          # no tokens: nothing to do
    assert binding.lib.sarathi_linear(None, None, None, 4, 128, 64, None, 0, None) == binding.EINVAL


def test_linear_split_k_workspace_sizes():
    """A small batch on big weights asks for partial tiles; a batch that fills the chip by itself asks for none."""
    assert binding.linear_workspace_bytes(2048, 8192, 4096) == 0
    small = binding.linear_workspace_bytes(128, 4096, 14336)
    assert small > 0 and small % (128 * 4096 * 4) == 0 and small // (128 * 4096 * 4) <= 16


FEW_DECODES = [  # shape, q_len, ctx, whether something has to be cut
    (wl.AttnShape(32, 8, 128), [1] * 8, [4096] * 8, True),                             # equal, a multiple of every piece
    (wl.AttnShape(32, 8, 128), [1] * 8, [257, 385, 513, 4095, 4096, 4097, 2049, 1], True),  # around the piece sizes
    (wl.AttnShape(32, 8, 128), [1] * 65, [4096] * 65, False),                          # 520 blocks: not a few any more
    (wl.AttnShape(32, 8, 128), [1], [300], False),                                     # one short decode
    (wl.AttnShape(58, 2, 64), [1] * 5, [6000, 5900, 5800, 100, 5700], True),           # two column tiles per decode
    (wl.AttnShape(8, 2, 128), [1, 1, 1], [9000, 2000, 3000], True),                    # one holds half of the keys
    (wl.AttnShape(16, 2, 128), [512] + [1] * 4, [2383, 4000, 100, 300, 4000], True),   # next to a chunk, which is cut too
    (wl.AttnShape(32, 8, 128), [700] + [1] * 16, [700] + [3000] * 16, True),
]


@pytest.mark.parametrize("case", range(len(FEW_DECODES)))
@pytest.mark.parametrize("window", [0, 1000])
def test_few_decodes_are_cut_and_covered(case, window):
    """Small batches are cut until the chip is filled: every key is still covered once, pieces stay within two blocks
    per compute unit's worth of rounding, and a decode that holds half of the batch's keys is cut alone."""
    shape, q_len, ctx, cut = FEW_DECODES[case]
    info = _coverage_check(wl._make("few%d" % case, shape, q_len, ctx, 90 + case), **({"window": window} if window else {}))
    if not window:
        assert (info.num_reduce_items > 0) == cut
    if case == 5 and not window:
        assert info.num_reduce_items == 1


@pytest.mark.parametrize("shape,chunks,cut", [
    (wl.AttnShape(64, 8, 128), [(1299, 1299), (749, 4960)], False),   # two prompts that fill the chip whole
    (wl.AttnShape(56, 8, 128), [(1024, 11825), (512, 8627), (384, 3123)], True),  # several rounds, alike by the estimate
    (wl.AttnShape(64, 8, 128), [(578, 3500), (231, 231)], False),     # one round, a cut promises less than 5 %
    (wl.AttnShape(32, 8, 128), [(512, 2383)], True),                  # 128 blocks of 75 steps
    (wl.AttnShape(32, 8, 128), [(1000, 1100), (400, 9400)], True),    # one long prefix among short ones
    (wl.AttnShape(32, 8, 128), [(300, 300)], False),
    (wl.AttnShape(4, 1, 64), [(278, 6572), (987, 987)], True),        # more groups than units
    (wl.AttnShape(320, 320, 64), [(40, 3000), (3000, 3000)], False),  # more KV heads than compute units, more than 8192 blocks
    (wl.AttnShape(64, 8, 128), [(4096, 70000)], False)])              # every slot busy to the end
def test_chunk_only_batches_are_cut_where_it_pays(shape, chunks, cut):
    """The cut of a chunk-only launch comes from playing it through; whatever it says, every key is covered once."""
    b = wl._make("chunks", shape, [q for q, _ in chunks], [c for _, c in chunks], 95)
    info = _coverage_check(b)
    assert (info.num_reduce_items > 0) == cut


@pytest.mark.parametrize("shape,q_len,meet", [(wl.AttnShape(58, 2, 64), [1] * 8, True),
                                              (wl.AttnShape(58, 2, 64), [1] * 9, False),          # a last, short window
                                              (wl.AttnShape(20, 1, 128), [1] * 7 + [3], False),   # two tiles and four
                                              (wl.AttnShape(12, 3, 64), [6, 1, 5, 1, 6], False)])  # two tiles and one
def test_column_tiles_of_a_sequence_meet_on_an_xcd(shape, q_len, meet):
    """With fewer than eight KV heads the wave tiles of one sequence are spread so that block % 8 is the same for each;
    every piece still appears once."""
    b = wl._make("pairs", shape, q_len, [2000 + 300 * i for i in range(len(q_len))], 96)
    _coverage_check(b)
    _coverage_check(b, split_keys=100)
    _coverage_check(b, split_keys=1 << 20)
    h = binding.Handle(shape.num_q_heads, shape.num_kv_heads, shape.head_dim, max_tokens=2048, max_seqs=128,
                       max_blocks_per_seq=b.max_blocks_per_seq)
    h.set_option("split_keys", 1 << 20)
    _, items = h.plan(b.q_start, b.q_len, b.ctx_len)
    where = {(it.seq, it.col_begin): i for i, it in enumerate(items)}
    assert len(where) == len(items) == sum(-(-q * shape.group // 16) for q in q_len)
    if meet:
        assert all((where[(s, 16)] - where[(s, 0)]) * shape.num_kv_heads % 8 == 0 for s in range(b.num_seqs))


def test_the_library_functions_refuse_length_arrays_of_another_type():
    """``binding.lib``'s functions take int32 pointers: an address or an array of 64-bit lengths is refused, not read as it is."""
    h = binding.Handle(8, 2, 128, max_tokens=64, max_seqs=4, max_blocks_per_seq=4)
    good = (ctypes.c_int32 * 1)(5)
    for bad in ((ctypes.c_int64 * 1)(5), ctypes.addressof(good), b"\5\0\0\0"):
        for name, args in (("sarathi_kv_append", (h._h, 1, 1, 1, 1, 1, good, bad, good, 1, 5, 9, 256, None)),
                           ("sarathi_hybrid_attention", (h._h, 1, 1, 1, 1, good, bad, good, 1, 5, 9, 0.1, 1, 256, None)),
                           ("sarathi_hybrid_attention_noalloc", (h._h, 1, 1, 1, 1, good, good, bad, 1, 5, 9, 0.1, 1, None))):
            with pytest.raises(ctypes.ArgumentError):
                getattr(binding.lib, name)(*args)


@pytest.mark.parametrize("rest", [[7000, 6500], [10000, 8000], [3000, 3000, 100]])
def test_decodes_around_half_of_the_keys_are_cut_alike(rest):
    """A plan that cuts only the decode that holds half of the batch's keys is an offer, not a must: just above and just below
    that half the longest piece is about the same, and no longer than what one block streams well within the launch."""
    shape, half, longest = wl.AttnShape(32, 8, 128), sum(rest), []
    for first in (half - 300, half, half + 300):
        b = wl._make("half", shape, [1] * (1 + len(rest)), [first] + rest, 97)
        _coverage_check(b)
        h = binding.Handle(32, 8, 128, max_tokens=64, max_seqs=8, max_blocks_per_seq=b.max_blocks_per_seq)
        _, items = h.plan(b.q_start, b.q_len, b.ctx_len)
        longest.append(max(it.key_end - it.key_begin for it in items))
    if rest[-1] > 100:
        assert max(longest) <= 1.5 * min(longest) and max(longest) <= 2304
    else:
        assert max(longest) <= 3000   # the 3000-key decodes stay whole above the half


@pytest.mark.parametrize("shape,chunks", [
    (wl.AttnShape(58, 2, 64), [(1000, 1100), (800, 830), (200, 12200)]),
    (wl.AttnShape(71, 1, 64), [(8192, 8192)]),
    (wl.AttnShape(71, 1, 64), [(1080, 1085), (1868, 1868), (179, 179), (1, 2394), (1, 5761), (1, 3000)])])
def test_choosing_the_cut_takes_no_longer_than_a_few_plans(shape, chunks):
    """The cut of a chunk-only batch is searched before its launch can be enqueued.  Planning it takes at most three times what the
    same plan takes with the cut given (both the fastest of many runs, on the same machine)."""
    import time
    b = wl._make("chunks", shape, [q for q, _ in chunks], [c for _, c in chunks], 98)
    h = binding.Handle(shape.num_q_heads, shape.num_kv_heads, shape.head_dim, max_tokens=16384, max_seqs=64,
                       max_blocks_per_seq=b.max_blocks_per_seq)

    def fastest():
        best = 1.0
        for _ in range(60):
            t = time.perf_counter()
            info, _ = h.plan(b.q_start, b.q_len, b.ctx_len, with_items=False)
            best = min(best, time.perf_counter() - t)
        return best * 1e6, info
    searched_us, searched = fastest()
    h.set_option("tile_split_keys", searched.tile_split_keys)
    given_us, given = fastest()
    assert given.num_items == searched.num_items
    assert searched_us <= 3 * given_us + 15, (searched_us, given_us)


@pytest.mark.parametrize("shape,short,long", [(wl.AttnShape(64, 8, 128), 32, (64, 60000)), (wl.AttnShape(32, 32, 128), 34, (100, 60000))])
def test_a_long_chunk_among_very_many_short_ones_is_cut(shape, short, long):
    """More than 8192 chunk blocks: a few tiles behind a long prefix are still cut, or they alone would set the launch's time."""
    n = 512 if shape.num_kv_heads == 8 else 1000
    b = wl._make("many", shape, [n] * short + [long[0]], [n] * short + [long[1]], 99)
    info = _coverage_check(b)
    assert 0 < info.num_reduce_items <= -(-long[0] * shape.group // 128)
    assert info.tile_split_keys <= long[1] // 4


def test_a_tile_that_no_kernel_has_is_an_error():
    """The launcher takes its kernels from the planner's table of tiles; a plan that names another tile is refused and not
    answered with success and an untouched output.  (The refusal comes before any device call.)"""
    launch = binding.lib["_ZN7sarathi13launch_linearERKNS_10LinearPlanEPKvS4_PviiiS5_S5_"]
    launch.argtypes = [ctypes.POINTER(ctypes.c_int32 * 6), ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
                       ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    for tokens, features, token_tile in [(100, 320, 128), (100, 128, 96), (100, 0, 0), (32, 192, 64)]:
        plan = (ctypes.c_int32 * 6)(features, token_tile, 1, 1, 1, 64)   # feature and token tile, their numbers, pieces, k per piece
        assert launch(ctypes.byref(plan), None, None, None, tokens, 128, 64, None, None) == 9   # hipErrorInvalidConfiguration


def test_linear_tile_cases_run_the_tiles_they_name():
    """The parity tests of the linear layer's tiles cover what they say, whatever the planner's constants become."""
    for cases in (linear_tile_cases.LARGE, linear_tile_cases.SMALL):
        for (T, N, K), (features, tokens, one_tile, pieces) in cases.items():
            p = binding.plan_linear(T, N, K)
            assert (p.feature_tile, p.token_tile, p.token_tiles == 1, p.pieces) == (features, tokens, one_tile, pieces), (T, N, K)
            assert p.feature_tiles == -(-N // features) and p.token_tiles == -(-T // tokens)
            assert p.k_per_piece % 64 == 0 and (p.pieces - 1) * p.k_per_piece < K <= p.pieces * p.k_per_piece
            assert binding.plan_linear(T, N, K, 0).pieces == 1                      # no workspace, no pieces


def test_linear_tile_cases_cover_every_kernel_the_planner_chooses():
    """Every tile that a sweep over tokens, features and k comes across is among the cases, with one token tile (which has a kernel
    of its own) and with several, cut along k and uncut."""
    covered = {(f, t, one, pieces > 1) for f, t, one, pieces in linear_tile_cases.LARGE.values()}
    small = {(f, t, one, pieces > 1) for f, t, one, pieces in linear_tile_cases.SMALL.values()}
    for T in (1, 20, 64, 65, 100, 129, 150, 193, 200, 256, 257, 300, 450, 577, 900, 1025):
        for N in range(128, 20000, 640):
            for K in (64, 704, 1984, 3008, 4032, 6144, 8128, 11776):
                p = binding.plan_linear(T, N, K)
                assert (p.feature_tile, p.token_tile, p.token_tiles == 1, p.pieces > 1) in (covered if T > 64 else small), (T, N, K)


@pytest.mark.parametrize("T,N,K,thin", [(16, 1536, 49152, False), (8, 1664, 49152, False), (12, 1664, 17152, False), (16, 4224, 49152, False),
                                        (14, 3456, 32768, False), (17, 1536, 10240, False), (16, 1536, 4096, True), (16, 3968, 14848, True), (8, 4096, 14336, True),
                                        (16, 12288, 16384, True), (8, 8192, 28672, True), (32, 8192, 2048, True), (24, 2048, 8128, True)])
def test_a_few_tokens_are_cut_along_k_where_workgroups_would_wait_for_long_ranges(T, N, K, thin):
    p = binding.plan_linear(T, N, K)
    assert ((p.token_tile, p.pieces) == (32, 1)) == thin and (thin or p.pieces > 1), (p.token_tile, p.pieces)


@pytest.mark.parametrize("T,N,K,uncut", [(81, 14848, 512, False), (96, 13824, 1024, False), (81, 13824, 2048, True), (77, 14848, 512, True),
                                         (96, 12288, 512, True), (96, 20480, 1024, True), (90, 14848, 3712, True)])
def test_81_to_96_tokens_on_short_ranges_of_64_features_run_in_larger_tiles(T, N, K, uncut):
    assert (binding.plan_linear(T, N, K).token_tile in (80, 96)) == uncut


@pytest.mark.parametrize("T,N,K,first,pieces_of_rest", [
    (700, 24704, 704, 21760, 0), (1300, 11264, 1984, 6912, 0), (1025, 13184, 1984, 13056, 7), (577, 26240, 3008, 26112, 10), (2048, 14336, 8192, 8192, 0),
    (2048, 8192, 7168, 8192, 0), (96, 65664, 704, 65664, 0), (577, 12416, 704, 12416, 0),      # full rounds, one token tile, fewer tiles than units
])
def test_features_behind_the_full_rounds_get_a_tiling_of_their_own(T, N, K, first, pieces_of_rest):
    p = binding.plan_linear(T, N, K)
    assert min(N, p.feature_tile * p.feature_tiles) == first
    ws = binding.linear_workspace_bytes(T, N, K)
    assert ws == 4 * pieces_of_rest * T * (N - first)
    if first < N:
        tiles = p.feature_tiles * p.token_tiles   # full rounds, as nearly as whole feature tiles fill them
        assert p.pieces == 1 and tiles >= 128 and -tiles % 256 < p.token_tiles
        assert binding.plan_linear(T, N, K, 0).pieces == 1


@pytest.mark.parametrize("T,N,K,rest", [(1025, 13184, 1984, (128, 64, 7)), (577, 26240, 3008, (128, 64, 10)), (2048, 14336, 8192, (192, 256, 1)), (2048, 8192, 7168, None)])
def test_plan_linear_rest_is_the_second_tiling(T, N, K, rest):
    p = binding.plan_linear_rest(T, N, K)
    assert (p and (p.feature_tile, p.token_tile, p.pieces)) == rest


def test_the_two_tilings_cover_the_features_and_ask_for_the_workspace():
    rng = np.random.default_rng(3)
    two = 0
    for _ in range(600):
        T, N, K = int(np.exp(rng.uniform(0, np.log(2500)))), 128 * int(rng.integers(1, 240)), 64 * int(rng.integers(1, 230))
        for ws in (None, 0, 1 << 22):
            first, rest = binding.plan_linear(T, N, K, ws), binding.plan_linear_rest(T, N, K, ws)
            covered = first.feature_tile * first.feature_tiles
            assert (covered < N) == (rest is not None)
            need = 0
            for p, features in ((first, min(N, covered)),) + (((rest, N - covered),) if rest else ()):
                assert p.feature_tile * (p.feature_tiles - 1) < features <= p.feature_tile * p.feature_tiles
                assert p.token_tile * (p.token_tiles - 1) < T <= p.token_tile * p.token_tiles
                assert p.k_per_piece * (p.pieces - 1) < K <= p.k_per_piece * p.pieces
                need = max(need, 4 * p.pieces * T * features if p.pieces > 1 else 0)
            if ws is None:
                assert binding.linear_workspace_bytes(T, N, K) == need
                two += rest is not None
            else:
                assert need <= ws
    assert two > 20


def test_plan_linear_refuses_what_linear_refuses():
    out = binding.LinearPlan()
    for plan in (binding.lib.sarathi_plan_linear, binding.lib.sarathi_plan_linear_rest):
        assert plan(0, 128, 64, 0, ctypes.byref(out)) == binding.EINVAL
        assert plan(4, 100, 64, 0, ctypes.byref(out)) == binding.ESHAPE
        assert plan(4, 128, 64, 0, None) == binding.EINVAL
