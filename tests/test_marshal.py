"""The native argument marshalling hands the C calls what the objects hold, in every form that they may come in."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2403_02310_amd import binding

vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
APPEND = ctypes.CFUNCTYPE(ctypes.c_int, *[vp] * 9, i32, i32, i64, vp, vp)
ATTENTION = ctypes.CFUNCTYPE(ctypes.c_int, *[vp] * 8, i32, i32, i64, ctypes.c_float, vp, vp, vp)
NOALLOC = ctypes.CFUNCTYPE(ctypes.c_int, *[vp] * 8, i32, i32, i64, ctypes.c_float, vp, vp)
MAX_BLOCKS = 5


@pytest.fixture
def calls():
    """Calls as the C side sees them: the arguments, lengths read out of memory."""
    got = []

    def record(kind, first_length):
        def f(*args):
            n = args[first_length + 3]
            lengths = [list((i32 * n).from_address(args[first_length + j])) for j in range(3)]
            got.append((kind, args[:first_length], lengths, args[first_length + 3:]))
            return -3
        return f
    fns = [APPEND(record("append", 6)), ATTENTION(record("attention", 5)), NOALLOC(record("noalloc", 5))]
    tail = (np.ndarray, binding._i32, lambda: 77, binding._check_block_table)
    binding._marshal.setup(*(ctypes.cast(f, vp).value for f in fns), *tail)
    yield got
    binding._marshal.setup(*(ctypes.cast(f, vp).value for f in (binding.lib.sarathi_kv_append, binding.lib.sarathi_hybrid_attention,
                                                               binding.lib.sarathi_hybrid_attention_noalloc)),
                           np.ndarray, binding._i32, binding._current_stream, binding._check_block_table)


def tensors():
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16)  # noqa: E731
    return {"q": bf(4, 2, 64), "k_new": bf(4, 1, 64), "v_new": bf(4, 1, 64), "k": bf(7, 1, 16, 64), "v": bf(7, 1, 64, 16),
            "table": torch.zeros(3, MAX_BLOCKS, dtype=torch.int32), "out": bf(4, 2, 64), "ws": bf(512)}


LENGTHS = [[0, 2, 3], [2, 1, 1], [2, 9, 30]]
FORMS = [lambda a: np.array(a, np.int32), list, tuple, lambda a: np.array(a, np.int64), lambda a: np.array(a, ">i4"),
         lambda a: np.repeat(np.array(a, np.int32), 2)[::2], lambda a: torch.tensor(a), lambda a: np.array(a, np.uint32)]


@pytest.mark.parametrize("form", range(len(FORMS)))
def test_lengths_of_every_form(calls, form):
    t = tensors()
    qs, ql, cl = (FORMS[form](a) for a in LENGTHS)
    m = binding._marshal
    assert m.kv_append(11, MAX_BLOCKS, t["k_new"], t["v_new"], t["k"], t["v"], t["table"], qs, ql, cl, None, None, t["ws"], None) == -3
    assert m.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], qs, ql, cl, None, None, 0.5, t["out"], 9, t["ws"]) == -3
    assert m.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], qs, ql, cl, 6, 3, 0.25, t["out"], None) == -3
    at = lambda *names: tuple(t[n].data_ptr() for n in names)  # noqa: E731
    assert calls == [
        ("append", (11, *at("k_new", "v_new", "k", "v", "table")), LENGTHS, (3, 4, 7, *at("ws"), 77)),
        ("attention", (11, *at("q", "k", "v", "table")), LENGTHS, (3, 4, 7, 0.5, *at("out", "ws"), 9)),
        ("noalloc", (11, *at("q", "k", "v", "table")), LENGTHS, (3, 3, 6, 0.25, *at("out"), 77)),
    ]


def unaligned(a):
    v = np.frombuffer(bytearray(4 * len(a) + 1), dtype=np.int32, offset=1, count=len(a))
    v[:] = a
    return v


@pytest.mark.parametrize("form", [lambda a: (i32 * len(a))(*a), lambda a: np.array((i32 * len(a))(*a)), unaligned, lambda a: unaligned(a + [7])[:len(a)],
                                  lambda a: memoryview(np.array(a, np.int32)), lambda a: np.array([(x, 1) for x in a], [("a", "i4"), ("b", "i1")])["a"]])
@pytest.mark.parametrize("which", range(3))
def test_int32_lengths_whose_buffers_name_their_type_otherwise(calls, form, which):
    """Unaligned arrays and ctypes arrays describe int32 as "=i" and "<i"."""
    t = tensors()
    lengths = [form(a) if j == which else a for j, a in enumerate(LENGTHS)]
    binding._marshal.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], *lengths, None, None, 0.5, t["out"], 9)
    assert [c[2] for c in calls] == [LENGTHS]


def test_addresses_none_and_streams(calls):
    class Stream:
        cuda_stream = 123
    qs, ql, cl = LENGTHS
    m = binding._marshal
    m.kv_append(None, MAX_BLOCKS, None, 1 << 63, 4096, True, 8192, qs, ql, cl, 2 ** 40, 2 ** 31 + 5, 256, Stream())
    assert calls == [("append", (None, None, 1 << 63, 4096, 1, 8192), LENGTHS, (3, -2 ** 31 + 5, 2 ** 40, 256, 123))]


def call(t, **over):
    """attention(..) with one argument replaced."""
    a = {**t, "pages": None, "tokens": None, "stream": 9, **over}
    return binding._marshal.attention(11, MAX_BLOCKS, a["q"], a["k"], a["v"], a["table"], *LENGTHS, a["pages"], a["tokens"], 0.5, a["out"], a["stream"])


class Tensor:
    """What marshalling asks a tensor for."""

    def __init__(self, address=4096, shape=(7, 1)):
        self.address, self.shape = address, shape

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return self.address


class Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


class Parameter:
    def __init__(self, value):
        self._as_parameter_ = value


@pytest.mark.parametrize("over,at,value", [
    (dict(tokens=i32(6)), (3, 1), 6), (dict(tokens=np.int64(6)), (3, 1), 6), (dict(tokens=torch.tensor(6)), (3, 1), 6), (dict(tokens=Parameter(6)), (3, 1), 6),
    (dict(tokens=Parameter(i32(-6))), (3, 1), -6), (dict(pages=i64(2 ** 40)), (3, 2), 2 ** 40), (dict(pages=np.int32(5)), (3, 2), 5), (dict(pages=True), (3, 2), 1),
    (dict(k=Tensor(shape=(7.5, 1))), (3, 2), 7), (dict(k=Tensor(shape=(np.int64(7), 1))), (3, 2), 7), (dict(k=Tensor(shape=["7", 1])), (3, 2), 7),
    (dict(q=Tensor(None)), (1, 1), None), (dict(q=Tensor(vp(64))), (1, 1), 64), (dict(q=Tensor(Parameter(64))), (1, 1), 64),
    (dict(stream=Stream(None)), (3, 5), None), (dict(stream=Stream(vp(64))), (3, 5), 64), (dict(stream=Stream(True)), (3, 5), 1),
])
def test_integers_and_addresses_in_what_a_ctypes_call_takes(calls, over, at, value):
    call(tensors(), **over)
    assert calls[0][at[0]][at[1]] == value


@pytest.mark.parametrize("over", [
    dict(tokens=6.0), dict(tokens="6"), dict(tokens=i64(6)), dict(tokens=np.float32(6)), dict(pages=i32(7)), dict(pages=7.0), dict(pages=b"7"), dict(q=Tensor(np.int64(64))),
    dict(q=Tensor(64.0)), dict(q=Tensor(i64(64))), dict(stream=Stream(np.int64(5))), dict(stream=Stream(5.0)), dict(stream=Stream(i32(5))),
])
def test_integers_and_addresses_that_a_ctypes_call_refuses(calls, over):
    with pytest.raises(ctypes.ArgumentError):
        call(tensors(), **over)
    assert calls == []


@pytest.mark.parametrize("form", [list, lambda a: np.array(a, np.int32), unaligned])
def test_lengths_that_end_before_the_batch_are_refused(calls, form):
    """The C call reads as many of each as q_len has; more are taken, as buffers of a full batch are handed over."""
    t, m = tensors(), binding._marshal
    for j in (0, 2):
        for short in ([], LENGTHS[j][:2]):
            lengths = [form(short if i == j else a) for i, a in enumerate(LENGTHS)]
            with pytest.raises(ValueError, match="one for each sequence"):
                m.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], *lengths, None, None, 0.5, t["out"], 9)
            with pytest.raises(ValueError, match="one for each sequence"):
                m.kv_append(11, MAX_BLOCKS, t["k_new"], t["v_new"], t["k"], t["v"], t["table"], *lengths, None, None, t["ws"], 9)
    assert calls == []
    m.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], form(LENGTHS[0] + [9]), form(LENGTHS[1]), form(LENGTHS[2] + [9, 9]), None, None, 0.5, t["out"], 9)
    m.attention(11, MAX_BLOCKS, t["q"], t["k"], t["v"], t["table"], form(LENGTHS[0]), np.array(LENGTHS[1])[:, None], np.array([LENGTHS[2]]), None, None, 0.5, t["out"], 9)
    assert [c[2] for c in calls] == [LENGTHS, LENGTHS]
    h = binding.Handle(2, 1, 64, max_tokens=64, max_seqs=8, max_blocks_per_seq=MAX_BLOCKS)
    for call_with in (h.plan, binding.PreparedBatch):
        for j in (0, 2):
            with pytest.raises(ValueError, match="one for each sequence"):
                call_with(*(form(a[:2] if i == j else a) for i, a in enumerate(LENGTHS)))


def test_refusals(calls):
    t = tensors()
    m = binding._marshal

    def attend(**over):
        a = {**t, "lengths": LENGTHS[1], "scale": 0.5, "stream": None, **over}
        return m.attention(11, MAX_BLOCKS, a["q"], a["k"], a["v"], a["table"], LENGTHS[0], a["lengths"], LENGTHS[2], None, None, a["scale"], a["out"],
                           a["stream"], a["ws"])
    wide, short = torch.zeros(3, MAX_BLOCKS + 1, dtype=torch.int32), torch.zeros(2, MAX_BLOCKS, dtype=torch.int32)
    for bad in (dict(table=wide), dict(table=short), dict(table=wide[:, :MAX_BLOCKS]), dict(table=torch.zeros(3, dtype=torch.int32)),
                dict(q=t["q"].transpose(0, 1)), dict(k=t["k"][:, :, ::2])):
        with pytest.raises(ValueError):
            attend(**bad)
    for bad, error in ((dict(k=4096), AttributeError), (dict(lengths=object()), TypeError), (dict(q=object()), AttributeError), (dict(q=1.5), AttributeError)):
        with pytest.raises(error):
            attend(**bad)
    assert calls == []
    attend()
    assert len(calls) == 1
