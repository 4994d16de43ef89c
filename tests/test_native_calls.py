"""The binding's native argument conversion against its general one, on the CPU: every form of arguments that is accepted gives the
same results and tables either way, and what is refused is refused by both."""
import sysconfig

import numpy as np
import pytest
import torch

import paper_2506_15155_amd as E
from paper_2506_15155_amd import binding

NATIVE = ("decode", "append_decode", "append", "premap_next")
REAL = binding._calls


class Nothing:
    """In the place of the native calls: handles no form."""

    def __getattr__(self, name):
        return (lambda *a: None) if name in NATIVE else getattr(REAL, name)


class Address:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


def forms(values):
    a = np.asarray(values, np.int32)
    wide = np.zeros(2 * len(a), np.int32)
    wide[::2] = a
    fixed = a.copy()
    fixed.flags.writeable = False
    return {"array": a, "list": list(values), "int64": a.astype(np.int64), "int16": a.astype(np.int16), "strided": wide[::2],
            "read-only": fixed, "two dimensions": a.reshape(1, -1), "swapped": a.astype(a.dtype.newbyteorder()),
            "unsigned": a.astype(np.uint32), "subclass": a.view(np.recarray), "tensor": torch.tensor(a), "tuple": tuple(values)}


FORMS = list(forms([0]))
POINTERS = {"int": 0x1000, "none": None, "object": Address(0x2000), "tensor": torch.zeros(4, dtype=torch.bfloat16), "numpy": np.zeros(4, np.uint16),
            "numpy int": np.int64(0x1000), "bool": True, "text": "x", "huge": 1 << 70, "negative": -16, "method": Address("x")}


def walk(ids_form, n_form, pointer, stream):
    """What a sequence of calls returns or raises, and the tables afterwards."""
    P = E.ellm_pool_create(None, None, 1 << 14, 8, 2, 128, 4, 4, flags=1, device_bytes=12 << 14)
    for _ in range(3):
        E.ellm_tensor_create(P, 48)
    seen = []

    def call(f, *a, **k):
        try:
            seen.append(f(P, *a, **k))
        except Exception as e:
            seen.append((type(e).__name__, getattr(e, "code", None)))

    ids = lambda *v: forms(v)[ids_form]
    p = POINTERS[pointer]
    call(E.ellm_kv_premap_next, ids(0, 1, 2))
    call(E.ellm_kv_premap_next, ids(0, 1, 2), flags=1, check=False)
    call(E.ellm_kv_append, ids(0, 2), p, 0x3000, forms([3, 5])[n_form], stream=stream)
    call(E.ellm_kv_append, ids(1), 0x3000, p, stream=stream)
    call(E.ellm_kv_append, ids(1, 1), 0x3000, 0x3000, stream=stream, check=False)
    call(E.ellm_kv_append, ids(9), 0x3000, 0x3000, stream=stream)
    for f in (E.ellm_decode_attention, E.ellm_decode_attention_noalloc):
        for scale in (0.0, 1, np.float32(0.5), float("inf"), "x"):
            call(f, ids(0, 2), p, 0x3000, scale=scale, stream=stream)
        call(f, ids(0, 2), 0x3000, p, stream=stream, check=False)
    call(E.ellm_kv_append_decode, ids(0), p, 0x3000, 0x3000, 0x3000, stream=stream)
    call(E.ellm_kv_append_decode, ids(0), 0x3000, 0x3000, 0x3000, p, 0.5, stream=stream, check=False)
    call(E.ellm_kv_premap_next, ids(0, 7))
    tables = [(list(t), n) for t, n in (E.ellm_tensor_get_table(P, i) for i in range(3))]
    E.ellm_pool_destroy(P)
    return seen, tables


@pytest.mark.parametrize("ids_form,n_form,pointer,stream",
                         [(f, "array", "int", 0) for f in FORMS] + [("array", f, "object", 0) for f in FORMS] +
                         [("array", "array", p, 0) for p in POINTERS] + [("array", "array", "tensor", s) for s in (None, 7, Address(1), "x")])
def test_the_same_either_way(monkeypatch, ids_form, n_form, pointer, stream):
    native = walk(ids_form, n_form, pointer, stream)
    monkeypatch.setattr(binding, "_calls", Nothing())
    assert walk(ids_form, n_form, pointer, stream) == native


def test_the_stand_in_passes_on_what_it_does_not_replace(monkeypatch):
    """With torch up, the general way hands torch's names to the native module: as it is, and not to the stand-in for ever."""
    monkeypatch.setattr(binding, "_calls", Nothing())
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x1230, raising=False)
    assert binding._stream(None) == 0x1230


def test_the_native_module_is_this_interpreters():
    """Built for another one, it is missing and not loaded as it is."""
    assert binding._calls.__file__ == binding.CALLS_PATH and binding.CALLS_PATH.endswith("_calls" + sysconfig.get_config_var("EXT_SUFFIX"))


def test_plain_arguments_are_handled_natively():
    P = E.ellm_pool_create(None, None, 1 << 14, 8, 2, 128, 4, 4, flags=1, device_bytes=12 << 14)
    E.ellm_tensor_create(P, 48)
    ids, t = np.zeros(1, np.int32), torch.zeros(4, dtype=torch.bfloat16)
    assert binding._calls.premap_next(P, ids, 0) == 1
    assert binding._calls.append(P, ids, t, t, None, 0) == 0 and binding._calls.append(P, ids, t, t, ids + 2, 0) == 0
    assert binding._calls.decode(False, P, ids, t, t, 0.0, 0) == E.ERR.NO_DEVICE == binding._calls.decode(True, P, ids, t, t, 0.0, 0)
    assert binding._calls.append_decode(P, ids, t, t, t, t, 0.0, 0) == E.ERR.NO_DEVICE
    assert E.ellm_tensor_get_table(P, 0)[1] == 3
    with pytest.raises(TypeError):
        binding._calls.decode(P, ids)
    E.ellm_pool_destroy(P)


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("form", ["array", "list", "int64"])
def test_arrays_shorter_than_their_count_are_refused(monkeypatch, native, form):
    """Token counts for fewer requests than are named, chunks for fewer slots, owners for fewer chunks: nothing behind the array
    is read, and nothing changes. What is left over is ignored, as ever."""
    if not native:
        monkeypatch.setattr(binding, "_calls", Nothing())
    P = E.ellm_pool_create(None, None, 1 << 14, 8, 2, 128, 4, 4, flags=1, device_bytes=12 << 14)
    ids = np.arange(3, dtype=np.int32)
    for _ in ids:
        E.ellm_tensor_create(P, 48)
    E.ellm_kv_premap_next(P, ids)
    tables = lambda: [(list(t), n) for t, n in (E.ellm_tensor_get_table(P, i) for i in range(3))]
    before = tables()
    some = np.array([1, 2, 3, 1], np.int32)                 # (the numbers behind the array would be taken for counts)
    for n in (0, 1, 2):
        for check in (True, False):
            with pytest.raises(ValueError):
                E.ellm_kv_append(P, ids, 0x3000, 0x3000, forms(some)["array"][:n] if form == "array" else forms(some[:n])[form], stream=0, check=check)
    with pytest.raises(ValueError):
        E.ellm_tensor_map_chunks(P, 0, 1, 2, forms([7])[form])
    with pytest.raises(ValueError):
        E.ellm_chunk_inflate_from_host(P, 0, 0, 2, forms([7])[form])
    with pytest.raises(ValueError):
        E.ellm_pool_create(None, None, 1 << 14, 8, 2, 128, 4, 4, initial_owner=[0] * 11, flags=1, device_bytes=12 << 14)
    assert tables() == before and E.ellm_pool_self_check(P) == 0
    assert E.ellm_kv_append(P, ids, 0x3000, 0x3000, forms(some)[form], stream=0) == 0
    assert [n for _, n in tables()] == [1, 2, 3]
    E.ellm_pool_destroy(P)


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_no_stream_is_torchs_current_one(monkeypatch, native):
    """While a stream is captured: what is called without a stream is recorded there, and runs when the graph does."""
    tokens, kv, dim, n = 64, 2, 64, 3
    cb = tokens * 4 * kv * dim
    dev = torch.empty(4 * n * cb, dtype=torch.uint8, device="cuda")
    pool = E.ellm_pool_create(dev, None, cb, kv, kv, dim, n, 4)
    ids = np.array([E.ellm_tensor_create(pool, 4 * tokens) for _ in range(n)], np.int32)
    for i in ids:
        E.ellm_tensor_map_chunks(pool, int(i), 0, 4)
    rows = torch.randn(100 * n, kv, dim, device="cuda").to(torch.bfloat16)
    E.ellm_kv_append(pool, ids, rows, rows, np.full(n, 100, np.int32))
    q = torch.randn(n, kv, dim, device="cuda").to(torch.bfloat16)
    want = torch.empty_like(q)
    E.ellm_decode_attention(pool, ids, q, want)
    torch.cuda.synchronize()
    if not native:
        monkeypatch.setattr(binding, "_calls", Nothing())
    outs = torch.zeros(2, *q.shape, dtype=q.dtype, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        if native:
            assert binding._calls.decode(False, pool, ids, q, outs[0], 0.0, None) == 0
        E.ellm_decode_attention(pool, ids, q, outs[0])
        E.ellm_decode_attention_noalloc(pool, ids, q, outs[1])
    torch.cuda.synchronize()
    assert not outs.any()
    for _ in range(3):
        outs.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[0], want) and torch.equal(outs[1], want)
    E.ellm_pool_destroy(pool)
