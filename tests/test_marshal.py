"""The binding's native argument marshalling, against recording stand-ins for
the library's functions: every field of every struct arrives where the C
declaration has it, and what is no int, tensor or layout is refused."""
import ctypes
from ctypes import CFUNCTYPE, POINTER, c_int, c_int32, c_int64, c_size_t, c_void_p

import pytest

import paper_2605_22850_amd as oc
from paper_2605_22850_amd import _lib

P = {"st": POINTER(_lib.c_staging), "bt": POINTER(_lib.c_block_table), "kp": POINTER(_lib.c_kv_pool),
     "lay": POINTER(_lib.c_layout), "w": POINTER(_lib.c_layer_weights), "b": POINTER(_lib.c_layer_buffers)}
SIGS = {
    "oc_kv_layer_ingest": (P["st"], P["bt"], P["kp"], c_int32, c_void_p),
    "oc_kv_chunks_ingest": (P["st"], c_int64, P["bt"], P["kp"], c_void_p),
    "oc_kv_layer_gather": (P["bt"], P["kp"], c_int32, c_void_p, c_int64, c_int64, c_void_p),
    "oc_kv_chunks_gather": (P["bt"], P["kp"], c_int64, c_int64, c_void_p, c_void_p),
    "oc_kv_suffix_append": (c_void_p, c_void_p, c_int64, P["bt"], P["kp"], c_int32, c_void_p),
    "oc_suffix_prefill_layer": (c_void_p, c_void_p, c_void_p, c_int64, P["kp"], P["bt"], c_int32, c_void_p, c_void_p,
                                c_size_t, c_void_p),
    "oc_suffix_prefill_layer_noalloc": (c_void_p, c_void_p, c_void_p, c_int64, P["kp"], P["bt"], c_int32, c_void_p,
                                        c_void_p),
    "oc_rest_of_layer": (c_void_p, c_int64, P["lay"], P["w"], c_int32, P["b"], c_void_p),
}


class Tensor:
    def __init__(self, ptr, numel=1, size=2):
        self.ptr, self.n, self.size = ptr, numel, size

    def data_ptr(self):
        return self.ptr

    def numel(self):
        return self.n

    def element_size(self):
        return self.size


def plain(v):
    if isinstance(v, ctypes._Pointer):
        return plain(v.contents)
    if isinstance(v, ctypes.Structure):
        return {f[0]: plain(getattr(v, f[0])) for f in v._fields_}
    return v


@pytest.fixture
def calls():
    m = _lib._native()
    seen, keep = [], []
    for name in _lib._FAST:
        cb = CFUNCTYPE(c_int, *SIGS[name])(lambda *a, name=name: seen.append((name, [plain(x) for x in a])) or 0)
        keep.append(cb)
    m.bind(lambda: 0x5150, *(ctypes.cast(cb, c_void_p).value for cb in keep))
    try:
        yield seen
    finally:
        m.bind(_lib._current_stream, *(ctypes.cast(getattr(_lib.lib(), f), c_void_p).value for f in _lib._FAST))


LAY = oc.Layout(3, 8, 2, 64, 16, 32, 1 << 33)
LAY_C = {"num_layers": 3, "num_q_heads": 8, "num_kv_heads": 2, "head_dim": 64, "page_size": 16, "chunk_tokens": 32,
         "num_pages": 1 << 33}
S = 2 * 32 * 2 * 64 * 2
POOL = {"base": 0x7000, "layout": LAY_C}
TABLE = {"pages": 0x300, "num_entries": 9, "num_tokens": 130}


class Stream:
    cuda_stream = 0x99


def test_every_argument_arrives(calls):
    t, pages, pool = Tensor, Tensor(0x300, 9, 4), Tensor(0x7000)
    oc.oc_kv_layer_ingest(t(0x10), 4, pages, 130, pool, LAY, 2)
    oc.oc_kv_chunks_ingest(t(0x11), 4, 5, pages, 130, pool, LAY, stream=7)
    oc.oc_kv_layer_gather(pages, 130, pool, LAY, 1, t(0x12), 4, stream=Stream())
    oc.oc_kv_chunks_gather(pages, 130, pool, LAY, 6, 7, t(0x13))
    oc.oc_kv_suffix_append(t(0x14), t(0x15), 21, pages, 130, pool, LAY, 2)
    oc.oc_suffix_prefill_layer(t(0x16), t(0x17), t(0x18), 21, pool, LAY, pages, 130, 2, t(0x19), t(0x1a, 100, 4))
    oc.oc_suffix_prefill_layer_noalloc(t(0x16), t(0x17), t(0x18), 21, pool, LAY, pages, 130, 2, t(0x19))
    w = oc.LayerWeights(48, t(0x20), t(0x21), t(0x22), t(0x23))
    oc.oc_rest_of_layer(t(0x24), 21, LAY, w, 1, t(0x25), t(0x26), t(0x27), t(0x28), t(0x29))
    cur = 0x5150

    def st(p):
        return {"data": p, "num_chunks": 4, "per_layer_chunk_bytes": S}
    assert calls == [
        ("oc_kv_layer_ingest", [st(0x10), TABLE, POOL, 2, cur]),
        ("oc_kv_chunks_ingest", [st(0x11), 5, TABLE, POOL, 7]),
        ("oc_kv_layer_gather", [TABLE, POOL, 1, 0x12, 4, S, 0x99]),
        ("oc_kv_chunks_gather", [TABLE, POOL, 6, 7, 0x13, cur]),
        ("oc_kv_suffix_append", [0x14, 0x15, 21, TABLE, POOL, 2, cur]),
        ("oc_suffix_prefill_layer", [0x16, 0x17, 0x18, 21, POOL, TABLE, 2, 0x19, 0x1a, 400, cur]),
        ("oc_suffix_prefill_layer_noalloc", [0x16, 0x17, 0x18, 21, POOL, TABLE, 2, 0x19, cur]),
        ("oc_rest_of_layer", [0x24, 21, LAY_C, {"ffn_dim": 48, "w_o": 0x20, "w_gate_up": 0x21, "w_down": 0x22,
                                                "w_qkv": 0x23}, 1,
                              {"o": 0x25, "gate_up": 0x26, "act": 0x27, "h": 0x28, "qkv": 0x29}, cur]),
    ]


def test_none_and_empty_tables_are_null(calls):
    oc.oc_kv_layer_ingest(None, 0, None, 0, None, LAY, 0)
    oc.oc_kv_layer_ingest(None, 0, Tensor(0x300, 0), 0, None, LAY, 0)
    empty = {"pages": None, "num_entries": 0, "num_tokens": 0}
    for _, a in calls:
        assert a[0]["data"] is None and a[1] == empty and a[2]["base"] is None


def test_refused_arguments(calls):
    t, pages, pool = Tensor, Tensor(0x300, 9, 4), Tensor(0x7000)
    for bad in (1.0, "4", None):
        with pytest.raises(TypeError):
            oc.oc_kv_layer_ingest(t(0x10), bad, pages, 130, pool, LAY, 2)
        with pytest.raises(TypeError):
            oc.oc_kv_layer_ingest(t(0x10), 4, pages, 130, pool, LAY, bad)
    with pytest.raises(AttributeError):
        oc.oc_kv_layer_ingest(object(), 4, pages, 130, pool, LAY, 2)
    with pytest.raises(AttributeError):
        oc.oc_kv_layer_ingest(t(0x10), 4, pages, 130, pool, object(), 2)
    with pytest.raises(AttributeError):
        oc.oc_suffix_prefill_layer(t(1), t(2), t(3), 1, pool, LAY, pages, 130, 0, t(4), None)
    assert calls == []


def test_integers_that_are_no_int(calls):
    """Counts and layout fields are taken as ctypes takes them: whatever has
    __index__, such as a NumPy integer or an integer tensor of one element."""
    import numpy as np
    import torch
    t, pages, pool = Tensor, Tensor(0x300, np.int64(9), 4), Tensor(0x7000)
    for num in (np.int32, np.int64, lambda v: np.array([v])[0], torch.tensor, lambda v: torch.tensor([v])):
        lay = oc.Layout(*(num(f) for f in (3, 8, 2, 64, 16, 32, 1 << 20)))
        lay_c = dict(LAY_C, num_pages=1 << 20)
        p = {"base": 0x7000, "layout": lay_c}
        st = {"data": 0x10, "num_chunks": 4, "per_layer_chunk_bytes": S}
        calls.clear()
        oc.oc_kv_layer_ingest(t(0x10), num(4), pages, num(130), pool, lay, num(2))
        oc.oc_kv_chunks_ingest(t(0x10), num(4), num(5), pages, num(130), pool, lay)
        oc.oc_kv_layer_gather(pages, num(130), pool, lay, num(1), t(0x12), num(4))
        oc.oc_kv_chunks_gather(pages, num(130), pool, lay, num(6), num(7), t(0x13))
        oc.oc_kv_suffix_append(t(0x14), t(0x15), num(21), pages, num(130), pool, lay, num(2))
        oc.oc_suffix_prefill_layer(t(1), t(2), t(3), num(21), pool, lay, pages, num(130), num(2), t(4), t(5, 100, 4))
        oc.oc_suffix_prefill_layer_noalloc(t(1), t(2), t(3), num(21), pool, lay, pages, num(130), num(2), t(4))
        w = oc.LayerWeights(num(48), t(0x20), t(0x21), t(0x22), t(0x23))
        oc.oc_rest_of_layer(t(6), num(21), lay, w, num(1), t(7), t(8), t(9), t(10), t(11))
        cur = 0x5150
        assert calls == [
            ("oc_kv_layer_ingest", [st, TABLE, p, 2, cur]),
            ("oc_kv_chunks_ingest", [st, 5, TABLE, p, cur]),
            ("oc_kv_layer_gather", [TABLE, p, 1, 0x12, 4, S, cur]),
            ("oc_kv_chunks_gather", [TABLE, p, 6, 7, 0x13, cur]),
            ("oc_kv_suffix_append", [0x14, 0x15, 21, TABLE, p, 2, cur]),
            ("oc_suffix_prefill_layer", [1, 2, 3, 21, p, TABLE, 2, 4, 5, 400, cur]),
            ("oc_suffix_prefill_layer_noalloc", [1, 2, 3, 21, p, TABLE, 2, 4, cur]),
            ("oc_rest_of_layer", [6, 21, lay_c, {"ffn_dim": 48, "w_o": 0x20, "w_gate_up": 0x21, "w_down": 0x22,
                                                 "w_qkv": 0x23}, 1,
                                  {"o": 7, "gate_up": 8, "act": 9, "h": 10, "qkv": 11}, cur]),
        ]


def test_addresses(calls):
    """Pointers and stream handles: an int, None or a c_void_p; a NumPy integer
    is no address."""
    import numpy as np

    class Handle:
        def __init__(self, h):
            self.cuda_stream = h
    pages, pool = Tensor(0x300, 9, 4), Tensor(0x7000)
    for h, want in ((0x99, 0x99), (None, None), (0, None), (c_void_p(0x98), 0x98), (c_void_p(), None)):
        calls.clear()
        oc.oc_kv_layer_ingest(Tensor(0x10), 4, pages, 130, pool, LAY, 2, stream=Handle(h))
        assert calls[0][1][4] == want
    calls.clear()
    oc.oc_kv_layer_ingest(Tensor(c_void_p(0x10)), 4, pages, 130, Tensor(c_void_p()), LAY, 2)
    assert calls[0][1][0]["data"] == 0x10 and calls[0][1][2]["base"] is None
    calls.clear()
    with pytest.raises(TypeError):
        oc.oc_kv_layer_ingest(Tensor(0x10), 4, pages, 130, pool, LAY, 2, stream=Handle(np.int64(5)))
    with pytest.raises(TypeError):
        oc.oc_kv_layer_ingest(Tensor(np.int64(0x10)), 4, pages, 130, pool, LAY, 2)
    assert calls == []


def test_errors_carry_the_library_message():
    with pytest.raises(oc.OcError) as e:
        oc.oc_kv_layer_ingest(Tensor(0x10), 4, Tensor(0x300, 9, 4), 128, Tensor(0x7000), LAY, 3, stream=0)
    assert e.value.status == _lib.OC_ERANGE and "layer out of range" in str(e.value)


@pytest.mark.parametrize("rows", [slice(0, 3), slice(2, 3), slice(2, None, -3)])
def test_chunk_object_pointers(rows, monkeypatch):
    """One pointer per object; a single row counts as contiguous whatever its
    stride, negative ones included."""
    import numpy as np
    objects = np.zeros((3, 64), np.int16)[rows]
    n, seen = objects.shape[0], []

    class Library:
        def oc_pipeline_run(self, ctx, reqs, n_reqs, stats):
            seen.extend(reqs[0].chunk_objects[j] for j in range(n))
            return 0
    monkeypatch.setattr(_lib, "lib", Library)
    t = Tensor(0x10)
    oc.oc_pipeline_run(None, [oc.Request(16 * n, 1, Tensor(0x300, 9, 4), t, t, t, t, chunk_objects=objects)], 1)
    assert seen == [objects[j:].ctypes.data for j in range(n)]
