"""Attention at the edges of its row tiles (32 and 64 rows whose wavefronts
split the keys, 256 rows) and of the rule that picks them: rows around a tile,
key counts around a unit of 32 and a round of 8 units, KV-head counts that
leave XCDs uneven, splits with short last ranges, prefixes that end at any slot
of a page, alone and batched; against the oracle.  The CPU tests of the
dispatch check that every shape takes the kernel it stands for."""
import numpy as np
import pytest

from tests.attention_cases import BATCHES, BY_PLAN, RAGGED
from tests.gpu_util import LayerCase, RequestSet, assert_attention_close, from_dev, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()
    import torch
    torch.cuda.synchronize()
    yield
    torch.cuda.synchronize()


def _check(nq, nkv, d, Tp, Ts):
    """One layer, pages past the prefix full of NaN; the prefix is one chunk
    where it is no multiple of 8 tokens."""
    import torch
    print(f"[attention tiles] nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}", flush=True)
    need = max(1, -(-Tp // 16))
    G = 8 if Tp % 8 == 0 else Tp
    c = LayerCase(nq, nkv, d, G, 16, Tp // G, Ts, need + 5, 2, 1, seed=Tp + Ts).upload()
    if Tp:
        c.run_ingest()
    out = c.run_attention()
    torch.cuda.synchronize()
    tile = 256 // (nq // nkv)       # both sides of a 256-row tile's edge among the sampled rows
    rows = None if Ts * (Tp + Ts) * nq < 2_000_000 else \
        sorted({0, 1, tile - 1, tile, Ts // 3, Ts // 2, Ts - 2, Ts - 1} & set(range(Ts)))
    got = from_dev(out)
    assert_attention_close(got if rows is None else got[rows], c.expected_attention(rows=rows),
                           f"nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}")


@pytest.mark.parametrize("nq,nkv,d,Tp,Ts", [c for cases in BY_PLAN.values() for c in cases])
def test_small_tiles_match_oracle(nq, nkv, d, Tp, Ts):
    _check(nq, nkv, d, Tp, Ts)


@pytest.mark.parametrize("nq,nkv,d,Tp,Ts", [c for cases in RAGGED.values() for c in cases])
def test_prefixes_that_end_inside_a_page(nq, nkv, d, Tp, Ts):
    _check(nq, nkv, d, Tp, Ts)


@pytest.mark.parametrize("nq,nkv,d,Tp,Ts", [cases[-1] for cases in BY_PLAN.values()])
def test_a_call_repeats_itself_bit_for_bit(nq, nkv, d, Tp, Ts):
    import torch
    print(f"[attention tiles] twice: nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}", flush=True)
    G = 8 if Tp % 8 == 0 else Tp
    c = LayerCase(nq, nkv, d, G, 16, Tp // G, Ts, -(-Tp // 16) + 5, 1, 0, seed=Ts).upload()
    c.run_ingest()
    first = c.run_attention()
    for _ in range(4):
        again = c.run_attention()
        torch.cuda.synchronize()
        assert torch.equal(first.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nkv,Tp,Ts", [b[:4] for b in BATCHES])
def test_batched_launch_with_prefixes_that_end_inside_a_page(nq, nkv, Tp, Ts, d):
    import paper_2605_22850_amd as oc
    print(f"[attention tiles] batch nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}", flush=True)
    pages = sum(-(-t // 16) for t in Tp)
    rs = RequestSet(1, nq, nkv, d, Tp, Ts, pages + 9, seed=sum(Tp), G=1).upload(with_payload=True)
    ctx = rs.context(oc.OC_MODE_DEVICE_STAGED)
    try:
        oc.oc_pipeline_run(ctx, rs.reqs, 1)
    finally:
        oc.oc_context_destroy(ctx)
    assert np.array_equal(from_dev(rs.d_pool).reshape(rs.pool_shape()), rs.expected_pool())
    tile = 256 // (nq // nkv)
    for r, ts in enumerate(Ts):
        rows = sorted({0, 1, tile - 1, tile, ts // 2, ts - 2, ts - 1} & set(range(ts)))
        assert_attention_close(from_dev(rs.reqs[r].out)[0][rows], rs.expected_out(r, 0, rows=rows), f"request {r}")


@pytest.mark.parametrize("pow2", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tile", [32, 64, 256])
def test_registers_leave_room_for_an_ingest_wavefront(tile, d, pow2):
    """512 VGPRs per SIMD lane, handed out in eights: two attention wavefronts
    and one of the ingest that runs beside them."""
    import ctypes
    import paper_2605_22850_amd as oc
    print(f"[attention tiles] registers, tile {tile} d {d}", flush=True)
    attn, ingest = ctypes.c_int32(), ctypes.c_int32()
    oc.lib().oc_internal_registers(tile, d, pow2, ctypes.byref(attn), ctypes.byref(ingest))
    assert attn.value > 0 and ingest.value > 0
    assert 2 * (-(-attn.value // 8) * 8) + -(-ingest.value // 8) * 8 <= 512
