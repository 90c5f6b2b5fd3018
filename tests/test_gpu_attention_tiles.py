"""Attention at the edges of its small row tiles (32 and 64 rows whose
wavefronts split the keys) and of the rule that picks them: rows around a
tile, key counts around a unit of 32 and a round of 8 units, KV-head counts
that leave XCDs uneven, splits with short last ranges; against the oracle."""
import pytest

from tests.gpu_util import LayerCase, assert_attention_close, from_dev, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()
    import torch
    torch.cuda.synchronize()
    yield
    torch.cuda.synchronize()


# (nq, nkv, d, prefix tokens (a multiple of 8), suffix tokens)
CASES = [
    # rows below, at and above one 32-row tile
    *[(4, 1, 128, 40, t) for t in (1, 7, 8, 9)], *[(6, 2, 64, 40, t) for t in (1, 10, 11)],
    (3, 3, 64, 24, 31), (3, 3, 64, 24, 32), (5, 5, 128, 24, 33),
    # key counts around one unit, one round of the 8 wavefronts and two; an odd
    # number of prefix pages puts prefix and suffix into one unit
    *[(8, 2, 128, tp, 3) for tp in (0, 8, 16, 24, 32, 240, 248, 256, 264, 520)],
    *[(8, 2, 64, tp, 5) for tp in (0, 8, 232, 256, 1000)],
    # several splits (few tiles, long prefix), the last one short
    (4, 1, 128, 4104, 2), (8, 8, 64, 8200, 1), (2, 1, 64, 20008, 1), (16, 2, 128, 6000, 20),
    # 64-row tiles: d = 128 with Q in LDS, d = 64 with Q in registers
    (32, 8, 128, 104, 400), (64, 8, 128, 1000, 200), (64, 8, 128, 104, 197), (32, 4, 64, 3000, 200),
    (12, 4, 64, 104, 1003), (40, 8, 128, 808, 201), (32, 4, 64, 8200, 200), (32, 8, 128, 16392, 64),
    (8, 8, 64, 30000, 100),
    # 256-row tiles with KV-head and split counts that are no multiple of 8
    (24, 3, 128, 2000, 700), (20, 5, 64, 4000, 1500), (8, 1, 128, 4000, 1200),
    # one query head per KV head, and many
    (16, 16, 64, 72, 50), (64, 1, 128, 264, 9), (48, 3, 128, 488, 30),
]


@pytest.mark.parametrize("nq,nkv,d,Tp,Ts", CASES)
def test_small_tiles_match_oracle(nq, nkv, d, Tp, Ts):
    import torch
    print(f"[attention tiles] nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}", flush=True)
    need = max(1, -(-Tp // 16))
    c = LayerCase(nq, nkv, d, 8, 16, Tp // 8, Ts, need + 5, 2, 1, seed=Tp + Ts).upload()
    if Tp:
        c.run_ingest()
    out = c.run_attention()
    torch.cuda.synchronize()
    rows = None if Ts * (Tp + Ts) * nq < 2_000_000 else sorted({0, 1, Ts // 3, Ts // 2, Ts - 2, Ts - 1} & set(range(Ts)))
    got = from_dev(out)
    assert_attention_close(got if rows is None else got[rows], c.expected_attention(rows=rows),
                           f"nq {nq} nkv {nkv} d {d} Tp {Tp} Ts {Ts}")


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
