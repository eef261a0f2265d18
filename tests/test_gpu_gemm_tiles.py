"""GPU parity of the grouped-GEMM tiles at the sizes where they change shape.

Every expert is selected by every token (top_k = experts), so each expert has
exactly as many rows as the batch has tokens, and enough column blocks keep the
planner at one tile per expert and column block: T walks the tile through its
row-block counts (1 to 8 blocks of 32 rows), both sides of each edge.
"""
import numpy as np
import pytest

from paper_2511_05814_amd import workload as wl
from tests._gpu_rig import Rig, _say
from tests.test_gpu_prefill import prefill_and_check

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")

EDGES = [17, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257]


def check(d, d_ff, experts, tokens, slots=None):
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=experts, top_k=experts, d_model=d, d_ff=d_ff, dtype="bf16",
                                         tokens=1, prefill_tokens=max(tokens))
    rig = Rig(cfg)
    slots = experts if slots is None else slots
    for T in tokens:
        _say("tiles", d, d_ff, experts, T)
        moe = rig.cache(slots, "lfu", max_prefill_tokens=T)
        prefill_and_check(rig, moe, "lfu", slots, T, sorted({0, 31, T // 2, T - 2, T - 1} & set(range(T))))
        moe.close()
    rig.store.close()


def test_up_tile_heights():
    # 321 column blocks up, reduction over 72 columns: a K tail of one chunk in
    # the second slice; down reduces over 40968 (a K tail) with one column block
    check(72, 40968, 1, EDGES)


def test_down_tile_heights():
    # 64 column blocks x 4 experts down, reduction over 72; up reduces over
    # 16384 whole slices with one partial column block
    check(16384, 72, 4, EDGES)


@pytest.mark.parametrize("d,d_ff", [(8, 8), (64, 64), (136, 192), (192, 136), (320, 264)])
def test_small_and_ragged_tiles(d, d_ff):
    # one to five slices (fewer than the ring holds, with and without a K
    # tail), partial column blocks, narrow tiles (at most 48 rows an expert)
    # and, from 49 rows on, wide ones
    check(d, d_ff, 3, [17, 31, 48, 49, 100])


@pytest.mark.parametrize("T", [300, 384])
@pytest.mark.parametrize("slots", [2, 8])
def test_experts_of_one_and_of_several_short_tiles(T, slots):
    # one expert a token, chosen unevenly: at most 48 rows an expert on average,
    # so narrow tiles, of which experts with more than 64 rows take several
    # (weights read by more than one tile) and the others one
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=8, top_k=1, d_model=136, d_ff=192, dtype="bf16", tokens=1,
                                         prefill_tokens=T)
    _say("short tiles", T, slots)
    rig = Rig(cfg)
    moe = rig.cache(slots, "lfu", max_prefill_tokens=T)
    prefill_and_check(rig, moe, "lfu", slots, T, list(range(0, T, 7)))
    moe.close()
    rig.store.close()
