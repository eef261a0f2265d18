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
    # and, from 49 rows on, wide ones; 17 and 31 rows take the small-M kernels
    check(d, d_ff, 3, [17, 31, 48, 49, 100])


@pytest.mark.parametrize("d,d_ff", [(48, 200), (64, 64), (136, 192), (192, 136), (320, 264)])
def test_tiles_of_few_rows(d, d_ff):
    # more than 32 tokens, so tiles, but one expert a token of 4: tiles of one
    # row block over one to five slices.  (Rounding x and act to bf16 alone,
    # in fp64 arithmetic, puts the worst of these rows off by 4.4e-3 at 48 by
    # 200, but by 6.2e-3 at 40 by 72, above the bound of 6e-3: the errors of few
    # columns do not average.)
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=4, top_k=1, d_model=d, d_ff=d_ff, dtype="bf16", tokens=1,
                                         prefill_tokens=40)
    _say("tiles of few rows", d, d_ff)
    rig = Rig(cfg)
    moe = rig.cache(4, "lfu", max_prefill_tokens=40)
    prefill_and_check(rig, moe, "lfu", 4, 40, list(range(0, 40, 3)))
    moe.close()
    rig.store.close()


@pytest.mark.parametrize("T", [16, 17, 31, 32])
@pytest.mark.parametrize("d,d_ff", [(40, 200), (136, 72), (264, 520)])
def test_small_m_row_blocks(d, d_ff, T):
    # too few tiles for the chip, so the small-M kernels: one full 16-row block
    # and two, each with a K tail
    check(d, d_ff, 3, [T])


@pytest.mark.parametrize("d,d_ff", [(520, 4104), (4104, 520), (512, 4104), (4104, 512)])
def test_one_launch_of_tiles_one_of_small_m(d, d_ff):
    # 4 experts, all rows of every token: 260 narrow tiles one way and 20 the
    # other, of weight rows on 128-byte lines and across them
    check(d, d_ff, 4, [17, 32])


@pytest.mark.parametrize("d,d_ff", [(448, 4104), (456, 4104), (392, 4104)])
def test_weight_rows_on_and_across_lines(d, d_ff):
    # 24 tokens of top-1 over 8 experts: up takes tiles (528 narrow) but for rows of
    # 400 columns and more that are no multiple of 64
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=8, top_k=1, d_model=d, d_ff=d_ff, dtype="bf16", tokens=1,
                                         prefill_tokens=24)
    _say("rows across lines", d, d_ff)
    rig = Rig(cfg)
    moe = rig.cache(8, "lfu", max_prefill_tokens=24)
    prefill_and_check(rig, moe, "lfu", 8, 24, list(range(24)))
    moe.close()
    rig.store.close()


@pytest.mark.parametrize("T", [20, 32, 40])
@pytest.mark.parametrize("slots", [2, 5])
def test_host_planned_small_m(T, slots):
    # groups whose experts have a few to some 30 rows, resident and streamed
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=6, top_k=2, d_model=136, d_ff=200, dtype="bf16", tokens=1,
                                         prefill_tokens=T)
    _say("host-planned small-M", T, slots)
    rig = Rig(cfg)
    moe = rig.cache(slots, "lfu", max_prefill_tokens=T)
    prefill_and_check(rig, moe, "lfu", slots, T, list(range(T)))
    moe.close()
    rig.store.close()


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
