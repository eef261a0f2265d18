"""GPU parity of the batched route and plan kernels at the sizes where their
split changes: token counts around a block of 16 and around the plan's
workgroup limit, 1 to 4 expert groups, column ranges and K tails of the gate."""
import pytest

from paper_2511_05814_amd import workload as wl
from tests._gpu_rig import Rig, _say
from tests.test_gpu_prefill import prefill_and_check

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


def check(experts, top_k, slots, d, T, policy="lfu"):
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=experts, top_k=top_k, d_model=d, d_ff=64, dtype="bf16", tokens=1,
                                         prefill_tokens=T)
    _say("route", experts, top_k, slots, d, T, policy)
    rig = Rig(cfg)
    moe = rig.cache(slots, policy, max_prefill_tokens=T + 3)
    prefill_and_check(rig, moe, policy, slots, T, sorted({0, T // 2, T - 1}))
    moe.close()
    rig.store.close()


@pytest.mark.parametrize("T", [1, 15, 16, 17, 255, 257, 1025])
@pytest.mark.parametrize("experts,top_k", [(3, 1), (16, 16), (17, 4), (33, 8), (49, 5), (64, 16)])
def test_token_and_expert_edges(T, experts, top_k):
    # every expert resident, and (LRU, whose key needs each expert's last pair)
    # the smallest number of slots
    check(experts, top_k, experts, 136, T)
    check(experts, top_k, top_k, 136, T, "lru")


@pytest.mark.parametrize("d", [8, 40, 256, 520, 1032, 2056, 4096, 4104])
def test_column_edges(d):
    # one range of a few columns up to 32 ranges; rows within and beyond the
    # columns a wave keeps in registers (512, 1024, 2048, 4096)
    check(20, 3, 20, d, 18)


@pytest.mark.parametrize("T", [1, 13, 16])
@pytest.mark.parametrize("d", [40, 512, 520, 1024, 1032, 2048, 2056, 4104])
def test_one_block(d, T):
    # at most 16 tokens: route and plan in one launch up to 2048 columns (rows
    # held in 2, 4 or 8 registers a lane), in two above.  40 columns at least:
    # rounding x and act to bf16 alone puts a row of 40 off by 2.9e-3 (median)
    # and 5.6e-3 (one in 1000), a row of 8, whose few errors do not average, by
    # 2.9e-3 and 1.2e-2 (fp64 arithmetic on N(0, 0.02^2) weights), against a
    # bound of 6e-3
    check(20, 3, 20, d, T)


@pytest.mark.parametrize("T", [17, 31, 32])
@pytest.mark.parametrize("experts,d", [(20, 40), (32, 512), (20, 520), (32, 1024), (20, 1032), (20, 2048), (20, 2056),
                                       (33, 520)])
def test_two_blocks(experts, d, T):
    # 17 to 32 tokens: one launch up to 1024 columns (2048 with experts as small
    # as these) and 32 experts, a wave taking a token of each block (whole and
    # partial second blocks)
    check(experts, 3, experts, d, T)


def test_more_blocks_than_plan_workgroups():
    # 67 x 1024 pairs: the plan kernel's 64 workgroups take more than one pair a thread
    check(16, 16, 16, 64, 4300)
