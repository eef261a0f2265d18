"""GPU parity of the decode down projection of wide experts around its two
forms (one launch up to 24 MiB of weights, chunks and a reduction above) and
over the one-launch form's unit and row splits, bf16 and fp32.

The check reads y as the difference of two fp32 hidden states, which is off by
up to 2^-24 |h'| / |y| whatever the kernel does.  With N(0, 0.02^2) weights and
unit-rms input |y| is about 0.02 sqrt(d_ff) * 0.5 * 0.02^2 d, so the sizes keep
d large enough for that to stay below the bounds: at d 64, d_ff 2056 (bf16)
|y| is about 0.012, 7e-6 against 1e-4; at d 200, d_ff 1032 (fp32) 0.026, 3e-6
against 1e-5 (at d 8 it would be 1e-4)."""
import numpy as np
import pytest

from paper_2511_05814_amd import workload as wl
from tests._gpu_rig import Rig, _say, _tol
from tests._parity import check_decode

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,top_k,d,d_ff", [
    ("bf16", 1, 64, 2056), ("bf16", 2, 72, 2064), ("bf16", 3, 264, 3592), ("bf16", 5, 136, 4096), ("bf16", 2, 520, 14336),
    ("bf16", 7, 1032, 2568), ("bf16", 1, 1024, 12288), ("bf16", 1, 1032, 12288), ("f32", 1, 200, 1032), ("f32", 3, 264, 2056),
    ("f32", 2, 1024, 3072), ("f32", 2, 1032, 3072)])
def test_wide_down(dtype, top_k, d, d_ff):
    run(dtype, top_k, d, d_ff)


def one_launch(dtype, top_k, d, d_ff):
    """Rows of h a workgroup owns and column steps of a unit, as the one-launch
    form chooses them."""
    elem = 4 if dtype == "f32" else 2
    steps = -(-d_ff // (64 * 16 // elem))
    assert steps > 4 and top_k * d * d_ff * elem <= 24 << 20, "this size takes another kernel"
    cost = {n: -(-top_k * -(-steps // n) // 8) * (n + 0.5) for n in range(8, 0, -1)}
    return max(2, -(-d // 512)), min(cost, key=cost.get)


@pytest.mark.parametrize("dtype,top_k,d,d_ff,rows,steps", [
    ("bf16", 1, 4096, 2568, 8, 1), ("f32", 1, 4096, 1288, 8, 1), ("bf16", 1, 2056, 4104, 5, 2), ("f32", 2, 2056, 1288, 5, 2),
    ("bf16", 1, 1040, 9000, 3, 3), ("bf16", 3, 1040, 3592, 3, 4), ("bf16", 7, 360, 2056, 2, 5), ("bf16", 7, 520, 2568, 2, 6),
    ("bf16", 2, 264, 12808, 2, 7), ("bf16", 7, 264, 3592, 2, 8)])
def test_rows_and_units_of_the_one_launch_form(dtype, top_k, d, d_ff, rows, steps):
    # two to eight rows a workgroup (several trips through the row loop, two rows
    # at a time up to 3 steps and one above), a last workgroup with fewer, and
    # every unit length
    assert one_launch(dtype, top_k, d, d_ff) == (rows, steps)
    run(dtype, top_k, d, d_ff)


def run(dtype, top_k, d, d_ff):
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=top_k + 1, top_k=top_k, d_model=d, d_ff=d_ff, dtype=dtype, tokens=3)
    _say("wide down", dtype, top_k, d, d_ff)
    rig = Rig(cfg)
    moe = rig.cache(cfg.experts, "lfu")
    hs, recs, _ = rig.run(moe, cfg.tokens)
    check_decode(cfg, rig.model, hs, recs, cfg.experts, "lfu", prefetch=False, pmax=0, tol=_tol(cfg))
    moe.close()
    rig.store.close()
