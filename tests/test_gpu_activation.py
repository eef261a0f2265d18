"""The batch path's activation does not depend on how a batch is cut: with one
non-zero weight a row every sum is exact, so tiles and small-M kernels have to
give the same bits (SiLU(v) u rounded to bf16, from the same fp32 quotient)."""
import numpy as np
import pytest

from paper_2511_05814_amd import workload as wl
from tests._gpu_rig import _say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T", [40, 1024])
def test_tiles_match_small_m(T):
    from paper_2511_05814_amd import offload
    n = 4096
    cfg = wl.CONFIGS["tiny-stack"].with_(layers=1, experts=1, top_k=1, d_model=n, d_ff=n, dtype="bf16", tokens=1,
                                         prefill_tokens=T)
    _say("activation", T)
    rng = np.random.default_rng(7)
    store = offload.HostStore(cfg, fill=False)
    w = store.layer_array(0).reshape(-1).view(np.uint16).reshape(3, n, n)
    w[:] = 0
    i = np.arange(n)
    for j, scale in enumerate((rng.standard_normal(n) * 2, rng.standard_normal(n), np.ones(n))):
        w[j, i, i] = wl.f32_to_bf16_bits(scale.astype(np.float32))
    moe = offload.OffloadedMoE(cfg, store, offload.DeviceGates(cfg), 1, "lfu", max_prefill_tokens=T)
    h = torch.from_numpy(rng.standard_normal((T, n)).astype(np.float32)).cuda()
    torch.cuda.synchronize()
    whole, parts = h.clone(), h.clone()
    with torch.cuda.stream(moe.compute):
        moe.prefill(whole)
        for t in range(0, T, 16):
            moe.prefill(parts[t:t + 16])
    moe.sync()
    assert not torch.equal(whole, h)
    differ = int((whole != parts).sum())
    moe.close()
    store.close()
    assert differ == 0
