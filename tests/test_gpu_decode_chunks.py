"""Decode attention of small batches: the launcher takes 128 or 256 tokens a block where the grid is small, and the merge of the
partial states walks them in groups.  Contexts on and around the chunk edges and around the groups' turns (4 groups of 4 splits), against the
oracle, and against the pinned 512-token chunks, whose partial states are merged from fewer splits."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import SMALL, check_iteration, custom_workload

pytestmark = pytest.mark.gpu

EDGES = [0, 126, 127, 128, 255, 256, 257]


@pytest.mark.parametrize("hq,hkv,hd", [(8, 2, 64), (4, 4, 64), (4, 4, 128), (16, 2, 128)])
@pytest.mark.parametrize("longest", [500, 2046, 2047, 2048, 4400])      # 4, 16, 16, 17 and 35 splits of 128
def test_short_chunks(torch_mod, hq, hkv, hd, longest):
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL)
    wl = custom_workload("short_chunks", dims, prefill=[], decode=EDGES + [longest], n_pairs=0, prompt=3, resp=(2, 9))
    check_iteration(torch_mod, wl, f"128-token chunks Hq{hq} Hkv{hkv} hd{hd} longest {longest}")


@pytest.mark.parametrize("hq,hkv,hd", [(32, 8, 64), (16, 16, 128)])
def test_batches_on_both_sides_of_the_rule(torch_mod, hq, hkv, hd):
    """Up to 4096 blocks of 128 tokens and 10240 of 256: 11 requests of up to 2000 tokens are 1408 and 2816 blocks of 128, 33 requests 4224 and
    8448, which makes their chunks 256."""
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL)
    for n in (11, 33):
        ctx = [(i * 197) % 2000 for i in range(n - 1)] + [2000]
        wl = custom_workload("rule", dims, prefill=[], decode=ctx, n_pairs=0, prompt=3, resp=(2, 9))
        check_iteration(torch_mod, wl, f"{n} requests Hq{hq} Hkv{hkv} hd{hd}")


@pytest.mark.parametrize("hd", [64, 128])
def test_an_infinite_value_stays_in_its_head(torch_mod, hd):
    """An infinite cached value makes its own element infinite (the norm of its head shows it: an infinity, not a NaN), wherever among the
    splits of its request it lies: alone, first, last, and in splits that fill the merge's turns to different degrees."""
    import numpy as np
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(n_q_heads=2, n_kv_heads=2, head_dim=hd, **SMALL)
    at = [(60, 30), (300, 10), (300, 290), (2100, 100), (2100, 2090), (1000, 500), (500, None)]      # context, position of the infinity
    wl = custom_workload("infinite", dims, prefill=[], decode=[c for c, _ in at], n_pairs=0, prompt=3, resp=(2, 9))
    for j, (_, p) in enumerate(at):
        if p is not None:
            wl.ctx_v[j][p, 1, 5] = np.inf
    it = DeviceIteration(wl)
    it.forward()
    torch_mod.cuda.synchronize()
    norms = it.head_norms.cpu().numpy()
    it.close()
    assert np.isfinite(norms[:, 0]).all(), norms
    assert [bool(np.isinf(n)) for n in norms[:, 1]] == [p is not None for _, p in at] and not np.isnan(norms).any(), norms
