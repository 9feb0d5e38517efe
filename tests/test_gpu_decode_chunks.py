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
