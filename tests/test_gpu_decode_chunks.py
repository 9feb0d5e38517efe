"""Decode attention with short chunks: the launcher takes 128, 256 or 512 tokens a block by the work of the grid, and the merge of the
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
    """11 requests of up to 2000 tokens take chunks of 256 (8 kv heads) and 128 (16), 33 requests of 512 and 256."""
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL)
    for n in (11, 33):
        ctx = [(i * 197) % 2000 for i in range(n - 1)] + [2000]
        wl = custom_workload("rule", dims, prefill=[], decode=ctx, n_pairs=0, prompt=3, resp=(2, 9))
        check_iteration(torch_mod, wl, f"{n} requests Hq{hq} Hkv{hkv} hd{hd}")


@pytest.mark.parametrize("hq,hkv,hd,ctx", [
    (8, 2, 64, EDGES + [500, 2046, 4400]),      # 128 against 512
    (4, 4, 128, EDGES + [2048, 4400]),
    (8, 1, 64, [1300] * 100),                   # 256
    (16, 16, 64, [257] * 320),                  # 10240 blocks of 256: the last batch whose chunk is priced (128), and the first of the others (512)
    (16, 16, 64, [257] * 321),
], ids=["edges64", "edges128", "256", "priced", "stream"])
def test_against_pinned_chunks(torch_mod, hq, hkv, hd, ctx):
    """Norms of the heads' outputs: a lane adds at most 4400 / 8 products, then the states of lanes, waves and splits are merged in about 20 steps, so either
    evaluation is within 600 * 2^-24 = 3.5e-5 of the sum.  y: the merged outputs round to bf16 either way, which the oracle's bar for y covers."""
    import numpy as np
    from paper_2510_03283_amd import binding
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL)
    synth.CONFIGS["pinned"] = synth.ConfigSpec("pinned", 77, dims, [], None, list(ctx), None, 0, 3, None, (2, 9), ref_mode="len", block_size=16)
    try:
        wl = synth.make_workload("pinned", with_cache=False)
    finally:
        del synth.CONFIGS["pinned"]
    got = []
    for options in (None, {binding.MACE_OPT_DECODE_CHUNK: 512}):
        it = DeviceIteration(wl, device_cache_seed=5, options=options)
        it.forward()
        torch_mod.cuda.synchronize()
        got.append((it.y.cpu().numpy(), it.head_norms.cpu().numpy()))
        it.close()
    (y, n), (y512, n512) = got
    assert np.isfinite(y).all() and n512.min() > 0
    assert np.abs(n / n512 - 1).max() <= 7e-5
    assert np.abs(y - y512).max() <= 1e-2 * np.abs(y512).max()


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


@pytest.mark.parametrize("hq,hkv,hd,bf16,block", [(8, 2, 64, True, 16), (4, 4, 128, True, 16), (4, 4, 128, True, 2), (4, 2, 64, False, 16)])
def test_unused_blocks_of_the_pool_may_hold_anything(torch_mod, hq, hkv, hd, bf16, block):
    """A pool is not cleared before its blocks are handed out: with NaN in every block that no request owns, and behind the last token of those that are
    owned, the pool's first block among the unused ones, y and the head norms are what they are with zeros there."""
    import numpy as np
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, io_bf16=bf16, **SMALL)
    for seed in range(77, 177):
        wl = custom_workload("pool", dims, prefill=[], decode=EDGES + [700, 1111], n_pairs=0, prompt=3, resp=(2, 9), block_size=block, seed=seed)
        b = wl.batch
        used = np.zeros((b.num_blocks, block), bool)
        for j, n in enumerate(b.decode_ctx):
            for t in range(int(n) + 1):
                used[b.decode_block_tables[j][t // block], t % block] = True
        if not used[0].any():
            break
    assert not used[0].any()
    free = torch_mod.from_numpy(~used).cuda()
    got = []
    for fill in (0.0, float("nan")):
        it = DeviceIteration(wl)
        for c in (it.cache_k, it.cache_v):
            c.masked_fill_(free[:, None, :, None], fill)
        it.forward()
        torch_mod.cuda.synchronize()
        got.append((it.y.cpu().numpy(), it.head_norms.cpu().numpy()))
        it.close()
    for a, z in zip(got[1], got[0]):
        assert np.isfinite(z).all() and np.array_equal(a, z)
