"""GPU parity of the causal attention at the edges of its tiles: sequence lengths on either side of a wave's 32 queries,
of the 64-row key tiles and of the 128- and 256-row blocks, one-row sequences, grouped queries, both head sizes, both
storage types (single and two-term operands), forward and backward.  Bars as in test_gpu_parity.  (The shortest sequence
has two prompt rows: behind one, the only row with a gradient sees one key, and the query gradient is zero.)"""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import SMALL, check_iteration, custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,hd,bf", [(8, 2, 64, True), (2, 2, 128, True), (4, 1, 128, False)])
@pytest.mark.parametrize("prompt,resp", [(2, (1, 1)), (31, (1, 2)), (63, (1, 2)), (127, (1, 2)), (256, (1, 1))])
def test_tile_edges(torch_mod, hq, hkv, hd, bf, prompt, resp):
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, io_bf16=bf, **SMALL)
    wl = custom_workload("tiles", dims, prefill=[1, 31, 32, 33, 64, 65, 128, 129, 257], decode=[3], n_pairs=2, prompt=prompt, resp=resp,
                         seed=900 + prompt)
    check_iteration(torch_mod, wl, f"tiles Hq{hq} Hkv{hkv} hd{hd} bf{bf} prompt{prompt} resp{resp}")


@pytest.mark.parametrize("hq,hkv,hd,bf", [(8, 2, 64, True), (2, 2, 128, True), (4, 1, 128, False)])
@pytest.mark.parametrize("prefill,decode,n_pairs", [((1, 17, 33, 65, 5, 129, 40), (3, 40), 3), ((1, 17, 9, 5, 2), (3, 40), 0)])
def test_sequences_do_not_reach_into_each_other(torch_mod, hq, hkv, hd, bf, prefill, decode, n_pairs):
    """A tile that hangs over the end of its sequence reads zeros there, not its neighbour's rows: with NaN in the input of
    every other sequence (preference pair) the rest come out as without, bit for bit - outputs, log-probabilities, row gradients."""
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, io_bf16=bf, **SMALL)
    wl = custom_workload("leak", dims, prefill=prefill, decode=decode, n_pairs=n_pairs, prompt=13, resp=(2, 90), seed=990)
    it = DeviceIteration(wl)
    try:
        seg = wl.batch.seg_offsets
        inf = len(prefill) + len(decode)
        bad = [i for i in range(inf) if i % 2] + [inf + s for s in range(2 * n_pairs) if (s // 2) % 2 == 0]
        keep = torch_mod.ones(it.T, dtype=torch_mod.bool, device="cuda")
        for s in bad:
            keep[int(seg[s]):int(seg[s + 1])] = False
        cache = it.cache_k.clone(), it.cache_v.clone()
        it.step()
        want = [t.clone() for t in (it.y, it.dx, it.logp)]
        it.cache_k.copy_(cache[0]); it.cache_v.copy_(cache[1])
        it.x[~keep] = float("nan")
        it.step()
        assert torch_mod.isnan(it.y[~keep]).all()
        assert torch_mod.equal(it.y[keep], want[0][keep])
        if n_pairs:
            seqs = torch_mod.tensor([(s // 2) % 2 == 1 for s in range(2 * n_pairs)], device="cuda")
            assert torch_mod.isnan(it.logp[~seqs]).all() and torch_mod.equal(it.logp[seqs], want[2][seqs])
            assert torch_mod.equal(it.dx[keep[it.Ti:]], want[1][keep[it.Ti:]])
    finally:
        it.close()
