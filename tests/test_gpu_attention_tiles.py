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
