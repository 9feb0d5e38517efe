"""GPU parity of the attention kernels where a grid is small: the dK/dV kernel with two teams of waves a block (the number of query
tiles odd and even, one tile, keys that a team's tiles all precede) on both sides of its rule, and sequences turned by the row tile
(more and fewer sequences than row tiles, ragged)."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import SMALL, check_iteration, custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,hd", [(8, 2, 64), (4, 4, 128), (8, 1, 128)])
@pytest.mark.parametrize("pairs,prompt,resp", [(1, 3, (2, 60)), (1, 60, (5, 70)), (2, 130, (1, 330)), (5, 200, (1, 90))])
def test_two_teams(torch_mod, hq, hkv, hd, pairs, prompt, resp):
    dims = synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL)
    wl = custom_workload("teams", dims, prefill=[5, 300, 129], decode=[7], n_pairs=pairs, prompt=prompt, resp=resp)
    check_iteration(torch_mod, wl, f"Hq{hq} Hkv{hkv} hd{hd} pairs {pairs} prompt {prompt} resp {resp}")


def test_one_team(torch_mod):
    """32 kv heads and 20 sequences: past the rule."""
    dims = synth.ModelDims(n_q_heads=32, n_kv_heads=32, head_dim=64, **SMALL)
    wl = custom_workload("one_team", dims, prefill=[40], decode=[7], n_pairs=10, prompt=20, resp=(5, 120))
    check_iteration(torch_mod, wl, "one team")


# (query heads, kv heads, head width, pairs, prompt, responses, prompt stored once) -> teams of a dK/dV block (test_launch_order holds them to it).  With the
# prompt stored once, key tiles that later rows do not see: whole and in part, in both forms of the kernel.
FORMS = {
    (4, 4, 128, 2, 330, (2, 60), False): 2, (4, 4, 128, 2, 470, (2, 60), False): 2, (8, 2, 128, 2, 90, (5, 70), False): 2, (8, 2, 64, 3, 129, (1, 3), True): 2, (4, 2, 128, 3, 200, (120, 300), True): 2,
    (4, 4, 128, 3, 129, (60, 90), True): 2, (32, 32, 64, 8, 200, (60, 120), True): 1, (8, 8, 64, 12, 20, (5, 44), False): 1, (16, 16, 128, 6, 300, (100, 260), True): 1,
}


def form_workload(hq, hkv, hd, pairs, prompt, resp, shared):
    wl = custom_workload("teams", synth.ModelDims(n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, **SMALL), prefill=[40], decode=[7], n_pairs=pairs, prompt=prompt, resp=resp)
    return synth.to_shared_prompt(wl) if shared else wl


@pytest.mark.parametrize("form", FORMS, ids=str)
def test_forms(torch_mod, form):
    check_iteration(torch_mod, form_workload(*form), f"{FORMS[form]} teams {form}")
