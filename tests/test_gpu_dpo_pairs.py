"""GPU parity of the pair losses around the number of waves (16): one wave to a pair with fewer pairs than waves, a full
round, one more, and several rounds, and two to sixteen waves sharing a pair of long responses; responses of unequal
length.  Bars as in test_gpu_parity."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pairs", [1, 16, 17, 35])
def test_pairs_over_waves(torch_mod, n_pairs):
    dims = synth.ModelDims(256, 4, 2, 64, 704, 2048, io_bf16=True)
    wl = custom_workload("pairs", dims, prefill=(), decode=(5,), n_pairs=n_pairs, prompt=3, resp=(2, 70), seed=40 + n_pairs)
    check_iteration(torch_mod, wl, f"pairs {n_pairs}")


@pytest.mark.parametrize("n_pairs,rows", [(1, 4200), (1, 600), (2, 2100), (3, 1100), (5, 520), (8, 700), (9, 700)])
def test_waves_that_share_a_pair(torch_mod, n_pairs, rows):
    # 16, 2, 8, 4, 2, 2 waves to a pair and one
    dims = synth.ModelDims(256, 4, 2, 64, 704, 2048, io_bf16=True)
    wl = custom_workload("long_pairs", dims, prefill=(), decode=(), n_pairs=n_pairs, prompt=3, resp=(rows, rows + 70), seed=60 + n_pairs)
    check_iteration(torch_mod, wl, f"{n_pairs} pairs of {rows}", check_grads=False)
