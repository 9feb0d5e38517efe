"""GPU parity of the pair losses around the number of waves that share the pairs (16): one pair, a full round, one more,
and several rounds, with responses of unequal length.  Bars as in test_gpu_parity."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pairs", [1, 16, 17, 35])
def test_pairs_over_waves(torch_mod, n_pairs):
    dims = synth.ModelDims(256, 4, 2, 64, 704, 2048, io_bf16=True)
    wl = custom_workload("pairs", dims, prefill=(), decode=(5,), n_pairs=n_pairs, prompt=3, resp=(2, 70), seed=40 + n_pairs)
    check_iteration(torch_mod, wl, f"pairs {n_pairs}")
