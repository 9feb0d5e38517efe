"""RMSNorm reads a row in chunks of 1024 columns, all asked for together, and threads past the end read the last four columns again: rows that
end inside a chunk, at each number of chunks, alone and with the slices of the product in front of them, against the oracle."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu


# fp32 boundary up to 2112: at 4160 the inference rows' single bf16 operands put y at 1.06e-2 of its largest value (1.37e-2 at 8192, with
# chunks loaded one by one as well), where the bar is 1e-2
@pytest.mark.parametrize("d,bf16", [(d, True) for d in (64, 1024, 1088, 2112, 4160, 8192)] + [(d, False) for d in (64, 1024, 1088, 2112)])
def test_rows_that_end_inside_a_chunk(torch_mod, d, bf16):
    dims = synth.ModelDims(d, 4, 2, 64, 128, 256, io_bf16=bf16)
    wl = custom_workload("rows", dims, prefill=[70, 3], decode=[0, 17], n_pairs=1, prompt=5, resp=(2, 9), seed=d)
    check_iteration(torch_mod, wl, f"d {d} bf16 {bf16}")


@pytest.mark.parametrize("d", [1088, 4160])
def test_rows_behind_a_product_cut_along_k(torch_mod, d):
    # o and down of 200 rows reduce over 4096 and 5632: the slices are added by the norms and the sum behind them
    dims = synth.ModelDims(d, 64, 8, 64, 5632, 256, io_bf16=True)
    wl = custom_workload("cut", dims, prefill=[200], decode=[3], n_pairs=0, prompt=3, resp=(2, 9), seed=d)
    check_iteration(torch_mod, wl, f"cut, d {d}")
