"""GPU parity of the weight-streaming products where blocks share the row groups evenly (a reduction of at least 1024): row
groups per block from one to eight, blocks that own one group less than the others, and batches of 65 - 128 rows with every
number of 16-row tiles, the last of them partly or not at all filled.  Bars as in test_gpu_skinny."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_loop import _check_logits
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu

# d_ff, vocabulary -> groups of 16 weight rows of gate / up and of the head
SHAPES = {(2752, 10304): (344, 644), (5504, 20800): (688, 1300), (704, 32064): (88, 2004)}


@pytest.mark.parametrize("F,V", SHAPES, ids=lambda v: str(v))
@pytest.mark.parametrize("rows", [5, 17, 48, 65, 80, 96, 97, 128, 129])
def test_even_blocks(torch_mod, F, V, rows):
    assert SHAPES[F, V] == (F // 8, V // 16)
    dims = synth.ModelDims(1024, 32, 8, 64, F, V, io_bf16=True)
    ctx = (0, 15, 300, 16, 33, 128, 1)
    wl = custom_workload("even", dims, prefill=(), decode=[ctx[i % 7] + i // 7 for i in range(rows)], n_pairs=0, prompt=3, resp=(2, 9), seed=700 + rows)
    check_iteration(torch_mod, wl, f"rows {rows} F{F} V{V}")
    _check_logits(torch_mod, wl, f"rows {rows} F{F} V{V}")
