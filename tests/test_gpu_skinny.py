"""GPU parity of the weight-streaming products (batches of at most 64 inference rows and nothing else): every row
tile boundary of the kernel, with RMSNorm in its prologue and in a kernel of its own, both head sizes, grouped
queries, prefill and decode rows, cache append, and the logits behind it.  Bars as in test_gpu_parity: the
operands are single bf16 values and the sums fp32, as in every other inference row."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_loop import _check_logits
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,hd", [(8, 2, 64), (4, 4, 128)])
@pytest.mark.parametrize("rows", [3, 16, 17, 32, 33, 48, 63, 64, 65])
def test_few_rows(torch_mod, hq, hkv, hd, rows):
    # K of 320 and 704 leaves waves without a chunk, d_ff / 8 is odd; contexts on and off block edges
    dims = synth.ModelDims(320, hq, hkv, hd, 704, 4096, io_bf16=True)
    n_dec = 3 if rows < 16 else 7
    wl = custom_workload("skinny", dims, prefill=() if rows == n_dec else (rows - n_dec,),
                         decode=(0, 15, 700, 16, 33, 512, 1)[:n_dec], n_pairs=0, prompt=3, resp=(2, 9), seed=300 + rows)
    check_iteration(torch_mod, wl, f"rows {rows} Hq{hq} Hkv{hkv} hd{hd}")
    _check_logits(torch_mod, wl, f"rows {rows} Hq{hq} Hkv{hkv} hd{hd}")


@pytest.mark.parametrize("n_decode", [1, 2, 32])
def test_edge_decode_rows(torch_mod, n_decode):
    """The edge configuration's decode requests alone (two and one row group per block, 8-row groups)."""
    wl = synth.make_workload("edge", n_prefill=0, n_decode=n_decode, n_pairs=0)
    check_iteration(torch_mod, wl, f"edge decode {n_decode}")
