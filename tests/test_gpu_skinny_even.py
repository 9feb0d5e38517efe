"""GPU parity of the weight-streaming products where blocks share the row groups evenly (a reduction of at least 1024): every epilogue (QKV,
gate / up, fp32) with several row groups per block, blocks that own one group less than the others, and batches of 5 - 128 rows with every
number of 16-row tiles, the last of them partly or not at all filled.  Bars as in test_gpu_skinny."""
import dataclasses
import functools

import pytest

from helpers import max_abs_norm_err, run_oracle
from oracle import mace_oracle as O
from paper_2510_03283_amd import synth
from paper_2510_03283_amd import binding as B
from paper_2510_03283_amd.harness import DeviceIteration
from test_gpu_loop import _check_logits
from test_gpu_parity import TOL_OUT, check_iteration, custom_workload

pytestmark = pytest.mark.gpu

# d_ff, vocabulary -> groups of 16 weight rows of gate / up and of the head
SHAPES = {(2752, 10304): (344, 644), (5504, 20800): (688, 1300), (704, 32064): (88, 2004)}


@pytest.mark.parametrize("F,V", SHAPES, ids=lambda v: str(v))
@pytest.mark.parametrize("rows", [5, 17, 48, 49, 64, 65, 80, 96, 97, 128, 129])
def test_even_blocks(torch_mod, F, V, rows):
    assert SHAPES[F, V] == (F // 8, V // 16)
    dims = synth.ModelDims(1024, 32, 8, 64, F, V, io_bf16=True)
    ctx = (0, 15, 300, 16, 33, 128, 1)
    wl = custom_workload("even", dims, prefill=(), decode=[ctx[i % 7] + i // 7 for i in range(rows)], n_pairs=0, prompt=3, resp=(2, 9), seed=700 + rows)
    check_iteration(torch_mod, wl, f"rows {rows} F{F} V{V}")
    _check_logits(torch_mod, wl, f"rows {rows} F{F} V{V}")


# model -> rows -> the most groups a block owns in QKV, gate / up and the head (test_launch_order holds the launches to it).  576, 1376 and 644 groups; 1200, 880 and 800; 800, 880 and 800; 2048,
# 1792 and 192: blocks of unequal shares but for the last model.
FORMS = {
    (1024, 72, 36, 64, 11008, 10304): {5: (3, 2, 3), 17: (3, 6, 3), 49: (3, 6, 3), 96: (3, 3, 3)},
    (1024, 50, 50, 128, 7040, 12800): {16: (2, 4, 4), 40: (6, 4, 4), 81: (3, 4, 4)},
    (1024, 100, 50, 64, 7040, 12800): {16: (4, 4, 4), 64: (4, 4, 4), 128: (4, 4, 4)},
    (1024, 256, 128, 64, 14336, 3072): {47: (8, 8, 1), 70: (4, 4, 1)},
}


@functools.lru_cache(maxsize=1)
def form_spec(dims):
    spec = synth.ConfigSpec("even_forms", 900, synth.ModelDims(*dims, io_bf16=True), [], None, [], None, 0, 3, None, (2, 9), ref_mode="len")
    return spec, synth.make_weights(spec)


@pytest.mark.parametrize("dims,rows", [(d, r) for d, by_rows in FORMS.items() for r in by_rows], ids=lambda v: "_".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_groups_of_every_epilogue(torch_mod, monkeypatch, dims, rows):
    """QKV with the cache append, gate / up and the fp32 products of the layer, and the head, with every number of groups a block."""
    spec, weights = form_spec(dims)
    ctx = (0, 15, 300, 16, 33, 128, 1)
    monkeypatch.setitem(synth.CONFIGS, "even_forms", dataclasses.replace(spec, decode_ctx=[ctx[i % 7] + i // 7 for i in range(rows)]))
    wl = synth.make_workload("even_forms", weights=weights)
    ref = run_oracle(wl, backward=False)
    it = DeviceIteration(wl)
    try:
        it.forward()
        logits = torch_mod.empty((rows, dims[5]), dtype=torch_mod.float32, device="cuda")
        B.mace_next_token_logits(it.h, it.y, None, rows, it.gf, it.E, logits, None, it.ws)
        torch_mod.cuda.synchronize()
        want, _ = O.next_token_logits(wl.dims, wl.weights, ref["y"])
        got = {"y": it.y, "head_norms": it.head_norms, "cache_k": it.cache_k, "cache_v": it.cache_v, "logits": logits}
        for k, v in got.items():
            e = max_abs_norm_err(v.float().cpu().numpy(), want if k == "logits" else ref[k])
            print(f"rows {rows} {dims} {k}: {e:.2e}", flush=True)
            assert e <= TOL_OUT, (k, e)      # (a NaN is no less than the bar)
    finally:
        it.close()
