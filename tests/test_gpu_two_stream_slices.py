"""Weight gradients of one backward whose cut products are spread over both streams (attention or MLP narrower than the
model, many rows): the two-stream run against the single-stream run of the same inputs, which has to give the same bits.
Slices that overwrite each other's partial results change a gradient by whole addends."""
import numpy as np
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import custom_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,F", [(8, 4, 5632), (16, 16, 512)])
def test_slices_on_both_streams(torch_mod, hq, hkv, F):
    torch = torch_mod
    from paper_2510_03283_amd import binding as B
    from paper_2510_03283_amd.harness import DeviceIteration
    rows = 16384 if F > 2048 else 32768
    wl = custom_workload("two_streams", synth.ModelDims(2048, hq, hkv, 128, F, 512), prefill=(), decode=(), n_pairs=rows // 4096,
                         prompt=2000, resp=(48, 48), seed=900 + hq)
    got = []
    for options in ({}, {B.MACE_OPT_SINGLE_STREAM: 1}):
        it = DeviceIteration(wl, options=options)
        try:
            plans = it.step_with_plans()
            torch.cuda.synchronize()
            if not options:
                cut = {(r["name"], r["on_side_stream"]) for r in plans["bwd"] if r["layout"] == 2 and r["k_splits"] > 1}
                print("cut weight gradients:", sorted(cut), flush=True)
                assert {s for _, s in cut} == {0, 1}
            got.append({k: v.cpu().numpy() for k, v in {"dx": it.dx, **it.grads}.items()})
        finally:
            it.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
