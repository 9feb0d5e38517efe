"""GPU parity of products whose reduction is cut into slices (partial results added by the kernel behind the product):
the launch plan has to show slices for the named products, and every output and gradient is compared with the oracle at
the bars of test_gpu_parity.  Sizes leave ragged tiles in both directions, reductions that do not divide evenly, row
groups cut into different numbers of slices, both storage types, both head sizes, and one row class at a time."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu

CASES = {
    # both row classes, 128-wide heads: the QKV slices replace the fused rotary form
    "mixed": (synth.ModelDims(2048, 16, 2, 128, 1408, 2048), dict(prefill=[130, 75], decode=[40, 300], n_pairs=1, prompt=100, resp=(60, 90)),
              {"qkv gemm", "o gemm", "down gemm", "gate/up gemm", "dhm gemm", "db gemm", "da gemm"}),
    # a wide model with a narrow attention: the bf16 gradient of the attention output comes from slices
    "wide": (synth.ModelDims(4096, 4, 2, 128, 512, 1024), dict(prefill=[30], decode=[20], n_pairs=1, prompt=60, resp=(40, 70)), {"dattn gemm", "dhm gemm", "gate/up gemm", "qkv gemm"}),
    # fine-tune rows only, 64-wide heads, a reduction of 11 x 64
    "ft": (synth.ModelDims(704, 4, 4, 64, 1408, 2048), dict(prefill=[], decode=[], n_pairs=2, prompt=60, resp=(50, 150)), {"qkv gemm", "down gemm", "db gemm"}),
    # inference rows only, more than the weight-streaming kernel takes
    "inference": (synth.ModelDims(1024, 8, 4, 64, 2816, 4096), dict(prefill=[250, 37], decode=[9, 700], n_pairs=0, prompt=3, resp=(2, 9)),
                  {"qkv gemm", "down gemm"}),
    # fp32 storage: three passes
    "fp32": (synth.ModelDims(512, 4, 2, 128, 1408, 2048, io_bf16=False), dict(prefill=[70], decode=[33], n_pairs=1, prompt=30, resp=(20, 60)), {"qkv gemm", "o gemm", "down gemm", "db gemm", "da gemm"}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_sliced_products(torch_mod, name):
    from paper_2510_03283_amd.harness import DeviceIteration
    dims, batch, expect = CASES[name]
    wl = custom_workload(f"slices_{name}", dims, seed=4100, **batch)
    it = DeviceIteration(wl)
    try:
        plans = it.step_with_plans()
        torch_mod.cuda.synchronize()
        sliced = {r["name"]: r["k_splits"] for p in plans.values() for r in p if r["k_splits"] > 1}
        print(f"[{name}] slices: {sliced}", flush=True)
        assert expect <= set(sliced), expect - set(sliced)
    finally:
        it.close()
    check_iteration(torch_mod, wl, f"slices {name}")
