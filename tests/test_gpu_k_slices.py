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


@pytest.mark.parametrize("single_stream", [0, 1])
def test_sliced_weight_gradients_are_accumulated(torch_mod, single_stream):
    """All four weight-gradient products of a layer in slices, on the side stream and on the caller's: the sum of the slices
    is added to what the gradient held (in place), and alone it is the oracle's gradient."""
    from helpers import rel_fro_err, run_oracle
    from paper_2510_03283_amd import binding as B
    from paper_2510_03283_amd.harness import DeviceIteration
    torch = torch_mod
    wl = custom_workload("slices_acc", synth.ModelDims(512, 4, 2, 128, 1408, 2048), prefill=[], decode=[], n_pairs=2, prompt=400, resp=(350, 450), seed=4200)
    ref = run_oracle(wl)
    it = DeviceIteration(wl, options={B.MACE_OPT_SINGLE_STREAM: 1} if single_stream else None)
    try:
        plans = it.step_with_plans()
        torch.cuda.synchronize()
        once = {k: v.clone() for k, v in it.grads.items()}
        for k, v in once.items():
            e = rel_fro_err(v.cpu().numpy(), ref["grads"][k])
            print(f"d{k}: {e:.2e}", flush=True)
            assert e <= 2e-2, (k, e)
        gen = torch.Generator(device="cuda").manual_seed(7)
        before = {k: torch.randn(v.shape, generator=gen, device="cuda") * v.std() for k, v in once.items()}
        for k, v in it.grads.items():
            v.copy_(before[k])
        B.mace_hybrid_layer_bwd(it.h, it.w_struct, it.batch, it.x, it.dh, it.saved, it.dx, it.g_struct, 1, it.ws)
        for p in (plans["bwd"], B.mace_launch_plan(it.h)):
            cut = {(r["name"], r["on_side_stream"]) for r in p if r["layout"] == 2 and r["k_splits"] > 1}
            assert cut == {(n, 1 - single_stream) for n in ("dWd gemm", "dWg/dWu gemm", "dWo gemm", "dWqkv gemm")}, cut
        torch.cuda.synchronize()
        for k, v in it.grads.items():      # one fp32 addition more than the gradient alone
            assert torch.allclose(v, before[k] + once[k], rtol=3e-7, atol=3e-7 * float(once[k].std())), k
    finally:
        it.close()


def test_sliced_adapter_products(torch_mod):
    """Adapter products in slices, read by the scaling split and the gradient extraction; the vocabulary reduction of the
    head in slices beside them."""
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(2048, 4, 4, 128, 512, 4096)
    wl = custom_workload("slices_lora", dims, prefill=[130], decode=[5, 300], n_pairs=2, prompt=170, resp=(90, 130), seed=4300)
    spec = synth.ConfigSpec("slices_lora", 4300, dims, None, None, None, None, 2, 170, None, (90, 130))
    lora = synth.make_lora(spec, rank=16, scale=2.0)
    it = DeviceIteration(wl, lora=lora)
    try:
        plans = it.step_with_plans()
        torch_mod.cuda.synchronize()
        sliced = {r["name"]: r["k_splits"] for p in plans.values() for r in p if r["k_splits"] > 1}
        print(f"slices: {sliced}", flush=True)
        expect = {f"lora {n} gemm" for n in ("t_qkv", "t_o", "dt_o", "dt_qkv", "dB_o", "dA_o", "dB_qkv", "dA_qkv")} | {"dn gemm"}
        assert expect <= set(sliced), expect - set(sliced)
    finally:
        it.close()
    check_iteration(torch_mod, wl, "sliced adapters", lora=lora)
