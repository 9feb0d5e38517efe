"""Rotary embedding, operand split and cache append in the epilogue of the QKV product (four-wave GEMM kernel): heads of 64
(two to a wave's 128 columns) and of 128, inference rows alone and beside fine-tune rows (the shared angle table in either
buffer), row counts that leave the last row tile partly filled, and caches of different page sizes.  Outputs and cache against
the oracle at the bars of test_gpu_parity; then against the kernel of its own, which a cache that is not 16-byte aligned, or an
fp32 one, still takes."""
import pytest

from paper_2510_03283_amd import synth
from test_gpu_parity import check_iteration, custom_workload

pytestmark = pytest.mark.gpu

CASES = {
    "hd64_inference": (synth.ModelDims(2048, 32, 8, 64, 1024, 512, io_bf16=True), (1501, 1030), (40, 7, 0), 0, 16),
    "hd64_mixed_more_inference": (synth.ModelDims(2048, 32, 8, 64, 1024, 512, io_bf16=True), (1999,), (5,), 2, 256),
    "hd64_mixed_more_fine_tune": (synth.ModelDims(2048, 32, 4, 64, 1024, 512, io_bf16=True), (333,), (17,), 6, 1),
    "hd128_inference": (synth.ModelDims(2048, 16, 2, 128, 1024, 512, io_bf16=True), (2100, 37), (), 0, 32),
    "hd128_mixed": (synth.ModelDims(2048, 16, 4, 128, 1024, 512, io_bf16=True), (1400,), (100, 3), 3, 16),
}


def workload(name, with_decode=True):
    dims, prefill, decode, pairs, block = CASES[name]
    decode = decode if with_decode else ()
    return custom_workload("rope_epi", dims, prefill, decode, pairs, prompt=200, resp=(130, 200), block_size=block, seed=31)


@pytest.mark.parametrize("name", CASES)
def test_epilogue_against_oracle(torch_mod, name):
    from paper_2510_03283_amd.harness import DeviceIteration
    wl = workload(name)
    it = DeviceIteration(wl)
    try:
        names = [r["name"] for r in it.step_with_plans()["fwd"]]
        torch_mod.cuda.synchronize()
        assert "qkv gemm + rope" in names, names
    finally:
        it.close()
    check_iteration(torch_mod, wl, name, check_grads=False)


@pytest.mark.parametrize("name", CASES)
def test_epilogue_against_own_kernel(torch_mod, name):
    """The same prefill rows into an aligned cache and into one that starts 8 bytes later; a slot of -1 is written by neither.  Both sides
    round the same fp32 rotation (up to its fused multiply-add and the order of the product's sum, together below 2^-15 of the largest
    value) to bf16, whose steps are at most 2^-7 of a value: one step, where the two lie on either side of a tie."""
    from paper_2510_03283_amd import binding as B
    from paper_2510_03283_amd.harness import DeviceIteration
    torch = torch_mod
    wl = workload(name, with_decode=False)
    it = DeviceIteration(wl)
    try:
        n = it.cache_k.numel()
        skipped = int(it.slot_mapping_host[1])
        it.slot_dev[1] = -1
        got = []
        for shift in (0, 4):
            flat = [torch.full((n + 8,), 7.0, dtype=it.cache_k.dtype, device=it.dev) for _ in range(2)]
            for f, src in zip(flat, (it.cache_k, it.cache_v)):
                f[shift:shift + n] = src.flatten()
            views = [f[shift:shift + n].view(it.cache_k.shape) for f in flat]
            it.cache = B.kv_cache_struct(views[0], views[1], wl.batch.num_blocks, wl.batch.block_size)
            it.forward()
            torch.cuda.synchronize()
            assert all((f[:shift] == 7).all() and (f[shift + n:] == 7).all() for f in flat)
            got.append([v.float().clone() for v in views])
        bs = wl.batch.block_size
        for a, b, before in zip(got[0], got[1], (it.cache_k, it.cache_v)):
            assert ((a - b).abs() <= 2.0 ** -7 * b.abs() + 2.0 ** -15 * b.abs().max()).all(), (a - b).abs().max()
            assert torch.equal(a[skipped // bs, :, skipped % bs], before.float()[skipped // bs, :, skipped % bs])
            assert (a != before.float()).any()
    finally:
        it.close()


def test_fp32_cache_keeps_its_kernel(torch_mod):
    """An fp32 layer with more inference than fine-tune rows: only the latter are rotated in the epilogue."""
    from paper_2510_03283_amd.harness import DeviceIteration
    dims = synth.ModelDims(1024, 16, 4, 64, 1024, 512, io_bf16=False)
    wl = custom_workload("rope_fp32", dims, (1501, 900), (9,), 3, prompt=200, resp=(130, 200), block_size=16, seed=32)
    it = DeviceIteration(wl)
    try:
        names = [r["name"] for r in it.step_with_plans()["fwd"]]
        torch_mod.cuda.synchronize()
        print(it.Ti, it.Tf, names, flush=True)
        assert it.Ti > it.Tf and "qkv gemm + rope" in names, names
    finally:
        it.close()
    check_iteration(torch_mod, wl, "fp32", check_grads=False)
