"""Kernel-level parity of the four-wave contraction on tiles of 224 and 192 rows, which the launcher takes for row counts and rounds of
tiles that 256 rows fill badly: the last tile of one row, of some and of all rows, odd and even numbers of k tiles and the padded
loops, one and two passes, every output form.  The launch plan confirms the height.  Definition, buffers and bars as in test_gpu_gemm_kernel."""
import numpy as np
import pytest

from test_gpu_gemm_kernel import SENT, bf16_of, check_out, f64, handle, operands, out_buffer  # noqa: F401

pytestmark = pytest.mark.gpu

# rows -> tile height, for 11000 columns (43 tiles): one round of tiles of 224 rows, full and not; tiles of 192 rows, the last of one, of 107 and of all rows
ROWS = {1120: 224, 1009: 224, 577: 192, 299: 192, 576: 192}


def plan_tile(binding, handle):
    (r,) = binding.mace_launch_plan(handle)
    return tuple(r["tile"])


@pytest.mark.parametrize("M", sorted(ROWS))
@pytest.mark.parametrize("lb,K", [(0, 832), (0, 1600), (1, 896)])
def test_products(torch_mod, handle, M, lb, K):
    torch = torch_mod
    from paper_2510_03283_amd import binding
    N = 11000
    rng = np.random.default_rng(K + 7 * M + lb)
    a, b, A, B = operands(torch, rng, 0, lb, M, N, K)
    ref = A @ B.T
    for dtype, tol in ((torch.float32, 1e-5), (torch.bfloat16, 4e-3)):
        c = out_buffer(torch, M + 5, N + 24, dtype)
        binding.mace_gemm_bf16(handle, 0, lb, M, N, K, a, b, c, ldc=N + 24)
        assert plan_tile(binding, handle) == (ROWS[M], 256)
        torch.cuda.synchronize()
        check_out(c, ref, M, N, tol, f"{lb} {M}x{N}x{K} {dtype}")
    for dtype in (torch.float32, torch.bfloat16):
        r = bf16_of(torch, rng.uniform(-20, 20, (M, N))).to(dtype)
        c = out_buffer(torch, M + 5, N + 24, torch.float32)
        binding.mace_gemm_bf16(handle, 0, lb, M, N, K, a, b, c, resid=r, ldc=N + 24, ldr=N)
        torch.cuda.synchronize()
        check_out(c, ref + f64(r), M, N, 1e-5, f"{lb} {M}x{N}x{K} residual {dtype}")


@pytest.mark.parametrize("M", sorted(ROWS))
@pytest.mark.parametrize("K", [448, 832, 2048])
def test_two_terms_and_swiglu(torch_mod, handle, M, K):
    torch = torch_mod
    from paper_2510_03283_amd import binding
    N = 11000
    rng = np.random.default_rng(K + 5 * M)
    a, b, A, B = operands(torch, rng, 0, 0, M, N, K)
    lo = bf16_of(torch, rng.uniform(-1, 1, (M, K)) * 2.0 ** -9)
    A2 = A + f64(lo)
    c = out_buffer(torch, M + 5, N + 24, torch.float32)
    binding.mace_gemm_bf16(handle, 0, 0, M, N, K, a, b, c, a_lo=lo, ldc=N + 24)
    assert plan_tile(binding, handle) == (ROWS[M], 256)
    torch.cuda.synchronize()
    check_out(c, A2 @ B.T, M, N, 1e-5, f"two terms {M}x{N}x{K}")
    # G and U of the same activations, kept beside silu(G) U in two terms
    F = 5504
    s = K ** -0.5
    bg, bu = (b[:F].float() * s).to(torch.bfloat16), (b[F - 8:2 * F - 8].float() * s).to(torch.bfloat16)
    g, u = A2 @ f64(bg).T, A2 @ f64(bu).T
    h = g / (1.0 + np.exp(-g)) * u
    hi, h_lo, gu = (out_buffer(torch, M + 5, w, torch.bfloat16) for w in (F + 8, F + 8, 2 * F))
    binding.mace_gemm_bf16(handle, 0, 0, M, F, K, a, bg, hi, a_lo=lo, b_up=bu, c_lo=h_lo, c_gu=gu, ldc=F + 8, swiglu=True)
    assert plan_tile(binding, handle) == (ROWS[M], 256)
    torch.cuda.synchronize()
    check_out(hi, h, M, F, 4e-3, f"swiglu {M}x{F}x{K}")
    two = f64(hi)[:M, :F] + f64(h_lo)[:M, :F]
    assert np.abs(two - h).max() / np.abs(h).max() <= 5e-5
    check_out(gu, np.concatenate([g, u], axis=1), M, 2 * F, 4e-3, "G | U")
    assert np.all(f64(h_lo)[M:] == SENT)


@pytest.mark.parametrize("rows,height", [(298, 192), (576, 192), (578, 192), (1010, 224), (1120, 224)])
def test_swiglu_backward(torch_mod, rows, height):
    """dG | dU in the epilogue of dHm, seen through dWg and dWu of a layer whose upstream gradient is zero but in one row of every sixteen, and then but in the
    last: a block of rows that goes wrong is a sixth of the result and more.  Bar: dy, dG and b are rounded to bf16 once, G and U (two factors of dG) as the
    forward keeps them, and its operands once more, 2^-9 each: 1.2e-2."""
    torch = torch_mod
    from helpers import max_abs_norm_err, run_oracle
    from oracle import mace_oracle as O
    from paper_2510_03283_amd import binding, synth
    from paper_2510_03283_amd.harness import DeviceIteration
    from test_gpu_parity import custom_workload
    n = rows // 2 - 40
    wl = custom_workload("swiglu_rows", synth.ModelDims(832, 4, 4, 64, 11008, 1024, io_bf16=True), prefill=(), decode=(), n_pairs=1, prompt=40, resp=(n, n))
    ref = run_oracle(wl, backward=False)
    it = DeviceIteration(wl)
    try:
        assert it.Tf == rows
        it.forward()
        for picked in ([16 * i + 5 * i % 16 for i in range(rows // 16)], [rows - 1]):
            dy = np.zeros((rows, 832), np.float32)
            dy[picked] = np.random.default_rng(rows).uniform(-1, 1, (len(picked), 832))
            it.backward(torch.from_numpy(dy).cuda())
            (r,) = [r for r in binding.mace_launch_plan(it.h) if r["name"] == "dhm gemm + swiglu bwd"]
            assert tuple(r["tile"]) == (height, 256)
            torch.cuda.synchronize()
            _, want = O.layer_backward(wl.dims, wl.weights, ref["saved"], [dy[:rows // 2], dy[rows // 2:]])
            for k in ("wg", "wu"):
                e = max_abs_norm_err(it.grads[k].cpu().numpy(), want[k])
                print(f"{rows} rows, {len(picked)} of them picked, d{k}: {e:.2e}", flush=True)
                assert e <= 1.2e-2, (rows, len(picked), k, e)
    finally:
        it.close()
