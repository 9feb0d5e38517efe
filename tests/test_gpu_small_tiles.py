"""Kernel-level parity of the dense contraction on the small tiles (64x64, 64x128) that the launcher takes for few rows and short
reductions: one block and one row or column past it, reductions of one k tile and with a remainder (token-contracting form), every
layout, output type and residual, and the SwiGLU form; the launch plan confirms the tile.  Definition, buffers and bars as in
test_gpu_gemm_kernel."""
import numpy as np
import pytest

from test_gpu_gemm_kernel import check_out, f64, handle, operands, out_buffer  # noqa: F401

pytestmark = pytest.mark.gpu


def check_tile(binding, handle, tiles):
    (r,) = binding.mace_launch_plan(handle)
    assert tuple(r["tile"]) in tiles, r["tile"]


@pytest.mark.parametrize("la,lb,M,N,K", [(0, 0, 1, 2, 64), (0, 0, 64, 64, 128), (0, 0, 65, 66, 64), (0, 0, 234, 768, 256), (0, 0, 400, 840, 704),
                                         (0, 1, 7, 8, 64), (0, 1, 64, 64, 64), (0, 1, 65, 72, 128), (0, 1, 128, 704, 256), (0, 1, 300, 256, 768),
                                         (1, 1, 8, 8, 1), (1, 1, 64, 64, 64), (1, 1, 72, 136, 65), (1, 1, 704, 256, 128), (1, 1, 256, 768, 100)])
def test_products(torch_mod, handle, la, lb, M, N, K):
    torch = torch_mod
    from paper_2510_03283_amd import binding
    rng = np.random.default_rng(K + 7 * M + la + 2 * lb)
    a, b, A, B = operands(torch, rng, la, lb, M, N, K)
    ref = A @ B.T
    for dtype, tol in ((torch.float32, 1e-5), (torch.bfloat16, 4e-3)):
        c = out_buffer(torch, M + 5, N + 24, dtype)
        binding.mace_gemm_bf16(handle, la, lb, M, N, K, a, b, c, ldc=N + 24)
        check_tile(binding, handle, [(64, 64), (64, 128)])
        torch.cuda.synchronize()
        check_out(c, ref, M, N, tol, f"{la}{lb} {M}x{N}x{K} {dtype}")
    for dtype in (torch.float32, torch.bfloat16):
        r = torch.from_numpy(rng.uniform(-20, 20, (M, N + 2)).astype(np.float32)).cuda().to(dtype)
        c = out_buffer(torch, M + 5, N + 24, torch.float32)
        binding.mace_gemm_bf16(handle, la, lb, M, N, K, a, b, c, resid=r, ldc=N + 24, ldr=N + 2)
        torch.cuda.synchronize()
        check_out(c, ref + f64(r)[:, :N], M, N, 1e-5, f"{la}{lb} {M}x{N}x{K} residual {dtype}")


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("M,F,K", [(3, 64, 64), (128, 704, 256), (65, 72, 192), (200, 2752, 384)])
def test_swiglu(torch_mod, handle, M, F, K, two):
    """silu(G) U of single or two-term activations; the second product of the launch, to one bf16 rounding of the result (2^-9 of each value,
    4e-3 of the largest as in test_gpu_gemm_kernel)."""
    torch = torch_mod
    from paper_2510_03283_amd import binding
    rng = np.random.default_rng(M + F + K + two)
    a, bg, A, G = operands(torch, rng, 0, 0, M, F, K)
    _, bu, _, U = operands(torch, rng, 0, 0, M, F, K)
    lo = (torch.from_numpy(rng.uniform(-1, 1, (M, K)).astype(np.float32)).cuda() * 2.0 ** -9).to(torch.bfloat16) if two else None
    if two:
        A = A + f64(lo)
    s = K ** -0.5
    bg, bu = (bg.float() * s).to(torch.bfloat16), (bu.float() * s).to(torch.bfloat16)
    g, u = A @ f64(bg).T, A @ f64(bu).T
    ref = g / (1.0 + np.exp(-g)) * u
    c = out_buffer(torch, M + 5, F + 8, torch.bfloat16)
    binding.mace_gemm_bf16(handle, 0, 0, M, F, K, a, bg, c, a_lo=lo, b_up=bu, ldc=F + 8, swiglu=True)
    check_tile(binding, handle, [(64, 128)])
    torch.cuda.synchronize()
    check_out(c, ref, M, F, 4e-3, f"swiglu {M}x{F}x{K} two terms {two}")
