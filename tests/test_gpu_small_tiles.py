"""Kernel-level parity of the dense contraction on the small tiles (64x64, 64x128) that the launcher takes for few rows and short
reductions: one block and one row or column past it, reductions of one k tile and with a remainder (token-contracting form), every
layout, output type and residual, and the SwiGLU form with what the forward keeps of it; the launch plan confirms the tile of every call.
Definition, buffers and bars as in test_gpu_gemm_kernel."""
import numpy as np
import pytest

from test_gpu_gemm_kernel import SENT, check_out, f64, handle, operands, out_buffer  # noqa: F401

pytestmark = pytest.mark.gpu


def check_tile(binding, handle, tile):
    (r,) = binding.mace_launch_plan(handle)
    assert tuple(r["tile"]) == tile, r["tile"]


# (layout of A, of B, M, N, K) -> tile.  64x128: more blocks than four small tiles a CU, tiles that end inside either half of a pair of fragments, columns that four do not divide
SHAPES = {(0, 0, 1, 2, 64): (64, 64), (0, 0, 64, 64, 128): (64, 64), (0, 0, 65, 66, 64): (64, 64), (0, 0, 234, 768, 256): (64, 64), (0, 0, 400, 840, 704): (64, 64),
          (0, 1, 7, 8, 64): (64, 64), (0, 1, 64, 64, 64): (64, 64), (0, 1, 65, 72, 128): (64, 64), (0, 1, 128, 704, 256): (64, 64), (0, 1, 300, 256, 768): (64, 64),
          (1, 1, 8, 8, 1): (64, 64), (1, 1, 64, 64, 64): (64, 64), (1, 1, 72, 136, 65): (64, 64), (1, 1, 704, 256, 128): (64, 64), (1, 1, 256, 768, 100): (64, 64),
          (0, 0, 1537, 3070, 64): (64, 128), (0, 0, 1536, 3080, 256): (64, 128), (0, 1, 1537, 3080, 192): (64, 128), (0, 1, 1600, 2976, 64): (64, 128),
          (1, 1, 1544, 3080, 1): (64, 128), (1, 1, 1544, 3080, 65): (64, 128), (1, 1, 1600, 2976, 128): (64, 128), (1, 1, 3072, 2048, 300): (64, 128)}


@pytest.mark.parametrize("la,lb,M,N,K", SHAPES)
def test_products(torch_mod, handle, la, lb, M, N, K):
    torch = torch_mod
    from paper_2510_03283_amd import binding
    rng = np.random.default_rng(K + 7 * M + la + 2 * lb)
    a, b, A, B = operands(torch, rng, la, lb, M, N, K)
    ref = A @ B.T
    for dtype, tol in ((torch.float32, 1e-5), (torch.bfloat16, 4e-3)):
        c = out_buffer(torch, M + 5, N + 24, dtype)
        binding.mace_gemm_bf16(handle, la, lb, M, N, K, a, b, c, ldc=N + 24)
        check_tile(binding, handle, SHAPES[la, lb, M, N, K])
        torch.cuda.synchronize()
        check_out(c, ref, M, N, tol, f"{la}{lb} {M}x{N}x{K} {dtype}")
    for dtype in (torch.float32, torch.bfloat16):
        r = torch.from_numpy(rng.uniform(-20, 20, (M, N + 2)).astype(np.float32)).cuda().to(dtype)
        for out, tol in ((torch.float32, 1e-5), (torch.bfloat16, 4e-3)):
            c = out_buffer(torch, M + 5, N + 24, out)
            binding.mace_gemm_bf16(handle, la, lb, M, N, K, a, b, c, resid=r, ldc=N + 24, ldr=N + 2)
            check_tile(binding, handle, SHAPES[la, lb, M, N, K])
            torch.cuda.synchronize()
            check_out(c, ref + f64(r)[:, :N], M, N, tol, f"{la}{lb} {M}x{N}x{K} {out} residual {dtype}")


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("M,F,K", [(3, 64, 64), (128, 704, 256), (65, 72, 192), (200, 2752, 384), (129, 1410, 192)])
def test_swiglu(torch_mod, handle, M, F, K, two, keep):
    """silu(G) U of single or two-term activations; the second product of the launch, to one bf16 rounding of the result (2^-9 of each value,
    4e-3 of the largest as in test_gpu_gemm_kernel).  keep: its second term (5e-5 as there) and G | U are written too."""
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
    c_lo, gu = (out_buffer(torch, M + 5, w, torch.bfloat16) if keep else None for w in (F + 8, 2 * F))
    binding.mace_gemm_bf16(handle, 0, 0, M, F, K, a, bg, c, a_lo=lo, b_up=bu, c_lo=c_lo, c_gu=gu, ldc=F + 8, swiglu=True)
    check_tile(binding, handle, (64, 128))
    torch.cuda.synchronize()
    check_out(c, ref, M, F, 4e-3, f"swiglu {M}x{F}x{K} two terms {two}")
    if keep:
        assert np.abs((f64(c) + f64(c_lo))[:M, :F] - ref).max() / np.abs(ref).max() <= 5e-5, "second term"
        assert np.all(f64(c_lo)[M:] == SENT) and np.all(f64(c_lo)[:M, F:] == SENT)
        check_out(gu, np.concatenate([g, u], axis=1), M, 2 * F, 4e-3, "G | U")
