"""Parameter gradients at the edges of the token-major product: token counts that are no multiple of a k-tile
(or of 4), widths inside a tile, reductions cut into slices, and serial runs whose layer count is no multiple of
the layers per gradient launch (4: batches of 4, 4 and 1, both sets of buffers reused), against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel
from test_gpu_param_grads import grad_blocks, run_case

pytestmark = pytest.mark.gpu

BF16, F32 = wls.DTYPE_BF16, wls.DTYPE_F32


@pytest.mark.parametrize("arch,dtype,d,H,f,B,S,Sm,N,cf,levels", [
    (wls.ARCH_CAUSAL, BF16, 72, 2, 136, 1, 21, 0, 4, 1, 1),        # 21 tokens, widths of one tile plus a chunk
    (wls.ARCH_ENCODER, BF16, 64, 1, 64, 2, 515, 0, 13, 1, 1),      # 17 k-tiles, the last with 6 tokens; batches 4 4 4 1
    (wls.ARCH_ENCODER, BF16, 64, 1, 128, 64, 64, 0, 2, 1, 1),      # 64 k-tiles of one output tile: slices
    (wls.ARCH_CAUSAL, BF16, 264, 3, 520, 1, 130, 0, 4, 2, 2),      # one 8-row and 8-column chunk past whole 64x64 tiles
    (wls.ARCH_CROSS, BF16, 64, 1, 128, 1, 25, 19, 9, 1, 1),        # odd token and memory token counts, serial
    (wls.ARCH_CROSS, F32, 40, 2, 48, 1, 33, 7, 9, 1, 1),
    (wls.ARCH_ENCODER, F32, 64, 4, 64, 16, 64, 0, 4, 2, 2),        # slices in fp32
])
def test_weight_gradient_edges(arch, dtype, d, H, f, B, S, Sm, N, cf, levels):
    wl = wls.Workload("edges", arch, d, H, f, B, S, Sm, N, 1.0 / N, cf, levels, 2 if levels > 1 else 1, dtype, 77)
    run_case(wl, weight_std=0.05)


@pytest.mark.parametrize("tiles,slices,dtype", [
    (1, 0, BF16), (1, 3, BF16), (6, 0, BF16), (6, 3, BF16), (8, 0, BF16), (8, 2, BF16), (0, 3, F32)])
@pytest.mark.parametrize("arch,d,H,f,B,S,Sm", [
    (wls.ARCH_CAUSAL, 264, 3, 520, 1, 130, 0),       # one chunk past 256-wide and 128-wide tiles; k-tiles of 64, 64 and 2 tokens
    (wls.ARCH_CROSS, 200, 5, 136, 3, 45, 24),        # inside them; 135 and 72 tokens
])
def test_each_tile_and_slice_at_its_edges(arch, d, H, f, B, S, Sm, tiles, slices, dtype):
    wl = wls.Workload("edges", arch, d, H, f, B, S, Sm, 2, 0.5, 1, 1, 1, dtype, 79)
    print(f"[case] tile configuration {tiles}, {slices} slices", flush=True)
    mb.lib().mgrit_debug_gemm_tile_config(tiles)
    mb.lib().mgrit_debug_gradient_slices(slices)
    try:
        run_case(wl, weight_std=0.05)
    finally:
        mb.lib().mgrit_debug_gemm_tile_config(0)
        mb.lib().mgrit_debug_gradient_slices(0)


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("d,B,S", [(256, 32, 512), (1024, 8, 512)])     # tokens cut into slices; not cut
def test_bias_gradient_rounding(d, B, S, dtype):
    """The gradient of b2 is h times the sum over tokens of lambda.  Positive terms, so that a rounding of a partial sum
    is one of the result, most of them (fifth powers) far smaller than the sum.  Of the roundings a term takes part in,
    six are in the sums of 32 tokens of a k-tile, two each in the sums of k-tiles and of slices, which carry their
    errors, and one each in adding two halves and multiplying by h: twelve, however many tokens."""
    wl = wls.Workload("sums", wls.ARCH_ENCODER, d, d // 64, d, B, S, 0, 1, 0.3, 1, 1, 1, dtype, 78)
    print(f"[case] bias sums d={d} T={wl.tokens} dtype={dtype}", flush=True)
    dm = DeviceModel(wl, keep_host=False)
    opts = mb.mgrit_opts(1, wl.h, 1, 1, 0)
    gen = torch.Generator(device="cuda").manual_seed(3)
    lam = torch.randn((wl.tokens, d), generator=gen, device="cuda").abs_() ** 5
    Z, _ = mb.mgrit_forward(dm.desc, opts, torch.randn((wl.tokens, d), generator=gen, device="cuda"), dm.blocks)
    grad = grad_blocks(dm.desc, 1)
    mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lam, dtheta=grad)
    got = mb.unpack_grad(dm.desc, grad[0])["b2"].reshape(-1).astype(np.float64)
    terms = lam.bfloat16() if dtype == BF16 else lam
    ref = float(np.float32(wl.h)) * terms.double().sum(0).cpu().numpy()
    worst = np.abs(got / ref - 1.0).max()
    print(f"  largest relative error {worst:.2e}")
    assert worst <= 12 * 2.0 ** -24


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("slices", [1, 3])
def test_infinite_terms_stay_infinite(slices, dtype):
    """One infinite entry of lambda: its column of b2's gradient is infinite, the others are what they are without it."""
    wl = wls.Workload("inf", wls.ARCH_ENCODER, 64, 2, 64, 2, 200, 0, 1, 0.5, 1, 1, 1, dtype, 80)
    print(f"[case] infinite lambda, {slices} slices, dtype={dtype}", flush=True)
    dm = DeviceModel(wl, keep_host=False)
    opts = mb.mgrit_opts(1, wl.h, 1, 1, 0)
    gen = torch.Generator(device="cuda").manual_seed(4)
    lam = torch.randn((wl.tokens, wl.d_model), generator=gen, device="cuda")
    Z, _ = mb.mgrit_forward(dm.desc, opts, torch.randn((wl.tokens, wl.d_model), generator=gen, device="cuda"), dm.blocks)
    mb.lib().mgrit_debug_gradient_slices(slices)
    try:
        b2 = []
        for bad in (False, True):
            if bad:
                lam[70, 5], lam[150, 9] = float("inf"), -float("inf")      # in the first and in a later slice
            grad = grad_blocks(dm.desc, 1)
            mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lam, dtheta=grad)
            b2.append(mb.unpack_grad(dm.desc, grad[0])["b2"].reshape(-1))
    finally:
        mb.lib().mgrit_debug_gradient_slices(0)
    want = b2[0].copy()
    want[5], want[9] = np.inf, -np.inf
    assert np.array_equal(b2[1], want)
