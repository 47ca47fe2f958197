"""Parameter gradients at the edges of the token-major product: token counts that are no multiple of a k-tile
(or of 4), widths inside a tile, reductions cut into slices, and serial runs whose layer count is no multiple of
the layers per gradient launch (4: batches of 4, 4 and 1, both sets of buffers reused), against the CPU oracle."""
import pytest

from paper_2601_09026_amd import workloads as wls

from test_gpu_param_grads import run_case

pytestmark = pytest.mark.gpu

BF16, F32 = wls.DTYPE_BF16, wls.DTYPE_F32


@pytest.mark.parametrize("arch,dtype,d,H,f,B,S,Sm,N,cf,levels", [
    (wls.ARCH_CAUSAL, BF16, 72, 2, 136, 1, 21, 0, 4, 1, 1),        # 21 tokens, widths of one tile plus a chunk
    (wls.ARCH_ENCODER, BF16, 64, 1, 64, 2, 515, 0, 13, 1, 1),      # 17 k-tiles, the last with 6 tokens; batches 4 4 4 1
    (wls.ARCH_ENCODER, BF16, 64, 1, 128, 64, 64, 0, 2, 1, 1),      # 64 k-tiles of one output tile: slices
    (wls.ARCH_CAUSAL, BF16, 264, 3, 520, 1, 130, 0, 4, 2, 2),      # one row and column chunk past 256
    (wls.ARCH_CROSS, BF16, 64, 1, 128, 1, 25, 19, 9, 1, 1),        # odd token and memory token counts, serial
    (wls.ARCH_CROSS, F32, 40, 2, 48, 1, 33, 7, 9, 1, 1),
    (wls.ARCH_ENCODER, F32, 64, 4, 64, 16, 64, 0, 4, 2, 2),        # slices in fp32
])
def test_weight_gradient_edges(arch, dtype, d, H, f, B, S, Sm, N, cf, levels):
    wl = wls.Workload("edges", arch, d, H, f, B, S, Sm, N, 1.0 / N, cf, levels, 2 if levels > 1 else 1, dtype, 77)
    run_case(wl, weight_std=0.05)
