"""The fp32 matrix-core kernels where they can go wrong, against the CPU oracle: projections whose columns end
inside a 32- or 64-wide tile and whose reductions end inside a 64- or 32-deep k-tile (down to 8 elements), one row
and one row past a tile; attention (all fp32 heads, bf16 heads that are not 64 or 128 wide) at every padded head width,
sequences of one row, around 16-row parts, around 64-row tiles, over several tiles, and key counts unlike the query
counts.  The attention cases run forward and adjoint; sequences up to 64 take the one-launch backward."""
import pytest

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from test_gpu_layer_step import make, run_adjoint_case, run_forward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,f,B,S,G", [
    (8, 2, 8, 1, 1, 1),            # one row, a quarter of a k-tile
    (40, 2, 72, 1, 65, 2),         # one k-tile and 8 elements; one row past a 64-row tile
    (64, 4, 256, 2, 32, 4),        # whole tiles
    (200, 5, 600, 3, 43, 2),       # ragged columns and reductions, 129 rows
    (200, 5, 600, 16, 129, 4),     # many rows, ragged in every direction (32x32 tiles as well)
    (320, 5, 320, 16, 256, 5),     # enough rows for the 64x64 tiles
    (512, 8, 1024, 8, 256, 4),
])
def test_projection_tiles_fp32(d, H, f, B, S, G):
    wl = make(wls.ARCH_CAUSAL, wls.DTYPE_F32, d=d, H=H, f=f, B=B, S=S)
    run_forward_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
    if B * S <= 512:               # (the float64 oracle is slow at the largest shapes)
        run_adjoint_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)


@pytest.mark.parametrize("d,H,f,B,S", [
    (256, 4, 512, 3, 50),          # 150 rows: two row tiles and 22 rows
    (64, 4, 192, 1, 65),           # one row past a tile
    (192, 2, 320, 2, 64),          # whole tiles
])
def test_projection_on_64x64_tiles_fp32(d, H, f, B, S):
    """The tile of large launches, forward and adjoint, at sizes that the oracle can follow."""
    wl = make(wls.ARCH_CAUSAL, wls.DTYPE_F32, d=d, H=H, f=f, B=B, S=S)
    mb.lib().mgrit_debug_gemm_tile_config(1)
    try:
        run_forward_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
        run_adjoint_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
    finally:
        mb.lib().mgrit_debug_gemm_tile_config(0)


@pytest.mark.parametrize("dtype", [wls.DTYPE_F32, wls.DTYPE_BF16])
@pytest.mark.parametrize("arch,dh,S,Sm", [
    (wls.ARCH_ENCODER, 4, 1, 0), (wls.ARCH_CAUSAL, 16, 17, 0), (wls.ARCH_ENCODER, 20, 63, 0),
    (wls.ARCH_CAUSAL, 32, 64, 0), (wls.ARCH_CAUSAL, 36, 65, 0), (wls.ARCH_ENCODER, 48, 79, 0),
    (wls.ARCH_CAUSAL, 72, 130, 0), (wls.ARCH_ENCODER, 96, 192, 0), (wls.ARCH_CAUSAL, 116, 257, 0),
    (wls.ARCH_CROSS, 32, 20, 130), (wls.ARCH_CROSS, 24, 97, 5),
])
def test_attention_tiles_of_any_head_width(arch, dh, S, Sm, dtype):
    wl = make(arch, dtype, d=2 * dh, H=2, f=64, B=2, S=S, Sm=Sm)
    run_forward_case(wl, G=2, hstep=0.5, with_rhs=False, weight_std=0.05, force_simple=0)
    run_adjoint_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)


@pytest.mark.parametrize("arch,dh,S", [(wls.ARCH_CAUSAL, 64, 200), (wls.ARCH_ENCODER, 128, 130)])
def test_attention_tiles_of_usual_head_widths_fp32(arch, dh, S):
    wl = make(arch, wls.DTYPE_F32, d=2 * dh, H=2, f=64, B=2, S=S)
    run_forward_case(wl, G=2, hstep=0.5, with_rhs=False, weight_std=0.05, force_simple=0)
    run_adjoint_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
