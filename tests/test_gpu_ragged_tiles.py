"""Layer steps at widths and row counts off the matrix kernel's tiles: output columns that end inside a
64-, 128- or 256-wide tile, reductions that end inside a 64-deep k-tile (down to a single 8-element chunk),
one row, one row past a tile; forward and adjoint against the CPU oracle at the bf16 tolerance.  Left to the
rule, all but the last of the first list run on 64x64 tiles; the second list runs on every tile in turn."""
import pytest

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from test_gpu_layer_step import make, run_adjoint_case, run_forward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,f,B,S,G", [
    (8, 2, 8, 1, 1, 1),            # one row, one 16-byte chunk per matrix row
    (72, 2, 136, 1, 65, 2),        # one k-tile plus one chunk; one row past a 64-row tile
    (64, 1, 192, 2, 64, 5),        # whole tiles and k-tiles
    (200, 5, 600, 3, 43, 2),       # k tails of 8 and 24 elements, 129 rows
    (320, 5, 1280, 1, 129, 2),     # whole columns and k-tiles, one row past two tiles
    (960, 15, 960, 1, 257, 1),     # one row past four
    (320, 5, 320, 16, 256, 5),     # enough rows for the large tiles, ragged columns
])
def test_ragged_matrix_shapes_bf16(d, H, f, B, S, G):
    wl = make(wls.ARCH_CAUSAL, wls.DTYPE_BF16, d=d, H=H, f=f, B=B, S=S)
    run_forward_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
    if B * S <= 512:               # (the float64 oracle is slow at the largest shape)
        run_adjoint_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)


@pytest.mark.parametrize("tiles,d,H,f,B,S", [
    *[(t, 200, 5, 600, 3, 90) for t in (1, 4, 6, 8, 9)],     # every edge inside a tile: 270 rows, 200 and 600 columns, k tails of 8 and 24
    *[(t, 264, 3, 776, 1, 257) for t in (1, 4, 6, 8, 9)],    # one row and one 8-column chunk past a 256-wide tile
    (4, 192, 3, 384, 1, 257),                                # short reductions: four wavefronts to a 128x128 tile
    (3, 192, 3, 384, 1, 257),                                # 256x192: ragged rows only
])
def test_each_tile_at_its_edges_bf16(tiles, d, H, f, B, S):
    wl = make(wls.ARCH_CAUSAL, wls.DTYPE_BF16, d=d, H=H, f=f, B=B, S=S)
    print(f"[case] tile configuration {tiles}", flush=True)
    mb.lib().mgrit_debug_gemm_tile_config(tiles)
    try:
        run_forward_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
        run_adjoint_case(wl, G=2, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
    finally:
        mb.lib().mgrit_debug_gemm_tile_config(0)
