"""Layer steps at widths and row counts off the matrix kernel's tiles: output columns that end inside a
64-, 128- or 256-wide tile, reductions that end inside a 64-deep k-tile (down to a single 8-element chunk),
one row, one row past a tile; forward and adjoint against the CPU oracle at the bf16 tolerance."""
import pytest

from paper_2601_09026_amd import workloads as wls

from test_gpu_layer_step import make, run_adjoint_case, run_forward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,f,B,S,G", [
    (8, 2, 8, 1, 1, 1),            # one row, one 16-byte chunk per matrix row
    (72, 2, 136, 1, 65, 2),        # one k-tile plus one chunk; one row past a 64-row tile
    (64, 1, 192, 2, 64, 5),        # half a 128-wide tile, whole k-tiles
    (200, 5, 600, 3, 43, 2),       # k tails of 8 and 24 elements, 129 rows
    (320, 5, 1280, 1, 129, 2),     # two and a half 128-wide tiles
    (960, 15, 960, 1, 257, 1),     # seven and a half; one row past a 256-row tile
    (320, 5, 320, 16, 256, 5),     # enough rows for the large tiles, ragged columns
])
def test_ragged_matrix_shapes_bf16(d, H, f, B, S, G):
    wl = make(wls.ARCH_CAUSAL, wls.DTYPE_BF16, d=d, H=H, f=f, B=B, S=S)
    run_forward_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
    if B * S <= 512:               # (the float64 oracle is slow at the largest shape)
        run_adjoint_case(wl, G=G, hstep=0.5, with_rhs=True, weight_std=0.05, force_simple=0)
