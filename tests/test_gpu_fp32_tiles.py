"""The fp32 matrix-core kernels where they can go wrong, against the CPU oracle: projections whose columns end
inside a 32- or 64-wide tile and whose reductions end inside a 64- or 32-deep k-tile (down to 8 elements), one row
and one row past a tile; attention (all fp32 heads, bf16 heads that are not 64 or 128 wide) at every padded head width,
sequences of one row, around 16-row parts, around 64-row tiles, over several tiles, and key counts unlike the query
counts.  The attention cases run forward and adjoint; sequences up to 64 take the one-launch backward."""
import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel
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


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("d,T,G", [                # tiles of 64 x 64 of the products 256 wide (their reduction 256 and 512):
    (256, 8128, 1), (256, 8192, 1), (256, 8193, 1),            # 508, 512, 516: two rounds on 256 CUs, less, and a third begun
    (256, 4608, 2), (256, 4672, 2),                # 576, 584: the third round filled by a quarter, and by more
    (256, 4096, 3), (256, 4400, 3),                # 768, 828: three rounds, and a fourth filled by a quarter
    (256, 4097, 4)])                               # 1040: four
def test_lines_between_the_tiles_fp32(d, T, G, adjoint):
    """Either side of the lines of the rule that chooses a launch's tile, against both tiles: the same bits."""
    print(f"[case] fp32 tiles T={T} G={G} adjoint={adjoint}", flush=True)
    wl = make(wls.ARCH_ENCODER, wls.DTYPE_F32, d=d, H=4, f=512, B=T, S=1)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    ins, lin = (list(torch.randn((G, T, d), generator=gen, device="cuda")) for _ in range(2))
    out = []
    mb.mgrit_set_lanes(1)
    try:
        for cfg in (0, 1, 8):
            mb.lib().mgrit_debug_gemm_tile_config(cfg)
            out.append([torch.full_like(x, float("nan")) for x in ins])
            mb.layer_step_batched(dm.desc, adjoint, ins, out[-1], dm.blocks, 0.5, lin_state=lin if adjoint else None)
            torch.cuda.synchronize()
    finally:
        mb.lib().mgrit_debug_gemm_tile_config(0)
        mb.mgrit_set_lanes(2)
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert torch.isfinite(x).all() and torch.equal(x, y)


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
