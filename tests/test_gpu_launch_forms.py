"""Forms of a launch that a rule on its size chooses, at the edges of those rules: the walking form of the
multiply-by-GELU' products (more than one 256x256 tile per compute unit) against 128x128 tiles, bit for bit; bf16
attention at the edges of its 32-row units, 64-row tiles and rings of three tiles against the CPU oracle; many layers of
few tokens in one launch against one layer per launch, bit for bit; keys and values of the decoder's memory formed once
per layer against formed in every step, bit for bit."""
import ctypes as C

import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel, dev
from test_gpu_layer_step import make, run_adjoint_case, run_forward_case
from test_gpu_param_grads import run_case

pytestmark = pytest.mark.gpu


def step(dm, wl, adjoint, G, seed=3):
    rng = torch.Generator(device="cuda")
    rng.manual_seed(seed)
    ins, lin = (list(torch.randn((G, wl.tokens, wl.d_model), generator=rng, device="cuda")) for _ in range(2))
    mem = wls.cross_memory(wl)
    outs = [torch.full_like(x, float("nan")) for x in ins]
    mb.layer_step_batched(dm.desc, adjoint, ins, outs, dm.blocks, 0.5, lin_state=lin if adjoint else None,
                          memory=None if mem is None else dev(mem))
    torch.cuda.synchronize()
    return outs


@pytest.mark.parametrize("d,H,f,B,S,G", [
    (128, 2, 512, 4, 2050, 4),      # two k-tiles a tile, 264 tiles, two columns of them; the last row tile holds 8 rows
    (192, 3, 1280, 1, 3329, 4),     # three k-tiles, five columns, one row past 13 row tiles
    (256, 4, 2048, 8, 256, 5),      # whole tiles, eight columns in 4x4 patches
])
def test_walking_products_bits(d, H, f, B, S, G):
    wl = make(wls.ARCH_ENCODER, wls.DTYPE_BF16, d=d, H=H, f=f, B=B, S=S)
    print(f"[case] walking products d={d} f={f} B={B} S={S} G={G}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    mb.mgrit_set_lanes(1)
    mb.mgrit_set_max_groups_per_launch(G)
    try:
        out = {}
        for cfg in (4, 1):
            mb.lib().mgrit_debug_gemm_tile_config(cfg)
            out[cfg] = step(dm, wl, True, G)
    finally:
        mb.lib().mgrit_debug_gemm_tile_config(0)
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    for g in range(G):
        assert torch.isfinite(out[1][g]).all(), f"group {g}"
        assert torch.equal(out[1][g], out[4][g]), f"group {g}"


@pytest.mark.parametrize("arch,dh,S,Sm", [
    *[(wls.ARCH_CAUSAL, 64, S, 0) for S in (32, 33, 64, 65, 96, 97, 128, 129, 161, 192, 193, 257)],
    *[(wls.ARCH_ENCODER, 64, S, 0) for S in (1, 63, 127, 160, 191, 225)],
    *[(wls.ARCH_CROSS, 64, S, Sm) for S, Sm in ((33, 129), (65, 31), (129, 257), (130, 64), (1, 200))],
    *[(wls.ARCH_CAUSAL, 128, S, 0) for S in (33, 129, 193)], (wls.ARCH_CROSS, 128, 97, 161), (wls.ARCH_ENCODER, 128, 257, 0),
])
def test_attention_edges_bf16(arch, dh, S, Sm):
    wl = make(arch, wls.DTYPE_BF16, d=2 * dh, H=2, f=128, B=1, S=S, Sm=Sm)
    run_forward_case(wl, G=1, hstep=0.5, with_rhs=False, weight_std=0.1, force_simple=0)
    run_adjoint_case(wl, G=1, hstep=0.5, with_rhs=False, weight_std=0.1, force_simple=0)


@pytest.mark.parametrize("dh,arch,B,S,Sm,counts", [
    (64, wls.ARCH_ENCODER, 8, 300, 0, (1, 4, 5)),        # 192 blocks of 128 queries a layer: pipelined up to 768 of them
    (64, wls.ARCH_CAUSAL, 8, 300, 0, (4, 5)),
    (64, wls.ARCH_CROSS, 16, 40, 200, (1, 6, 7)),        # 128 blocks of 64 queries
    (128, wls.ARCH_CROSS, 16, 64, 330, (4, 5, 9)),       # 64 blocks: three sets up to 256, two up to 512, then one
    (128, wls.ARCH_CROSS, 16, 100, 190, (4, 8, 9)),
    (64, wls.ARCH_CROSS, 16, 24, 1030, (1, 9)), (128, wls.ARCH_CROSS, 16, 24, 1030, (1, 9)),  # 304 MB of keys and values
])
def test_attention_ring_bits(dh, arch, B, S, Sm, counts):
    """How many tile sets a block of attention gets, and with which hint it loads, follows from the launch and must not
    show in the result."""
    wl = make(arch, wls.DTYPE_BF16, d=512, H=512 // dh, f=64, B=B, S=S, Sm=Sm)
    print(f"[case] attention rings dh={dh} arch={arch} B={B} S={S} Sm={Sm}", flush=True)
    G = max(counts)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.08, keep_host=False)
    out = {}
    mb.mgrit_set_lanes(1)
    try:
        for n in counts:
            mb.mgrit_set_max_groups_per_launch(n)
            out[n] = step(dm, wl, False, G) + step(dm, wl, True, G)
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    for n in counts[1:]:
        for g, (x, y) in enumerate(zip(out[counts[0]], out[n])):
            assert torch.isfinite(x).all() and torch.equal(x, y), f"{n} layers a launch, state {g}"


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("S,Sm", [
    (40, 200),          # dK/dV pass over one tile set of queries
    (65, 129), (128, 300),                     # over two: 64 KB of tiles at d_head 128, and the rows' scalars beside them
    (200, 40), (400, 50),                      # 64-row blocks of keys, a ring that comes round
])
def test_cross_gradients_unequal_lengths(dh, S, Sm):
    wl = wls.Workload("cross", wls.ARCH_CROSS, 2 * dh, 2, 128, 2, S, Sm, 2, 0.5, 2, 1, 1, wls.DTYPE_BF16, 71)
    run_case(wl, weight_std=0.1)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("arch,dtype,d,f,B,S,Sm,G", [
    (wls.ARCH_ENCODER, wls.DTYPE_F32, 64, 256, 2, 32, 0, 67),      # more than one launch of 64 layers, more than 128 pointers
    (wls.ARCH_CROSS, wls.DTYPE_BF16, 72, 136, 1, 33, 20, 9),       # matrices that are no multiple of the transposed tiles
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 64, 64, 4, 128, 0, 19),      # 4096 rows a launch: 8, 8 and 3 layers
    (wls.ARCH_ENCODER, wls.DTYPE_F32, 256, 1024, 1, 64, 0, 25),    # 16 MiB of intermediates a launch: 21 and 4 layers
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 128, 512, 1, 600, 0, 7),     # four would fit by that: the tile model's six and one
])
def test_few_tokens_bits(arch, dtype, d, f, B, S, Sm, G, adjoint):
    wl = make(arch, dtype, d=d, H=2, f=f, B=B, S=S, Sm=Sm)
    print(f"[case] few tokens arch={arch} dtype={dtype} d={d} B={B} S={S} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    rows, width = wl.tokens + B * Sm, 4 * (8 * d + f)
    fit = min(4096 // rows, (16 << 20) // (rows * width), 64)
    chunk = mb.lib().mgrit_default_groups_per_launch(C.byref(dm.desc), G)
    assert chunk == min(fit, G) if fit > 6 else chunk <= 6
    together = step(dm, wl, adjoint, G)
    mb.mgrit_set_lanes(1)
    mb.mgrit_set_max_groups_per_launch(1)
    try:
        alone = step(dm, wl, adjoint, G)
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    for g in range(G):
        assert torch.isfinite(together[g]).all() and torch.equal(together[g], alone[g]), f"group {g}"


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("arch,dtype,G", [
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 2), (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 3),        # 33.8 and 42.5 us by the tile model
    (wls.ARCH_CROSS, wls.DTYPE_BF16, 2), (wls.ARCH_CROSS, wls.DTYPE_BF16, 3)])
def test_sweeps_in_one_piece_and_split(arch, dtype, G, adjoint):
    """Sweeps that fit a launch, on either side of the line (40 us of products) from which on two lanes share them."""
    wl = make(arch, dtype, d=512, H=8, f=2048, B=8, S=128, Sm=64)
    print(f"[case] one piece or split arch={arch} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    out = {}
    try:
        for lanes in (2, 1):
            mb.mgrit_set_lanes(lanes)
            out[lanes] = step(dm, wl, adjoint, G)
    finally:
        mb.mgrit_set_lanes(2)
    for x, y in zip(out[1], out[2]):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype,d,B,S,G", [
    (wls.DTYPE_BF16, 512, 4, 512, 5), (wls.DTYPE_BF16, 768, 4, 512, 4),          # 108 and 163 us: the line is at 110
    (wls.DTYPE_F32, 512, 4, 256, 4), (wls.DTYPE_F32, 512, 8, 256, 4)])           # 291 and 570 us: at 300
def test_sweeps_around_the_line_of_two_lanes(dtype, d, B, S, G, adjoint):
    wl = make(wls.ARCH_CAUSAL, dtype, d=d, H=d // 64, f=4 * d, B=B, S=S)
    print(f"[case] two lanes or one dtype={dtype} d={d} B={B} S={S} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    out = {}
    try:
        for lanes in (2, 1):
            mb.mgrit_set_lanes(lanes)
            out[lanes] = step(dm, wl, adjoint, G)
    finally:
        mb.mgrit_set_lanes(2)
    for x, y in zip(out[1], out[2]):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("dtype,d,S,Sm,N,cf,levels,relax,lanes,mg", [
    (wls.DTYPE_BF16, 128, 40, 24, 16, 4, 2, 1, 2, 0),
    (wls.DTYPE_BF16, 128, 17, 65, 8, 2, 3, 0, 1, 0),
    (wls.DTYPE_BF16, 256, 40, 1, 32, 4, 3, 1, 2, 3),
    (wls.DTYPE_F32, 128, 24, 40, 8, 2, 2, 1, 2, 2),
])
def test_kept_memory_projections_bits(dtype, d, S, Sm, N, cf, levels, relax, lanes, mg):
    wl = wls.Workload("t", wls.ARCH_CROSS, d, d // 64, 2 * d, 2, S, Sm, N, 0.5, cf, levels, 2, dtype, 93, relax=relax)
    print(f"[case] kept memory projections dtype={dtype} d={d} S={S} Sm={Sm} N={N} cf={cf} L={levels}", flush=True)
    dm = DeviceModel(wl, weight_std=0.05, keep_host=False)
    opts, buf = mb.mgrit_opts(N, wl.h, cf, levels, 2, relax), mb.BufferOpts(0, 0, 0.0)
    mem, Z0 = dev(wls.cross_memory(wl)), dev(wls.initial_state(wl))
    mb.mgrit_set_lanes(lanes)
    mb.mgrit_set_max_groups_per_launch(mg)
    try:
        room = mb.mgrit_workspace_bytes(dm.desc, opts, 0)
        mb.mgrit_set_adjoint_cache(False)
        least = mb.mgrit_workspace_bytes(dm.desc, opts, 0)
        mb.mgrit_set_adjoint_cache(True)
        outs = []
        for size in (room, room - 256, least):
            ws = torch.full((size // 4,), float("nan"), device="cuda").view(torch.uint8)
            outs.append(mb.mgrit_forward(dm.desc, opts, Z0, dm.blocks, memory=mem, workspace=ws))
            torch.cuda.synchronize()
        Z, r = torch.empty_like(outs[0][0]), torch.empty_like(outs[0][1])         # a buffered run in the least space
        assert mb.lib().mgrit_forward_buffered(C.byref(dm.desc), C.byref(opts), C.byref(buf), mb._ptr(Z0),
                                               mb._ptr_array(dm.blocks), mb._ptr(mem), mb._ptr(Z), mb._ptr(r),
                                               mb._ptr(ws), ws.numel(), mb._stream_handle(None)) == mb.MGRIT_OK
        torch.cuda.synchronize()
        outs.append((Z, r))
        with pytest.raises(mb.MgritError) as e:
            mb.mgrit_forward(dm.desc, opts, Z0, dm.blocks, memory=mem, workspace=ws[:-256])
        assert e.value.status == mb.MGRIT_WORKSPACE_TOO_SMALL
    finally:
        mb.mgrit_set_adjoint_cache(True)
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    assert torch.isfinite(outs[0][0]).all() and torch.isfinite(outs[0][1]).all()
    for Z, r in outs[1:]:
        assert torch.equal(Z, outs[0][0]) and torch.equal(r, outs[0][1])
