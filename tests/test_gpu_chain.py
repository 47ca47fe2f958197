"""Layers 64 and 128 wide in bf16, and 64 wide in fp32, run what is local to a token row as one launch on either side of
attention.  These launches against the general path (one launch per operator, chosen by the hook that fixes the products' tiles) at the
edges of their tiles: 32 rows a wavefront, 64 or 128 a block, chunks of 64 hidden features, ring of eight weight tiles.

Bounds.  bf16: both paths round the same intermediates and differ in the order of fp32 sums, so an operand differs by at most
one step of bf16, which is at most 2^-7 of its value, and so does a row's increment if all its operands do, in the same sense:
row by row 2^-7 (measured up to 0.65 of that, in the rows of smallest increment among 16384; a fragment of 16 features that is
not what it should be moves its row by 0.3).  A layer as a whole differs less, most operands being the same: 2^-9 (measured
1e-7 to 1e-3).  In a training step such differences come in once more with each solve: one step for Z, two for lambda, whose
operands differ and which is linearised at states that do, three for the gradients formed from both, of 2^-7 for a row and of
2^-8 for the whole (measured up to 0.75 and 0.6 of these).  Rows and columns of a gradient are sums over the tokens, which may cancel
while the differences of their terms do not: theirs is 2^-7 of the root mean square over the rows where that is larger (one
wrong fragment of one token among 72 moves a column by 0.1 of it).  (The general path alone moves lambda by 3.7e-3 when 1e-5
is added to every Z; the paths differ by 4.0e-3 there.)
fp32, row by row: sums of up to 256 products in another order, 2^-24 times a random walk of 16 steps and as much again for each
of the four products on the way: 64 roundings of the increment; and the rounding of the state itself on either side."""
import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel, dev
from test_gpu_layer_step import make
from test_gpu_linearised import poisoned
from test_gpu_param_grads import grad_blocks

pytestmark = pytest.mark.gpu
STEP = 2.0 ** -7


def both_paths(run):
    out = []
    for cfg in (0, 4):
        mb.lib().mgrit_debug_gemm_tile_config(cfg)
        try:
            out.append(run())
        finally:
            mb.lib().mgrit_debug_gemm_tile_config(0)
    return out


def close_f32(a, b, base, what, roundings=1, steps=1):
    a, b, base = a.double(), b.double(), base.double()
    assert torch.isfinite(a).all(), what
    q = ((a - b).norm(dim=-1) / (2.0 ** -24 * (64 * roundings * (b - base).norm(dim=-1) + 4 * steps * b.norm(dim=-1)))).max().item()
    print(f"  {what}: {q:.3f} of the bound", flush=True)
    assert q <= 1, what


def close(a, b, base, what, roundings=1, whole=None, of_sums=False):
    a, b, base = a.double(), b.double(), base.double()
    assert torch.isfinite(a).all(), what
    rows = (b - base).norm(dim=-1)
    if of_sums:
        rows = torch.maximum(rows, rows.square().mean().sqrt())
    q = ((a - b).norm(dim=-1) / (roundings * STEP * rows)).max().item()
    w = ((a - b).norm() / (b - base).norm()).item()
    print(f"  {what}: {q:.4f} of the rows' bound; whole {w:.1e}", flush=True)
    assert q <= 1, what
    assert whole is None or w <= whole, what


def close_gradients(desc, a, b, near, layer):
    """Matrices by rows and by columns, vectors as a whole."""
    a, b = mb.unpack_grad(desc, a), mb.unpack_grad(desc, b)
    for name, x in a.items():
        x, y = torch.from_numpy(x), torch.from_numpy(b[name])
        near(x, y, torch.zeros_like(y), f"{name} of layer {layer}")
        if x.dim() == 2:
            near(x.t(), y.t(), torch.zeros_like(y.t()), f"{name} of layer {layer}, columns")


def states(wl, G, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [list(torch.randn((G, wl.tokens, wl.d_model), generator=gen, device="cuda")) for _ in range(3)]


def steps(dm, wl, adjoint, ins, lin, rhs):
    mem = wls.cross_memory(wl)
    outs = [torch.full_like(x, float("nan")) for x in ins]
    mb.layer_step_batched(dm.desc, adjoint, ins, outs, dm.blocks, 0.5, lin_state=lin if adjoint else None, rhs=rhs,
                          memory=None if mem is None else dev(mem))
    torch.cuda.synchronize()
    return outs


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("arch,d,H,f,B,S,Sm,G,rhs", [
    (wls.ARCH_ENCODER, 64, 1, 64, 1, 1, 0, 1, False),         # one token, one chunk: fewer tiles than the ring has slots
    (wls.ARCH_CAUSAL, 64, 4, 128, 1, 31, 0, 2, True),
    (wls.ARCH_ENCODER, 64, 1, 192, 1, 33, 0, 3, False),
    (wls.ARCH_CROSS, 64, 2, 256, 3, 43, 7, 2, True),          # 129 rows
    (wls.ARCH_ENCODER, 64, 1, 512, 2, 64, 0, 1, False),
    (wls.ARCH_ENCODER, 64, 2, 2048, 16, 129, 0, 1, True),     # 2064 tokens: launch by launch both times
    (wls.ARCH_ENCODER, 64, 2, 2048, 127, 130, 0, 1, True),    # 16510 tokens, the widest hidden layer
    (wls.ARCH_CAUSAL, 128, 1, 64, 1, 32, 0, 1, True),
    (wls.ARCH_ENCODER, 128, 2, 128, 1, 63, 0, 3, False),
    (wls.ARCH_CROSS, 128, 2, 192, 1, 127, 33, 2, True),       # (decoders of few tokens: launch by launch both times)
    (wls.ARCH_CROSS, 128, 2, 192, 9, 115, 33, 2, True),       # 1035 tokens
    (wls.ARCH_CROSS, 128, 2, 128, 1, 127, 33, 2, True),
    (wls.ARCH_CAUSAL, 128, 4, 256, 1, 128, 0, 2, False),
    (wls.ARCH_ENCODER, 128, 1, 128, 4, 4096, 0, 2, True),     # 256 blocks of 128 rows
    (wls.ARCH_CAUSAL, 128, 2, 512, 8, 257, 0, 5, True),       # 2056 tokens: launch by launch both times
    (wls.ARCH_CAUSAL, 128, 2, 512, 12, 257, 0, 5, True),      # 3084 tokens: 512 hidden features from 3072 on
    (wls.ARCH_CROSS, 128, 1, 448, 26, 239, 21, 1, False),     # 6214 tokens, seven chunks
])
def test_steps_match_general_path(arch, d, H, f, B, S, Sm, G, rhs, adjoint):
    wl = make(arch, wls.DTYPE_BF16, d=d, H=H, f=f, B=B, S=S, Sm=Sm)
    print(f"[case] chain steps arch={arch} d={d} f={f} B={B} S={S} Sm={Sm} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.08, keep_host=False)
    ins, lin, r = states(wl, G, 5)
    chain, general = both_paths(lambda: steps(dm, wl, adjoint, ins, lin, r if rhs else None))
    for g in range(G):
        close(chain[g], general[g], ins[g] + r[g] if rhs else ins[g], f"group {g}", whole=2.0 ** -9)


def profiled(run):
    """Launches of chains and the bytes reported for them."""
    mb.mgrit_profile_enable(256)
    try:
        mb.mgrit_profile_reset()
        run()
        torch.cuda.synchronize()
        c = mb.mgrit_profile_read().get("chain", {"launches": 0, "bytes": 0.0})
        return c["launches"], c["bytes"]
    finally:
        mb.mgrit_profile_enable(0)


@pytest.mark.parametrize("dtype,d,f,B,S,chain", [
    (wls.DTYPE_BF16, 64, 512, 1, 8, True), (wls.DTYPE_BF16, 64, 576, 1, 2047, False), (wls.DTYPE_BF16, 64, 576, 1, 2048, True),
    (wls.DTYPE_BF16, 64, 768, 1, 2048, True), (wls.DTYPE_BF16, 64, 832, 3, 2047, False), (wls.DTYPE_BF16, 64, 832, 3, 2048, True),
    (wls.DTYPE_BF16, 64, 1024, 3, 2048, True), (wls.DTYPE_BF16, 64, 1088, 127, 129, False), (wls.DTYPE_BF16, 64, 1088, 128, 128, True),
    (wls.DTYPE_BF16, 64, 2112, 128, 129, False),
    (wls.DTYPE_BF16, 128, 256, 1, 8, True), (wls.DTYPE_BF16, 128, 320, 1, 2047, False), (wls.DTYPE_BF16, 128, 384, 1, 2048, True),
    (wls.DTYPE_BF16, 128, 448, 1, 3071, False), (wls.DTYPE_BF16, 128, 512, 1, 3072, True),
    (wls.DTYPE_BF16, 128, 576, 5, 2047, False), (wls.DTYPE_BF16, 128, 1024, 5, 2048, True),
    (wls.DTYPE_BF16, 128, 1088, 127, 129, False), (wls.DTYPE_BF16, 128, 2048, 128, 128, True),
    (wls.DTYPE_BF16, 64, 96, 1, 64, False), (wls.DTYPE_BF16, 192, 192, 1, 64, False),
    (wls.DTYPE_F32, 64, 256, 1, 8, True), (wls.DTYPE_F32, 64, 192, 1, 8, False), (wls.DTYPE_F32, 128, 128, 1, 8, False)])
def test_where_the_lines_lie(dtype, d, f, B, S, chain):
    """Either side of each line of the rule: widths, hidden widths and the tokens from which wide hidden layers take chains."""
    check_path(wls.ARCH_ENCODER, dtype, d, f, B, S, chain)


@pytest.mark.parametrize("dtype,d,f,B,S,chain", [
    (wls.DTYPE_BF16, 64, 512, 1, 8, True), (wls.DTYPE_BF16, 64, 1024, 3, 2048, True), (wls.DTYPE_F32, 64, 256, 1, 8, True),
    (wls.DTYPE_BF16, 128, 128, 1, 8, True), (wls.DTYPE_BF16, 128, 192, 1, 1023, False), (wls.DTYPE_BF16, 128, 256, 1, 1024, True),
    (wls.DTYPE_BF16, 128, 320, 3, 1023, False), (wls.DTYPE_BF16, 128, 384, 3, 1024, True),
    (wls.DTYPE_BF16, 128, 448, 3, 2047, False), (wls.DTYPE_BF16, 128, 512, 3, 2048, True), (wls.DTYPE_BF16, 128, 576, 3, 2048, False)])
def test_where_the_lines_of_decoders_lie(dtype, d, f, B, S, chain):
    check_path(wls.ARCH_CROSS, dtype, d, f, B, S, chain)


def check_path(arch, dtype, d, f, B, S, chain):
    wl = make(arch, dtype, d=d, H=d // 64, f=f, B=B, S=S, Sm=16)
    print(f"[case] chain or not arch={arch} dtype={dtype} d={d} f={f} B={B} S={S}", flush=True)
    dm = DeviceModel(wl, n_layers=1, weight_std=0.08, keep_host=False)
    ins, lin, _ = states(wl, 1, 9)
    assert profiled(lambda: steps(dm, wl, False, ins, lin, None))[0] == (2 if chain else 0)
    assert profiled(lambda: steps(dm, wl, True, ins, lin, None))[0] == (4 if chain else 0)    # the layer's cache entries as well


@pytest.mark.parametrize("arch", [wls.ARCH_ENCODER, wls.ARCH_CROSS])
@pytest.mark.parametrize("dtype,d,f,e", [(wls.DTYPE_BF16, 64, 192, 2), (wls.DTYPE_BF16, 128, 128, 2), (wls.DTYPE_F32, 64, 128, 4)])
def test_reported_bytes(dtype, d, f, e, arch):
    """What a launch reports as its bytes: every row that it reads or writes, by the width of its type and if it is there."""
    G, cross = 3, arch == wls.ARCH_CROSS
    wl = wls.Workload("t", arch, d, 1, f, 1, 40, 24 if cross else 0, G, 0.5, 1, 1, 0, dtype, 23)
    print(f"[case] chain bytes dtype={dtype} d={d} arch={arch}", flush=True)
    dm = DeviceModel(wl, weight_std=0.08, keep_host=False)
    ins, lin, rhs = states(wl, G, 9)
    n, again = G * wl.tokens, 4 * d if d == 128 else 0                            # (X is read a second time)
    head, tail = 4 * d + 3 * e * d, (e + 4) * d + (4 * d if cross else 0)
    out, entries = 4 * d + again, e * d + e * (d + f)                             # the step's; normalised rows and gelu'
    assert profiled(lambda: steps(dm, wl, False, ins, lin, None))[1] == n * (head + tail + out)
    assert profiled(lambda: steps(dm, wl, False, ins, lin, rhs))[1] == n * (head + tail + out + 4 * d)
    adj_tail, adj_head = 4 * d + (2 * e + 4) * d + e * f, 4 * e * d + 12 * d      # from an fp32 cotangent
    assert profiled(lambda: steps(dm, wl, True, ins, lin, rhs))[1] == n * (head + tail + entries + adj_tail + adj_head + 4 * d)

    opts = mb.mgrit_opts(G, 0.5, 1, 1, 0)
    mem = dev(wls.cross_memory(wl)) if cross else None
    ws = torch.empty(mb.mgrit_workspace_bytes(dm.desc, opts, 2), dtype=torch.uint8, device="cuda")
    lamN, Z = dev(wls.terminal_adjoint(wl)), []
    kept = 2 * e * d + 4 * d + e * f                                              # both LayerNorms' outputs, ybar, gelu
    forward = lambda: Z.append(mb.mgrit_forward(dm.desc, opts, ins[0], dm.blocks, memory=mem, adjoint_workspace=ws,
                                                with_gradients=True)[0])
    assert profiled(forward)[1] == n * (head + tail + out + entries + kept)
    dE = torch.empty_like(mem) if cross else None
    adjoint = lambda: mb.mgrit_adjoint(dm.desc, opts, Z[0], dm.blocks, lamN, memory=mem, dtheta=grad_blocks(dm.desc, G),
                                       dmemory=dE, workspace=ws, linearised=True)
    left = e * f + 3 * e * d                                                      # dz, du, ds, du of the projection
    assert profiled(adjoint)[1] == n * (adj_tail - (4 - e) * d + adj_head + left + e * d)   # copies of the cotangents: read, written


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("arch,H,f,B,S,Sm,G,rhs", [
    (wls.ARCH_ENCODER, 1, 64, 1, 1, 0, 1, True),
    (wls.ARCH_CAUSAL, 4, 128, 1, 15, 0, 2, False),
    (wls.ARCH_ENCODER, 4, 256, 1, 17, 0, 3, True),
    (wls.ARCH_CROSS, 2, 256, 3, 11, 5, 2, True),              # 33 rows
    (wls.ARCH_ENCODER, 1, 256, 5, 205, 0, 16, True),          # 1025 rows: 65 tiles of 16, 1040 of them: two a block
    (wls.ARCH_CAUSAL, 2, 64, 16, 64, 0, 16, False),           # 1024 tiles, two a block
    (wls.ARCH_CAUSAL, 2, 128, 1, 1008, 0, 16, False),         # 1008, one a block
])
def test_fp32_steps_match_general_path(arch, H, f, B, S, Sm, G, rhs, adjoint):
    wl = make(arch, wls.DTYPE_F32, d=64, H=H, f=f, B=B, S=S, Sm=Sm)
    print(f"[case] fp32 chain steps arch={arch} f={f} B={B} S={S} Sm={Sm} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.08, keep_host=False)
    ins, lin, r = states(wl, G, 8)
    chain, general = both_paths(lambda: steps(dm, wl, adjoint, ins, lin, r if rhs else None))
    for g in range(G):
        close_f32(chain[g], general[g], ins[g] + r[g] if rhs else ins[g], f"group {g}")


@pytest.mark.parametrize("arch,dtype,d,H,f,S,Sm,N,cf,levels", [
    (wls.ARCH_ENCODER, wls.DTYPE_BF16, 64, 1, 128, 36, 0, 16, 4, 2),
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 128, 2, 256, 68, 0, 8, 2, 3),
    (wls.ARCH_CROSS, wls.DTYPE_BF16, 128, 1, 64, 20, 44, 8, 4, 2),
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 64, 2, 64, 132, 0, 5, 1, 1),   # serial: gradients beside the chain of steps
    (wls.ARCH_ENCODER, wls.DTYPE_F32, 64, 2, 256, 37, 0, 8, 4, 2),
    (wls.ARCH_CROSS, wls.DTYPE_F32, 64, 1, 128, 20, 45, 8, 2, 2),
    (wls.ARCH_CAUSAL, wls.DTYPE_F32, 64, 4, 64, 19, 0, 5, 1, 1),
])
@pytest.mark.parametrize("cache", [True, False])
def test_training_matches_general_path(arch, dtype, d, H, f, S, Sm, N, cf, levels, cache):
    """Both solves with every gradient, from the linearisation cache and with the internals recomputed."""
    iters = 2 if levels > 1 else 0
    wl = wls.Workload("t", arch, d, H, f, 2, S, Sm, N, 0.5, cf, levels, iters, dtype, 17)
    print(f"[case] chain training arch={arch} dtype={dtype} d={d} f={f} S={S} N={N} cf={cf} L={levels} cache={cache}", flush=True)
    dm = DeviceModel(wl, weight_std=0.08, keep_host=False)
    opts = mb.mgrit_opts(N, wl.h, cf, levels, iters)
    mem = wls.cross_memory(wl)
    mem = None if mem is None else dev(mem)
    Z0, lamN = dev(wls.initial_state(wl)), dev(wls.terminal_adjoint(wl))

    def run():
        Z, _ = mb.mgrit_forward(dm.desc, opts, Z0, dm.blocks, memory=mem)
        gb, dE = grad_blocks(dm.desc, N), None if mem is None else torch.full_like(mem, float("nan"))
        lam, _ = mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lamN, memory=mem, dtheta=gb, dmemory=dE)
        torch.cuda.synchronize()
        return Z, lam, gb, dE

    mb.mgrit_set_adjoint_cache(cache)
    try:
        chain, general = both_paths(run)
    finally:
        mb.mgrit_set_adjoint_cache(True)

    def near(x, y, base, what, roundings):
        if dtype == wls.DTYPE_F32:
            close_f32(x, y, base, what, roundings, N)
        else:
            close(x, y, base, what, roundings, roundings * 2.0 ** -8, of_sums=roundings == 3)
    near(chain[0][1:], general[0][1:], Z0.expand_as(chain[0][1:]), "Z", 1)
    near(chain[1][:-1], general[1][:-1], lamN.expand_as(chain[1][:-1]), "lambda", 2)
    if mem is not None:
        near(chain[3], general[3], torch.zeros_like(mem), "memory", 3)
    for n, (x, y) in enumerate(zip(chain[2], general[2])):
        close_gradients(dm.desc, x, y, lambda *a: near(*a, 3), n)


# 4 x ceil(4318 / 128) = 136 blocks of 128 rows, more than half of 256 compute units, and 1080 of 16: more than four each
@pytest.mark.parametrize("grads", [False, True])
@pytest.mark.parametrize("arch,dtype,d,f", [
    (wls.ARCH_ENCODER, wls.DTYPE_BF16, 64, 192), (wls.ARCH_CROSS, wls.DTYPE_BF16, 64, 64),
    (wls.ARCH_CAUSAL, wls.DTYPE_BF16, 128, 192), (wls.ARCH_CROSS, wls.DTYPE_BF16, 128, 256), (wls.ARCH_ENCODER, wls.DTYPE_BF16, 128, 512),
    (wls.ARCH_ENCODER, wls.DTYPE_F32, 64, 64), (wls.ARCH_CROSS, wls.DTYPE_F32, 64, 128), (wls.ARCH_CAUSAL, wls.DTYPE_F32, 64, 256)])
def test_block_size_does_not_show_in_training(arch, dtype, d, f, grads):
    """Blocks of 64 and 128 rows (fp32 of 16 and 32), with what the cache and the gradients keep stored beside the weight ring:
    the linearising pair of four layers in a launch against that of one and against the plain pair, and the cache itself."""
    N, B, S = 8, 34, 127
    wl = wls.Workload("t", arch, d, d // 64, f, B, S, 31 if arch == wls.ARCH_CROSS else 0, N, 0.25, 2, 2, 1, dtype, 19)
    print(f"[case] chain block size in training arch={arch} dtype={dtype} d={d} f={f} grads={grads}", flush=True)
    dm = DeviceModel(wl, weight_std=0.08, keep_host=False)
    opts = mb.mgrit_opts(N, wl.h, 2, 2, 1)
    mem = wls.cross_memory(wl)
    mem = None if mem is None else dev(mem)
    Z0, lamN = dev(wls.initial_state(wl)), dev(wls.terminal_adjoint(wl))

    def run(n, pair):
        mb.mgrit_set_max_groups_per_launch(n)
        ws = poisoned(mb.mgrit_workspace_bytes(dm.desc, opts, 2 if grads else 1))
        Z, _ = mb.mgrit_forward(dm.desc, opts, Z0, dm.blocks, memory=mem, adjoint_workspace=ws if pair else None, with_gradients=grads)
        cache = ws.clone() if pair else None
        gb = grad_blocks(dm.desc, N) if grads else None
        dE = torch.full_like(mem, float("nan")) if grads and mem is not None else None
        lam, _ = mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lamN, memory=mem, dtheta=gb, dmemory=dE, workspace=ws, linearised=pair)
        torch.cuda.synchronize()
        return cache, [Z, lam] + [b.view(torch.float32) for b in gb or []] + ([dE] if dE is not None else [])

    mb.mgrit_set_lanes(1)
    try:
        one, four, plain, plain1 = run(1, True), run(4, True), run(4, False), run(1, False)
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    n = min(one[0].numel(), four[0].numel())                  # (the cache comes first, the rest is as poisoned in both)
    assert torch.equal(one[0][:n], four[0][:n])
    for other in (four, plain, plain1):
        for i, (x, y) in enumerate(zip(one[1], other[1])):
            assert torch.isfinite(x).all() and torch.equal(x, y), f"output {i}"


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype,d,f,B,S,G", [
    (wls.DTYPE_BF16, 64, 256, 8, 512, 5), (wls.DTYPE_BF16, 128, 128, 8, 512, 5),   # blocks of 64 rows alone, of 128 together
    (wls.DTYPE_F32, 64, 256, 8, 512, 5), (wls.DTYPE_F32, 64, 64, 8, 512, 4)])      # 16 and 32
def test_block_size_does_not_show(dtype, d, f, B, S, G, adjoint):
    """How many rows a block takes follows from how many layers share the launch."""
    wl = make(wls.ARCH_CAUSAL, dtype, d=d, H=1, f=f, B=B, S=S)
    print(f"[case] chain block size d={d} f={f} B={B} S={S} G={G} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.08, keep_host=False)
    ins, lin, rhs = states(wl, G, 6)
    out = []
    mb.mgrit_set_lanes(1)
    try:
        for n in (1, G):
            mb.mgrit_set_max_groups_per_launch(n)
            out.append(steps(dm, wl, adjoint, ins, lin, rhs))
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)
    for x, y in zip(*out):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("dtype,d,f", [(wls.DTYPE_BF16, 64, 128), (wls.DTYPE_BF16, 128, 128), (wls.DTYPE_F32, 64, 128)])
def test_non_finite_rows_stay_where_they_are(dtype, d, f):
    """Single-token sequences: what is not finite in one row shows in that row, as on the general path, and nowhere else."""
    wl = make(wls.ARCH_ENCODER, dtype, d=d, H=1, f=f, B=70, S=1)
    print(f"[case] chain non-finite d={d}", flush=True)
    dm = DeviceModel(wl, n_layers=1, weight_std=0.08, keep_host=False)
    ins, lin, _ = states(wl, 1, 7)
    for t, v in ((ins, float("nan")), (lin, float("inf"))):
        t[0][3, 5] = v
        t[0][69, d - 1] = -float("inf")
    for adjoint in (False, True):
        chain, general = both_paths(lambda: steps(dm, wl, adjoint, ins, lin, None)[0])
        assert torch.equal(torch.isfinite(chain), torch.isfinite(general))
        assert torch.isfinite(chain).all(dim=1).sum() == 68
