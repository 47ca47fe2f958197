"""Many layers of few tokens share a launch, and the size queries count the buffers of such launches.  A workspace that
is enough for chunks of four layers (fp32) or six (bf16), as before that rule, is accepted by every entry point and gives
the same bits; less than that is refused."""
import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel, dev
from test_gpu_linearised import grad_blocks, poisoned

pytestmark = pytest.mark.gpu

N = 32


def model(arch, dtype, d):
    wl = wls.Workload("t", arch, d, 2 if d == 64 else 3, 2 * d, 2, 24, 16 if arch == wls.ARCH_CROSS else 0, N, 0.5, 2, 2, 2, dtype, 97)
    return wl, DeviceModel(wl, weight_std=0.05, keep_host=False), mb.mgrit_opts(N, wl.h, 2, 2, 2)


def sizes(query, dtype):
    """[as queried, in chunks of four or six]: the second is smaller."""
    full = query()
    try:
        mb.mgrit_set_max_groups_per_launch(4 if dtype == wls.DTYPE_F32 else 6)
        former = query()
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
    assert all(0 < f < a for a, f in zip(full, former)), (full, former)
    return full, former


def same(a, b):
    for x, y in zip(a, b):
        x, y = (t.view(torch.float32) if t.dtype == torch.uint8 else t for t in (x, y))
        assert torch.isfinite(x).all() and torch.equal(x, y)


def refused(call):
    with pytest.raises(mb.MgritError) as e:
        call()
    assert e.value.status == mb.MGRIT_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("d", [64, 192])                  # the row-local chains and launch by launch
@pytest.mark.parametrize("arch,dtype", [(wls.ARCH_ENCODER, wls.DTYPE_F32), (wls.ARCH_CROSS, wls.DTYPE_F32),
                                        (wls.ARCH_CAUSAL, wls.DTYPE_BF16), (wls.ARCH_CROSS, wls.DTYPE_BF16)])
def test_solves(arch, dtype, d):
    wl, dm, opts = model(arch, dtype, d)
    print(f"[case] small workspaces arch={arch} dtype={dtype} d={d}", flush=True)
    mem = wls.cross_memory(wl)
    mem = None if mem is None else dev(mem)
    Z0, lamN = dev(wls.initial_state(wl)), dev(wls.terminal_adjoint(wl))

    def pair(fwd, adj, linearised):
        ws = poisoned(adj)
        Z, r = mb.mgrit_forward(dm.desc, opts, Z0, dm.blocks, memory=mem, workspace=poisoned(fwd),
                                adjoint_workspace=ws if linearised else None, with_gradients=True)
        gb = grad_blocks(dm.desc, N)
        lam, ra = mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lamN, memory=mem, dtheta=gb, workspace=ws,
                                   linearised=linearised)
        torch.cuda.synchronize()
        return [Z, r, lam, ra] + gb
    full, former = sizes(lambda: [mb.mgrit_workspace_bytes(dm.desc, opts, m) for m in (0, 2)], dtype)
    want = pair(*full, False)
    for f, a, lin in ((former[0], former[1], False), (former[0], former[1], True), (former[0], full[1], True),
                      (full[0], former[1], True), (full[0], full[1], True)):
        same(want, pair(f, a, lin))
    if dtype == wls.DTYPE_F32:
        refused(lambda: pair(full[0], former[1] - 256, False))
        if mem is None:                                  # (a decoder can also do without its kept keys and values)
            refused(lambda: pair(former[0] - 256, full[1], False))
        refused(lambda: pair(full[0], former[1] - 256, True))


@pytest.mark.parametrize("d", [64, 192])                  # the row-local chains and launch by launch
@pytest.mark.parametrize("dtype", [wls.DTYPE_F32, wls.DTYPE_BF16])
def test_buffered_and_stacked(dtype, d):
    print(f"[case] small workspaces, buffered and stacked dtype={dtype} d={d}", flush=True)
    wl, _, opts = model(wls.ARCH_ENCODER, dtype, d)
    buf = mb.BufferOpts(3, 2, 1.0)
    dm = DeviceModel(wl, n_layers=N + 5, weight_std=0.05, keep_host=False)
    full, former = sizes(lambda: [mb.mgrit_buffered_linearised_workspace_bytes(dm.desc, opts, buf, True),
                                  mb.mgrit_buffered_workspace_bytes(dm.desc, opts, buf, 2)], dtype)
    Z0, lamN = dev(wls.initial_state(wl)), dev(wls.terminal_adjoint(wl))

    def buffered(lin, plain):
        ws = poisoned(lin or plain)
        Z, r = mb.mgrit_forward_buffered(dm.desc, opts, buf, Z0, dm.blocks, adjoint_workspace=ws if lin else None,
                                         with_gradients=True)
        gb = grad_blocks(dm.desc, N + 5)
        lam, ra = mb.mgrit_adjoint_buffered(dm.desc, opts, buf, Z, dm.blocks, lamN, dtheta=gb, workspace=ws,
                                            linearised=bool(lin))
        torch.cuda.synchronize()
        return [Z, r, lam, ra] + gb
    want = buffered(0, full[1])
    for lin, plain in ((full[0], 0), (former[0], 0), (0, former[1])):
        same(want, buffered(lin, plain))
    if dtype == wls.DTYPE_F32:
        refused(lambda: buffered(former[0] - 256, 0))
        refused(lambda: buffered(0, former[1] - 256))

    dec, _, _ = model(wls.ARCH_CROSS, dtype, d)
    desc = mb.model_desc(dec)
    sw = wls.StackedWorkload("s", wls.Workload("e", wls.ARCH_ENCODER, d, dec.n_heads, 2 * d, 2, 16, 0, 14, 0.5, 2, 2, 2, dtype, 98),
                             wls.Workload("d", wls.ARCH_CROSS, d, dec.n_heads, 2 * d, 2, 24, 16, N - 14, 0.5, 2, 2, 2, dtype, 99))
    descs = [mb.encoder_desc(desc)] * 14 + [desc] * (N - 14)
    blocks = [mb.pack_theta(x, wls.stacked_layer_params(sw, n, 0.05)) for n, x in enumerate(descs)]
    Z0, lamN = dev(wls.stacked_initial_state(sw)), dev(wls.stacked_terminal_adjoint(sw))
    full, former = sizes(lambda: [mb.mgrit_stacked_workspace_bytes(desc, opts, 14, m) for m in (0, 2)], dtype)

    def stacked(fwd, adj, linearised):
        ws = poisoned(adj)
        Z, r = mb.mgrit_forward_stacked(desc, opts, 14, Z0, blocks, workspace=poisoned(fwd),
                                        adjoint_workspace=ws if linearised else None, with_gradients=True)
        gb = [grad_blocks(x, 1)[0] for x in descs]
        lam, ra = mb.mgrit_adjoint_stacked(desc, opts, 14, Z, blocks, lamN, dtheta=gb, workspace=ws,
                                           linearised=linearised)
        torch.cuda.synchronize()
        return [Z, r, lam, ra] + gb
    want = stacked(*full, False)
    for f, a, lin in ((former[0], former[1], False), (former[0], full[1], True), (full[0], former[1], True)):
        same(want, stacked(f, a, lin))
    if dtype == wls.DTYPE_F32:
        refused(lambda: stacked(former[0] - 256, full[1], False))
        refused(lambda: stacked(full[0], former[1] - 256, True))


@pytest.mark.parametrize("d", [64, 192])                  # the row-local chains and launch by launch
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype", [wls.DTYPE_F32, wls.DTYPE_BF16])
def test_layer_step(dtype, adjoint, d):
    wl, _, _ = model(wls.ARCH_CAUSAL, dtype, d)
    G = 20
    print(f"[case] small workspaces, layer step dtype={dtype} d={d} adjoint={adjoint}", flush=True)
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    full, former = sizes(lambda: [mb.mgrit_layer_step_workspace_bytes(dm.desc, adjoint, G)], dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    ins, lin = (list(torch.randn((G, wl.tokens, d), generator=gen, device="cuda")) for _ in range(2))

    def run(size):
        outs = [torch.full_like(x, float("nan")) for x in ins]
        mb.layer_step_batched(dm.desc, adjoint, ins, outs, dm.blocks, 0.5, lin_state=lin if adjoint else None,
                              workspace=poisoned(size))
        torch.cuda.synchronize()
        return outs
    same(run(full[0]), run(former[0]))
    if dtype == wls.DTYPE_F32:
        refused(lambda: run(former[0] - 256))
