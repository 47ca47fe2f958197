"""How many layers share a launch decides which tiles and kernels run, and must not show in any result: states,
adjoint states and gradients of one and the same call, bit for bit, with one layer per launch and with several.
The sizes lie on both sides of the rules that look at the size of a launch."""
import numpy as np
import pytest
import torch

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import DeviceModel, dev
from test_gpu_layer_step import make

pytestmark = pytest.mark.gpu


def with_groups(counts, run):
    """run() with 1, 2, .. layers per launch on one lane; every result equal to the first."""
    mb.mgrit_set_lanes(1)
    try:
        first = None
        for n in counts:
            mb.mgrit_set_max_groups_per_launch(n)
            out = run()
            torch.cuda.synchronize()
            for name, t in out.items():
                assert torch.isfinite(t).all(), (n, name)
            if first is None:
                first = out
            for name, t in out.items():
                assert torch.equal(t, first[name]), f"{n} layers per launch: {name} differs"
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_lanes(2)


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("dtype,d,f,B,S", [
    (wls.DTYPE_F32, 256, 512, 4, 509),     # 128 row blocks x d/64 columns a layer: below two 64x64 tiles per CU alone, above with 4
    (wls.DTYPE_F32, 192, 320, 2, 150),     # 32x32 tiles always, reductions of 192 and 320
    (wls.DTYPE_BF16, 256, 512, 4, 509)])
def test_layer_step_bits(dtype, d, f, B, S, adjoint):
    wl = make(wls.ARCH_ENCODER, dtype, d=d, H=4, f=f, B=B, S=S)
    print(f"[case] groups per launch dtype={dtype} d={d} f={f} B={B} S={S} adjoint={adjoint}", flush=True)
    G = 4
    dm = DeviceModel(wl, n_layers=G, weight_std=0.05, keep_host=False)
    rng = np.random.default_rng(3)
    ins, lin = ([dev(rng.standard_normal((wl.tokens, d))) for _ in range(G)] for _ in range(2))

    def run():
        outs = [torch.full_like(x, float("nan")) for x in ins]
        mb.layer_step_batched(dm.desc, adjoint, ins, outs, dm.blocks, 0.5, lin_state=lin if adjoint else None)
        return {f"group {g}": o for g, o in enumerate(outs)}
    with_groups((1, 2, 4), run)


# (the gains and shifts of the LayerNorms are summed by a kernel of their own)
@pytest.mark.parametrize("norms", [True, False])
@pytest.mark.parametrize("arch,dtype,d,f,B,S,Sm", [
    (wls.ARCH_ENCODER, wls.DTYPE_BF16, 256, 1024, 4, 509, 0),    # token slices would pay for one or two layers only
    (wls.ARCH_CROSS, wls.DTYPE_BF16, 128, 256, 4, 515, 260),     # the row-local chains
    (wls.ARCH_CROSS, wls.DTYPE_BF16, 256, 512, 4, 515, 260),
    (wls.ARCH_ENCODER, wls.DTYPE_F32, 256, 512, 4, 509, 0)])
def test_gradient_bits(arch, dtype, d, f, B, S, Sm, norms):
    wl = wls.Workload("t", arch, d, 2, f, B, S, Sm, 4, 0.25, 1, 1, 1, dtype, 91)
    print(f"[case] groups per launch, gradients arch={arch} dtype={dtype} d={d} f={f} B={B} S={S} Sm={Sm}", flush=True)
    dm = DeviceModel(wl, weight_std=0.05, keep_host=False)
    opts = mb.mgrit_opts(wl.N, wl.h, 1, 1, 0)
    mem = wls.cross_memory(wl)
    mem = None if mem is None else dev(mem)
    Z, _ = mb.mgrit_forward(dm.desc, opts, dev(wls.initial_state(wl)), dm.blocks, memory=mem)
    lamN = dev(wls.terminal_adjoint(wl))
    floats = mb.grad_layout(dm.desc).block_bytes // 4

    def run():
        out = {}
        for lanes, cache, pair in ((1, True, False), (2, True, False), (2, False, False), (2, True, True)):
            mb.mgrit_set_lanes(lanes)            # two lanes: a serial chain hands its gradients over in batches ...
            mb.mgrit_set_adjoint_cache(cache)    # ... unless it has no cache, then they are formed layer by layer
            grads = [torch.zeros(floats, device="cuda") for _ in range(wl.N)]
            dmem = None if mem is None else torch.full_like(mem, float("nan"))
            try:
                ws = torch.empty(mb.mgrit_workspace_bytes(dm.desc, opts, 2), dtype=torch.uint8, device="cuda")
                if pair:                         # the forward solve fills the cache one layer after the other
                    Zp, _ = mb.mgrit_forward(dm.desc, opts, Z[0].clone(), dm.blocks, memory=mem, adjoint_workspace=ws,
                                             with_gradients=True)
                    assert torch.equal(Zp, Z), f"lanes={lanes}: states differ"
                lam, _ = mb.mgrit_adjoint(dm.desc, opts, Z, dm.blocks, lamN, memory=mem, workspace=ws, linearised=pair,
                                          dtheta=[g.view(torch.uint8) for g in grads], dmemory=dmem)
            finally:
                mb.mgrit_set_adjoint_cache(True)
                mb.mgrit_set_lanes(1)
            one = {"lambda": lam} if dmem is None else {"lambda": lam, "dmemory": dmem}
            for n, g in enumerate(grads):
                for name, t in mb.unpack_grad(dm.desc, g.view(torch.uint8)).items():
                    if norms == name.startswith("ln"):
                        one[f"{name} of layer {n}"] = torch.from_numpy(t)
            for name, t in one.items():
                assert torch.equal(t, out.setdefault(name, t)), f"lanes={lanes} cache={cache} pair={pair}: {name} differs"
        return out
    with_groups((1, 3, 4), run)
