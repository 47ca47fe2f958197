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
