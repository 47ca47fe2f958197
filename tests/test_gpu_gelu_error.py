"""Error of the bf16 path's GELU and GELU' against the exact functions, over |z| <= 12.  With the attention and W1
zero the pre-activation is the bias b1, with W2 = identity and Z = 0 a step of size 1 returns gelu(b1), and with
lambda = 1 the gradient of b1 is the number of tokens times gelu'(b1).  The polynomial's error in the distribution
function is 5.13e-5, largest where it is clamped; to it come one rounding to bf16 (2^-8 of the value) and a few
fp32 roundings."""
import numpy as np
import pytest
import torch
from scipy.special import ndtr

from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import dev
from test_gpu_param_grads import grad_blocks

pytestmark = pytest.mark.gpu

PHI_ERROR = 5.13e-5


def test_gelu_and_its_derivative_bf16():
    G, d = 8, 256
    wl = wls.Workload("gelu", wls.ARCH_ENCODER, d, 4, d, 1, 16, 0, G, 1.0, 1, 1, 1, wls.DTYPE_BF16, 5)
    desc = mb.model_desc(wl)
    z = np.linspace(-12.0, 12.0, G * d).astype(np.float32).reshape(G, d)
    blocks = []
    for g in range(G):
        p = {k: np.zeros_like(v) for k, v in wls.layer_params(wl, 0).items()}
        p["b1"], p["W2"] = z[g].reshape(p["b1"].shape), np.eye(d, dtype=np.float32)
        blocks.append(mb.pack_theta(desc, p))
    T = wl.tokens
    X = [torch.zeros(T, d, device="cuda") for _ in range(G)]
    out = [torch.full_like(x, float("nan")) for x in X]
    mb.layer_step_batched(desc, False, X, out, blocks, 1.0)
    opts = mb.mgrit_opts(G, 1.0, 1, 1, 0)
    Z, _ = mb.mgrit_forward(desc, opts, X[0], blocks)
    dtheta = grad_blocks(desc, G)
    mb.mgrit_adjoint(desc, opts, Z, blocks, dev(np.ones((T, d))), dtheta=dtheta)
    torch.cuda.synchronize()
    for g in range(G):
        x = z[g].astype(np.float64)
        cdf, pdf = ndtr(x), np.exp(-0.5 * x * x) / np.sqrt(2.0 * np.pi)
        got = out[g].cpu().numpy().astype(np.float64)
        bound = np.abs(x) * (PHI_ERROR * (1.0 + 2.0 ** -8) + 2.0 ** -22) + 2.0 ** -8 * np.abs(x * cdf)
        assert (np.abs(got - x * cdf) <= bound).all(), (np.abs(got - x * cdf) - bound).max()
        slope = mb.unpack_grad(desc, dtheta[g])["b1"].reshape(-1).astype(np.float64) / T
        ref = cdf + x * pdf
        bound = PHI_ERROR * (1.0 + 2.0 ** -8) + 2.0 ** -22 + 2.0 ** -8 * np.abs(ref)
        assert (np.abs(slope - ref) <= bound).all(), (np.abs(slope - ref) - bound).max()
