"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol the
header declares, reports a consistent parameter layout, counts evaluations like the oracle's
driver does, and rejects bad arguments before touching the device."""
import ctypes as C
import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import mgrit as omgrit
from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "mgrit.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    names = set(re.findall(r"\b(mgrit_[a-z_]+|layer_step_batched[a-z_]*)\s*\(", hdr))
    assert {"mgrit_forward", "mgrit_adjoint", "layer_step_batched", "mgrit_workspace_bytes",
            "mgrit_theta_layout", "mgrit_status_string", "layer_step_batched_static"} <= names
    L = mb.lib()
    for n in names:
        assert hasattr(L, n), n


def test_attention_kernels_do_not_spill():
    """The attention kernels on the bf16 matrix cores run at the register limit.  The kernel descriptions of
    the code objects inside the library say how many vector registers of each went to scratch memory."""
    raw = open(mb.LIB_PATH, "rb").read()
    spills = {}
    for m in re.finditer(rb"\.vgpr_spill_count", raw):
        v = raw[m.end():m.end() + 3]
        n = v[0] if v[0] < 0x80 else v[1] if v[0] == 0xcc else 256 * v[1] + v[2]
        names = re.findall(rb"\.symbol.*?(_Z[\x20-\x7e]+?)\.kd", raw[max(0, m.start() - 500):m.start()], re.S)
        spills[names[-1].decode()] = n
    attn = {k: n for k, n in spills.items() if "_mfma_kernel" in k and "attn" in k}
    assert len(attn) >= 20 and not any(attn.values()), {k: n for k, n in attn.items() if n}


@pytest.mark.parametrize("name", list(wls.named_workloads()))
def test_theta_layout_matches_the_documented_order(name):
    wl = wls.named_workloads()[name]
    desc = mb.model_desc(wl)
    lay = mb.mgrit_theta_layout(desc)
    shapes = wls.param_shapes(wl)
    prev_end = 0
    for i, pname in enumerate(mb.P_NAMES):
        if pname not in shapes:
            assert lay.offset[i] == -1
            continue
        shp = shapes[pname]
        rows, cols = (shp[0], 1) if len(shp) == 1 else shp
        assert (lay.rows[i], lay.cols[i]) == (rows, cols), pname
        eb = 4 if (len(shp) == 1 or wl.dtype == wls.DTYPE_F32) else 2
        assert lay.elem_bytes[i] == eb
        assert lay.offset[i] % 16 == 0 and lay.offset[i] >= prev_end      # in order, no overlap
        prev_end = lay.offset[i] + rows * cols * eb
    assert lay.block_bytes >= prev_end and lay.block_bytes % 256 == 0


def oracle_counts(N, cf, levels, iters, relax):
    step = omgrit.linear_propagator(-0.3, 0.1, cf)
    _, _, counts = omgrit.mgrit_solve(step, np.array([1.0]), N, cf, levels, iters, relax)
    return counts


@pytest.mark.parametrize("N,cf,levels,iters,relax", [
    (16, 4, 2, 2, 1), (64, 4, 2, 2, 1), (128, 4, 3, 2, 1), (32, 2, 2, 3, 1), (32, 4, 2, 2, 1),
    (16, 2, 4, 1, 0), (24, 3, 2, 3, 0), (16, 4, 1, 5, 1), (16, 1, 3, 2, 1)])
def test_evaluation_count_equals_oracle_minus_redundant_relaxations(N, cf, levels, iters, relax):
    """The library skips the opening F-relaxation of V-cycles 2..nu on level 0 (it would recompute
    what the previous cycle's closing F-relaxation left); everything else is counted alike."""
    got = mb.mgrit_step_evaluations(mb.mgrit_opts(N, 0.1, cf, levels, iters, relax))
    want = sum(oracle_counts(N, cf, levels, iters, "FCF" if relax else "F"))
    if levels > 1 and cf > 1 and iters > 1:
        want -= (iters - 1) * (N // cf) * (cf - 1)
    assert got == want
    if (N, cf, levels, iters, relax) == (64, 4, 2, 2, 1):
        assert got == 368            # BERT-shaped configuration: 304 fine + 64 coarse
    if (N, cf, levels, iters, relax) == (128, 4, 3, 2, 1):
        assert got == 880


@pytest.mark.parametrize("N,cf,levels,iters,relax,depth", [
    # two levels, FCF: per cycle F (cf-1) + C (1) + F (cf-1) + residual (1) + coarse right-hand side (1)
    # + N/cf coarse steps; the interpolation after a cycle is the next cycle's opening F; closing F (cf-1)
    (64, 4, 2, 2, 1, 2 * (3 + 1 + 3 + 1 + 1 + 16) + 3),
    # F-relaxation only, one cycle: F 3 + residual 1 + right-hand side 1 + 4 coarse steps + closing F 3
    (16, 4, 2, 1, 0, 12),
    # three levels: level 0 (8) + its right-hand side (1) + level 1 (8 + right-hand side 1 + 8 coarse steps
    # + interpolation 3) per cycle, closing F
    (128, 4, 3, 2, 1, 2 * (8 + 1 + 8 + 1 + 8 + 3) + 3),
    (64, 4, 1, 2, 1, 64), (16, 1, 3, 2, 1, 16)])       # serial propagation: N dependent steps
def test_dependent_depth_of_a_step(N, cf, levels, iters, relax, depth):
    """mgrit_step_depth counts the batched sweeps, each one evaluation deep (sec. 3.2: the sweeps are
    parallel over the intervals, the coarsest level is a serial chain)."""
    assert mb.mgrit_step_depth(mb.mgrit_opts(N, 0.1, cf, levels, iters, relax)) == depth
    assert mb.mgrit_step_depth(mb.mgrit_opts(10, 0.1, 4, 2, 1)) == -1


def test_ceiling_measurements_reject_bad_arguments_without_a_device():
    import ctypes as C
    out = C.c_double()
    L = mb.lib()
    assert L.mgrit_measure_mfma_ceiling(None, 1 << 20, 100, C.byref(out), None) == -1
    assert L.mgrit_measure_mfma_ceiling(C.c_void_p(4096), 1024, 100, C.byref(out), None) == -1      # scratch too small
    assert L.mgrit_measure_mfma_ceiling(C.c_void_p(4096), 1 << 20, 0, C.byref(out), None) == -1
    assert L.mgrit_measure_copy_ceiling(None, C.c_void_p(4096), 1 << 20, C.byref(out), None) == -1
    assert L.mgrit_measure_copy_ceiling(C.c_void_p(4096), C.c_void_p(8192), (1 << 20) + 8, C.byref(out), None) == -1
    assert L.mgrit_measure_copy_ceiling(C.c_void_p(4096), C.c_void_p(8192), 1 << 10, C.byref(out), None) == -1


def test_invalid_arguments_are_rejected_without_a_device():
    wl = wls.named_workloads()["tiny_encoder"]
    desc = mb.model_desc(wl)
    L = mb.lib()
    # N not divisible by cf^(levels-1)
    assert mb.mgrit_workspace_bytes(desc, mb.mgrit_opts(10, 0.1, 4, 2, 1), False) == 0
    assert mb.mgrit_step_evaluations(mb.mgrit_opts(10, 0.1, 4, 2, 1)) == -1
    assert mb.mgrit_step_evaluations(mb.mgrit_opts(16, 0.1, 0, 2, 1)) == -1
    assert mb.mgrit_step_evaluations(mb.mgrit_opts(16, 0.1, 4, 2, -1)) == -1
    ok = mb.mgrit_opts(16, 1 / 16, 4, 2, 2)
    assert mb.mgrit_workspace_bytes(desc, ok, False) > 0
    assert mb.mgrit_workspace_bytes(desc, ok, True) > mb.mgrit_workspace_bytes(desc, ok, False)
    # null pointers
    st = L.mgrit_forward(C.byref(desc), C.byref(ok), None, None, None, None, None, None, 0, None)
    assert st == -1
    # the linearising pair: no adjoint workspace, null pointers
    st = L.mgrit_forward_linearising(C.byref(desc), C.byref(ok), None, None, None, None, None, None, 0, None, 0, 0, None)
    assert st == -1
    st = L.mgrit_adjoint_linearised(C.byref(desc), C.byref(ok), None, None, None, None, None, None, None, None, None,
                                    0, None)
    assert st == -1
    bad = mb.ModelDesc(0, 65, 4, 256, 2, 32, 0, 0, 1e-5)        # d_model % n_heads != 0
    lay = mb.ThetaLayout()
    assert L.mgrit_theta_layout(C.byref(bad), C.byref(lay)) == -1
    odd = mb.ModelDesc(0, 36, 6, 72, 2, 32, 0, 0, 1e-5)         # head size 6: no kernel
    assert L.mgrit_theta_layout(C.byref(odd), C.byref(lay)) == -2
    cross_no_mem = mb.ModelDesc(2, 64, 4, 256, 2, 32, 0, 0, 1e-5)
    assert L.mgrit_theta_layout(C.byref(cross_no_mem), C.byref(lay)) == -1
    assert L.mgrit_status_string(-3) == b"workspace too small"
    dec = mb.model_desc(wls.named_workloads()["mt_decoder"])
    assert mb.mgrit_workspace_bytes(dec, mb.mgrit_opts(32, 1 / 32, 4, 2, 2), True) > \
        mb.mgrit_workspace_bytes(dec, mb.mgrit_opts(32, 1 / 32, 4, 2, 2), False) > 0


def test_parameter_gradient_workspace_and_support():
    desc = mb.model_desc(wls.named_workloads()["bert_base"])
    opts = mb.mgrit_opts(64, 1 / 64, 4, 2, 2)
    assert mb.mgrit_workspace_bytes(desc, opts, 2) > mb.mgrit_workspace_bytes(desc, opts, 1) > 0
    assert mb.mgrit_workspace_bytes(desc, opts, 3) == 0
    dec = mb.model_desc(wls.named_workloads()["mt_decoder"])
    dopts = mb.mgrit_opts(32, 1 / 32, 4, 2, 2)
    assert mb.mgrit_workspace_bytes(dec, dopts, 2) > mb.mgrit_workspace_bytes(dec, dopts, 1) > 0
    # a gradient block is the fp32 parameter block: same tensors, 4-byte entries, in order
    lay, glay = mb.mgrit_theta_layout(desc), mb.grad_layout(desc)
    for i in range(mb.P_COUNT):
        assert (lay.offset[i] < 0) == (glay.offset[i] < 0)
        if glay.offset[i] >= 0:
            assert (glay.rows[i], glay.cols[i], glay.elem_bytes[i]) == (lay.rows[i], lay.cols[i], 4)
    assert glay.block_bytes > lay.block_bytes


def test_buffered_workspace_and_argument_checks():
    desc = mb.model_desc(wls.named_workloads()["gpt2_small"])
    opts = mb.mgrit_opts(16, 1 / 16, 4, 2, 1)
    plain = mb.mgrit_workspace_bytes(desc, opts, 1)
    assert mb.mgrit_buffered_workspace_bytes(desc, opts, mb.BufferOpts(0, 0, 1.0), 1) == plain
    assert mb.mgrit_buffered_workspace_bytes(desc, opts, mb.BufferOpts(2, 2, 1.0), 1) >= plain
    assert mb.mgrit_buffered_workspace_bytes(desc, opts, mb.BufferOpts(-1, 2, 1.0), 1) == 0
    L = mb.lib()
    bad = mb.BufferOpts(1, -2, 1.0)
    assert L.mgrit_forward_buffered(C.byref(desc), C.byref(opts), C.byref(bad), None, None, None, None, None, None,
                                    0, None) == -1
    ok = mb.BufferOpts(1, 1, 1.0)
    assert L.mgrit_forward_buffered(C.byref(desc), C.byref(opts), C.byref(ok), None, None, None, None, None, None,
                                    0, None) == -1


def test_stacked_grid_workspace_and_argument_checks():
    """The stacked encoder-decoder entry points take the decoder's description: any other block type,
    a switch layer outside 1..N-1 or a missing buffer is refused before the device is touched."""
    dec = mb.model_desc(wls.named_workloads()["mt_decoder"])
    enc = mb.model_desc(wls.named_workloads()["mt_encoder"])
    opts = mb.mgrit_opts(64, 1 / 64, 4, 2, 2)
    fwd = mb.mgrit_stacked_workspace_bytes(dec, opts, 32, 0)
    adj = mb.mgrit_stacked_workspace_bytes(dec, opts, 32, 1)
    grad = mb.mgrit_stacked_workspace_bytes(dec, opts, 32, 2)
    assert 0 < fwd < adj < grad
    # both halves' work buffers are in it
    assert fwd > mb.mgrit_workspace_bytes(dec, opts, 0)
    for bad_n_enc in (0, 64, -3, 65):
        assert mb.mgrit_stacked_workspace_bytes(dec, opts, bad_n_enc, 0) == 0
    assert mb.mgrit_stacked_workspace_bytes(enc, opts, 32, 0) == 0
    assert mb.mgrit_stacked_workspace_bytes(dec, opts, 32, 3) == 0
    e = mb.encoder_desc(dec)
    assert (e.arch, e.seq, e.mem_seq, e.d_model) == (0, dec.mem_seq, 0, dec.d_model)
    L = mb.lib()
    assert L.mgrit_forward_stacked(C.byref(enc), C.byref(opts), 32, None, None, None, None, None, 0, None) == -1
    assert L.mgrit_forward_stacked(C.byref(dec), C.byref(opts), 0, None, None, None, None, None, 0, None) == -1
    assert L.mgrit_forward_stacked(C.byref(dec), C.byref(opts), 32, None, None, None, None, None, 0, None) == -1
    assert L.mgrit_adjoint_stacked(C.byref(dec), C.byref(opts), 32, None, None, None, None, None, None, None, 0,
                                   None) == -1


@pytest.mark.parametrize("B,S,Sm,levels", [(8, 16, 512, 2), (64, 64, 64, 2), (8, 16, 512, 1)])
def test_linearising_workspace_has_no_second_copy_of_the_memory(B, S, Sm, levels):
    """A decoder's keys and values of the memory for all layers (N x B Sm x 2d operands) belong to the forward
    solve's workspace, but to the adjoint's where there is one."""
    N, d = 128, 512
    desc, opts = mb.ModelDesc(2, d, 8, 2048, B, S, Sm, 1, 1e-5), mb.mgrit_opts(N, 1 / N, 4, levels, 2)
    kept = N * B * Sm * 2 * d * 2 if levels > 1 else 0
    plain, pair = mb.mgrit_workspace_bytes(desc, opts, 0), mb.mgrit_linearising_workspace_bytes(desc, opts)
    try:
        mb.mgrit_set_adjoint_cache(False)
        least = mb.mgrit_workspace_bytes(desc, opts, 0)
    finally:
        mb.mgrit_set_adjoint_cache(True)
    assert 0 < pair <= least and pair == plain - kept, (plain, pair, least)
    enc = mb.encoder_desc(desc)
    assert mb.mgrit_linearising_workspace_bytes(enc, opts) == mb.mgrit_workspace_bytes(enc, opts, 0)
    assert mb.mgrit_linearising_workspace_bytes(desc, mb.mgrit_opts(10, 0.1, 4, 2, 1)) == 0


@pytest.mark.parametrize("dtype,d,tokens,mode", [(1, 128, 64, 1), (1, 128, 64, 2), (0, 64, 64, 1), (0, 64, 64, 2)])
def test_recompute_mode_keeps_small_chunks(dtype, d, tokens, mode):
    """Without the adjoint cache the workspace holds the internals of one launch chunk per lane, so many layers of
    few tokens do not share a launch there: no more memory than with chunks of 6 (bf16) or 4 (fp32)."""
    desc = mb.ModelDesc(0, d, 2, 4 * d, 1, tokens, 0, dtype, 1e-5)
    dec = mb.ModelDesc(2, d, 2, 4 * d, 1, tokens // 2, tokens // 2, dtype, 1e-5)
    opts = mb.mgrit_opts(128, 1 / 128, 4, 2, 2)
    size = lambda: (mb.mgrit_workspace_bytes(desc, opts, mode), mb.mgrit_stacked_workspace_bytes(dec, opts, 64, mode))
    cached = size()
    try:
        mb.mgrit_set_adjoint_cache(False)
        auto = size()
        mb.mgrit_set_max_groups_per_launch(6 if dtype else 4)
        bound = size()
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
        mb.mgrit_set_adjoint_cache(True)
    assert all(a <= b < c for a, b, c in zip(auto, bound, cached)), (auto, bound, cached)


def test_default_groups_per_launch_follow_the_tile_model():
    """Without a caller's choice the launch chunk of the benchmark models comes from the GEMM tile model: 3..6 groups
    for bf16 (5 at d = 768, where five groups of 4096 tokens fill one round of 256x256 tiles for the d-wide outputs),
    and the workspace is sized for it.  The tiny fp32 model is one of few tokens: its sweeps of four go into one launch,
    wider ones up to 64 at a time."""
    L = mb.lib()
    for name, wl in wls.named_workloads().items():
        desc = mb.model_desc(wl)
        g = L.mgrit_default_groups_per_launch(C.byref(desc), wl.N // wl.cf)
        assert (g == 4) if wl.dtype == wls.DTYPE_F32 else (3 <= g <= 6), (name, g)
    tiny = mb.model_desc(wls.named_workloads()["tiny_encoder"])
    assert [L.mgrit_default_groups_per_launch(C.byref(tiny), n) for n in (1, 4, 9, 100)] == [4, 4, 9, 64]
    bert = mb.model_desc(wls.named_workloads()["bert_base"])
    assert L.mgrit_default_groups_per_launch(C.byref(bert), 16) == 5
    opts = mb.mgrit_opts(64, 1 / 64, 4, 2, 2)
    auto = mb.mgrit_workspace_bytes(bert, opts, 0)
    try:
        mb.mgrit_set_max_groups_per_launch(5)
        assert mb.mgrit_workspace_bytes(bert, opts, 0) == auto
        mb.mgrit_set_max_groups_per_launch(3)
        assert mb.mgrit_workspace_bytes(bert, opts, 0) < auto
    finally:
        mb.mgrit_set_max_groups_per_launch(0)
    bad = mb.ModelDesc(0, 770, 12, 3072, 32, 128, 0, 1, 1e-5)
    assert L.mgrit_default_groups_per_launch(C.byref(bad), 16) == 0


NO_MEMORY = """
import ctypes as C, resource, sys
L = C.CDLL(sys.argv[1])
n = 1 << 22
ptrs = (C.c_void_p * n)(*[256] * n)
desc = (C.c_int32 * 9)(0, 64, 4, 256, 1, 8, 0, 0, 0x3727c5ac)             # an fp32 encoder, ln_eps = 1e-5
fn = L.layer_step_batched
fn.argtypes = [C.c_void_p, C.c_int, C.c_int] + [C.c_void_p] * 6 + [C.c_float, C.c_void_p, C.c_size_t, C.c_void_p]
def call(adjoint, n):
    return fn(desc, adjoint, n, ptrs, ptrs, ptrs, ptrs if adjoint else None, None, None, 0.5, 256, 1 << 60, None)
first = call(0, 1)                                                     # whatever the runtime allocates, now
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (64 << 20), resource.RLIM_INFINITY))
print(first, call(0, n), call(1, n))
"""


@pytest.mark.skipif(torch.cuda.is_available(), reason="addresses that must not reach a GPU")
def test_layer_step_needs_no_host_memory_for_its_tables():
    """Four million layers with 64 MB of address space left: without a device the call ends in MGRIT_HIP_ERROR, not in an
    allocation that fails inside the library (an exception has no way out of a C function)."""
    run = subprocess.run([sys.executable, "-c", NO_MEMORY, mb.LIB_PATH], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, (run.returncode, run.stderr[-500:])
    assert run.stdout.split() == ["-4"] * 3, run.stdout


def test_workspace_grows_with_groups_and_levels():
    desc = mb.model_desc(wls.named_workloads()["bert_base"])
    a = mb.mgrit_layer_step_workspace_bytes(desc, False, 1)
    b = mb.mgrit_layer_step_workspace_bytes(desc, False, 4)
    assert 0 < a < b
    two = mb.mgrit_workspace_bytes(desc, mb.mgrit_opts(64, 1 / 64, 4, 2, 2), False)
    three = mb.mgrit_workspace_bytes(desc, mb.mgrit_opts(64, 1 / 64, 4, 3, 2), False)
    assert three > two
