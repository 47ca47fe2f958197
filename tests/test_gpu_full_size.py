"""Parity at the benchmark's full sizes, in the launch configuration bench.py times.

The GPU runs each configuration at its full batch.  Sequences are independent through the
whole method (attention never crosses a sequence boundary), so the oracle recomputes
sampled sequences one by one -- the complete MGRIT iteration for that sequence alone -- and
every state of those sequences is compared.  The residual norm couples the batch (a sum over
all sequences): it is compared with the value the oracle computed offline for the full batch
(tests/golden/resnorms.json, written by tests/golden/make_resnorm_golden.py from the oracle
only)."""
import json
import os

import numpy as np
import pytest
import torch

from oracle import mgrit as omgrit, transformer_ode as tode
from paper_2601_09026_amd import binding as mb
from paper_2601_09026_amd import workloads as wls

from gpu_util import TOL, DeviceModel, dev, increment_tolerance, relerr, resnorm_bounds

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "resnorms.json")


def golden(name):
    """Stored oracle values of a workload; a missing entry fails the test (it is never skipped)."""
    assert os.path.exists(GOLDEN), f"{GOLDEN} is missing: python tests/golden/make_resnorm_golden.py"
    entry = json.load(open(GOLDEN)).get(name)
    assert entry is not None, f"no stored oracle residual norms for {name}: python tests/golden/make_resnorm_golden.py {name}"
    return entry


def check_norms(what, got, ref, tol, increment_norm, inc_err):
    """Stored oracle residual norms (full batch) against the library's.  `inc_err`: the relative error of the
    library's increments measured against the oracle on the sampled sequences of this same run; the allowed
    interval is resnorm_bounds' (relative tol, widened upwards by the noise that error implies, added in
    quadrature); the convergence factors follow from the norms and are printed."""
    got = np.asarray(got, np.float64)
    noise = inc_err * increment_norm
    for i, r in enumerate(ref):
        lo, hi = resnorm_bounds(r, tol, increment_norm, inc_err)
        print(f"  {what} resnorm[{i}]: {got[i]:.6g} vs oracle {r:.6g} ({(got[i] - r) / r:+.2%}; allowed {lo:.6g} .. "
              f"{hi:.6g}; noise level {noise:.3g})")
        assert lo <= got[i] <= hi, f"{what} resnorm[{i}]: {got[i]} vs oracle {r}, allowed {lo} .. {hi}"
        if i > 0:
            print(f"  {what} convergence factor {i}: {got[i] / got[i - 1]:.5g} vs oracle {r / ref[i - 1]:.5g}")


def rows_of(wl, b, seq=None):
    s = wl.seq if seq is None else seq
    return slice(b * s, (b + 1) * s)


def check_sequence(what, got, ref, base_row, tol, n_steps_of):
    """Every state of one sequence; returns the worst increment error seen (far end and middle)."""
    worst = 0.0
    for n in range(len(ref)):
        e = relerr(got[n], ref[n])
        assert e <= tol, f"{what}[{n}]: value error {e:.3e} > {tol}"
    for n in (n_steps_of["far"], n_steps_of["mid"]):
        base = ref[base_row]
        if np.linalg.norm(ref[n] - base) > 0:
            e = relerr(got[n] - base, ref[n] - base)
            bar = increment_tolerance(tol, ref[n], base, abs(n - base_row))
            print(f"  {what}[{n}] value err {relerr(got[n], ref[n]):.2e} increment err {e:.2e} (bar {bar:.2e})")
            assert e <= bar, f"{what}[{n}]: increment error {e:.3e} > {bar:.3e}"
            worst = max(worst, e)
    return worst


def run_full(name, fwd_seqs, adj_seqs, memory=None, memory_host=None, prefix=None):
    """prefix: for causal models compare only the first `prefix` tokens of each sampled sequence.
    Under the causal mask a prefix never depends on later tokens, so the oracle may run on the
    prefix alone (forward only: the adjoint flows the other way)."""
    wl = wls.named_workloads()[name]
    assert prefix is None or (wl.arch == wls.ARCH_CAUSAL and not adj_seqs)
    print(f"[case] full size {name}: B={wl.batch} S={wl.seq} d={wl.d_model} N={wl.N} cf={wl.cf} L={wl.levels} "
          f"it={wl.iters}; oracle sequences fwd={fwd_seqs} adj={adj_seqs}", flush=True)
    tol = TOL[wl.dtype]
    dm = DeviceModel(wl)
    desc = dm.desc
    opts = mb.mgrit_opts(wl.N, wl.h, wl.cf, wl.levels, wl.iters)
    Z0 = wls.initial_state(wl)
    Zg, rg = mb.mgrit_forward(desc, opts, dev(Z0), dm.blocks, memory=memory)
    torch.cuda.synchronize()
    assert mb.mgrit_step_evaluations(opts) > 0
    plen = wl.seq if prefix is None else prefix
    sh1 = tode.Shape(wl.arch, wl.d_model, wl.n_heads, 1, plen, wl.mem_seq, wl.ln_eps)
    Zg_host = {}
    einc = 0.0
    for b in fwd_seqs:
        r = slice(b * wl.seq, b * wl.seq + plen)
        mem_b = None if memory_host is None else memory_host[rows_of(wl, b, wl.mem_seq)]
        Zr, _, _ = omgrit.mgrit_forward(Z0[r], dm.host, wl.h, wl.cf, wl.levels, wl.iters, sh1, mem_b)
        got = Zg[:, r, :].cpu().numpy().astype(np.float64)
        Zg_host[b] = got
        einc = max(einc, check_sequence(f"Z(seq {b})", got, Zr, 0, tol, {"far": wl.N, "mid": wl.N // 2}))
    gold = golden(name)
    rg_host = rg.cpu().numpy()
    check_norms("forward", rg_host, gold["forward"], tol, gold["increment_norm"], einc)
    assert all(rg_host[i + 1] < rg_host[i] for i in range(wl.iters - 1)), "residual norms must decrease"
    lg = None
    if adj_seqs:
        lamN = wls.terminal_adjoint(wl)
        lg, ag = mb.mgrit_adjoint(desc, opts, Zg, dm.blocks, dev(lamN), memory=memory)
        torch.cuda.synchronize()
        sh1 = tode.Shape(wl.arch, wl.d_model, wl.n_heads, 1, wl.seq, wl.mem_seq, wl.ln_eps)
        einc = 0.0
        for b in adj_seqs:
            r = rows_of(wl, b)
            Zlin = Zg_host.get(b)
            if Zlin is None:
                Zlin = Zg[:, r, :].cpu().numpy().astype(np.float64)
            mem_b = None if memory_host is None else memory_host[rows_of(wl, b, wl.mem_seq)]
            lr, _, _ = omgrit.mgrit_adjoint(lamN[r], list(Zlin), dm.host, wl.h, wl.cf, wl.levels, wl.iters, sh1,
                                            mem_b)
            got = lg[:, r, :].cpu().numpy().astype(np.float64)
            einc = max(einc, check_sequence(f"lambda(seq {b})", got, lr, wl.N, tol, {"far": 0, "mid": wl.N // 2}))
        ag_host = ag.cpu().numpy()
        # scale of the noise: the adjoint's own total increment
        inc = float(torch.linalg.vector_norm((lg[0] - lg[wl.N]).double()))
        check_norms("adjoint", ag_host, gold["adjoint"], tol, inc, einc)
        # the pair of calls that bench.py times (the forward solve leaves most of the adjoint's
        # linearisation cache): the same results, bit for bit, at this size too
        ws = torch.empty(mb.mgrit_workspace_bytes(desc, opts, 1), dtype=torch.uint8, device="cuda")
        Z2, r2 = mb.mgrit_forward(desc, opts, dev(Z0), dm.blocks, memory=memory, adjoint_workspace=ws)
        l2, a2 = mb.mgrit_adjoint(desc, opts, Z2, dm.blocks, dev(lamN), memory=memory, workspace=ws, linearised=True)
        torch.cuda.synchronize()
        assert torch.equal(Z2, Zg) and torch.equal(r2, rg) and torch.equal(l2, lg) and torch.equal(a2, ag)
        del Z2, l2, ws
    return Zg, lg


def test_full_bert_base():
    run_full("bert_base", fwd_seqs=[3, 29], adj_seqs=[29])


def test_full_vit_small():
    run_full("vit_small", fwd_seqs=[0, 41], adj_seqs=[41])


def test_full_mt_encoder_then_decoder():
    Zg, _ = run_full("mt_encoder", fwd_seqs=[5, 60], adj_seqs=[60])
    enc_out = Zg[-1].contiguous()
    run_full("mt_decoder", fwd_seqs=[5, 60], adj_seqs=[60], memory=enc_out, memory_host=enc_out.cpu().numpy())


def test_full_gpt2_small_forward():
    run_full("gpt2_small", fwd_seqs=[6], adj_seqs=[], prefix=160)


def stored_sequence(name, b):
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", f"{name}_seq{b}.npz")
    assert os.path.exists(path), f"{path} is missing: python tests/golden/make_sequence_golden.py {name} {b}"
    return np.load(path)


def check_against_stored_sequence(wl, g, Zg, lg, tol):
    """Z_n and lambda_n of the library's full-batch run against the oracle's complete MGRIT iterate of one
    sequence, stored by tests/golden/make_sequence_golden.py: element by element at every level-0 C-point
    (they include every coarser level's C-points: the points that the relaxation, the right-hand sides, the
    coarse solves and the corrections of all levels write) on the sampled token rows, plus the
    whole-sequence norms of the increments at every point, F-points included.  Returns the worst increment
    error of Z and of lambda."""
    b, points, tokens = int(g["sequence"]), g["points"], g["tokens"]
    assert list(points) == list(range(0, wl.N + 1, wl.cf))
    seq = rows_of(wl, b)
    einc = {}
    for what, got_all, ref_pts, base_n, inc_norm, val_norm in (("Z", Zg, g["Z"], 0, g["Z_inc_norm"], g["Z_norm"]),
                                                             ("lambda", lg, g["lam"], wl.N, g["lam_inc_norm"],
                                                              g["lam_norm"])):
        got_seq = got_all[:, seq, :].cpu().numpy().astype(np.float64)          # [N+1, S, d]
        base = got_seq[base_n][tokens]                                       # start value: identical on both sides
        worst_val = worst_inc = 0.0
        for i, n in enumerate(points):
            ref = ref_pts[i].astype(np.float64)
            got = got_seq[n][tokens]
            e = relerr(got, ref)
            assert e <= tol, f"{what}[{n}]: value error {e:.3e} > {tol}"
            worst_val = max(worst_val, e)
            if n != base_n:
                ei = relerr(got - base, ref - base)
                bar = increment_tolerance(tol, ref, base, abs(int(n) - base_n))
                assert ei <= bar, f"{what}[{n}]: increment error {ei:.3e} > {bar:.3e}"
                worst_inc = max(worst_inc, ei)
        print(f"  {what}: {len(points)} C-points x {len(tokens)} tokens: worst value err {worst_val:.2e}, worst increment "
              f"err {worst_inc:.2e} (bar {tol})")
        einc[what] = worst_inc
        # whole sequence, every point (F-points too): size of the increment over the start value
        for n in range(wl.N + 1):
            if n == base_n:
                continue
            mine = np.linalg.norm(got_seq[n] - got_seq[base_n])
            floor = 4.0 * np.sqrt(abs(n - base_n)) * 2.0 ** -24 * val_norm[n]
            assert abs(mine - inc_norm[n]) <= tol * inc_norm[n] + floor, f"|{what}[{n}] - start|: {mine} vs {inc_norm[n]}"
    return einc


def test_full_gpt2_small_forward_and_adjoint_against_the_stored_oracle_sequence():
    """The deepest configuration (three levels, N = 128, causal, forward + adjoint) at its full size, as
    bench.py launches it, against the oracle's complete MGRIT iterate of one sequence, computed offline
    (the oracle needs a quarter of an hour for it): see check_against_stored_sequence.  The stored adjoint
    is linearised about the oracle's own forward iterate and the library's about its own (sec. 3.2.2): the
    two differ by the forward tolerance, which moves lambda far less than the bar.  Then the full-batch
    residual norms against the stored ones."""
    wl = wls.named_workloads()["gpt2_small"]
    tol = TOL[wl.dtype]
    print(f"[case] full size gpt2_small forward + adjoint vs stored oracle sequence", flush=True)
    g = stored_sequence("gpt2_small", 5)
    dm = DeviceModel(wl, keep_host=False)
    opts = mb.mgrit_opts(wl.N, wl.h, wl.cf, wl.levels, wl.iters)
    Z0, lamN = wls.initial_state(wl), wls.terminal_adjoint(wl)
    Zg, rg = mb.mgrit_forward(dm.desc, opts, dev(Z0), dm.blocks)
    lg, ag = mb.mgrit_adjoint(dm.desc, opts, Zg, dm.blocks, dev(lamN))
    torch.cuda.synchronize()
    assert torch.equal(Zg[0].cpu(), torch.from_numpy(Z0))
    assert torch.equal(lg[wl.N].cpu(), torch.from_numpy(lamN))
    einc = check_against_stored_sequence(wl, g, Zg, lg, tol)
    # the pair of calls that bench.py times (the forward solve leaves three quarters of the adjoint's
    # linearisation cache): the same results, bit for bit, at this size too
    ws = torch.empty(mb.mgrit_workspace_bytes(dm.desc, opts, 1), dtype=torch.uint8, device="cuda")
    Z2, r2 = mb.mgrit_forward(dm.desc, opts, dev(Z0), dm.blocks, adjoint_workspace=ws)
    l2, a2 = mb.mgrit_adjoint(dm.desc, opts, Z2, dm.blocks, dev(lamN), workspace=ws, linearised=True)
    torch.cuda.synchronize()
    assert torch.equal(Z2, Zg) and torch.equal(r2, rg) and torch.equal(l2, lg) and torch.equal(a2, ag)
    del Z2, l2, ws
    gold = golden("gpt2_small")
    check_norms("forward", rg.cpu().numpy(), gold["forward"], tol, gold["increment_norm"], einc["Z"])
    inc = float(torch.linalg.vector_norm((lg[0] - lg[wl.N]).double()))
    check_norms("adjoint", ag.cpu().numpy(), gold["adjoint"], tol, inc, einc["lambda"])
    # after the closing F-relaxation every F-point satisfies lambda_n = Psi(lambda_{n+1}; Z_n) exactly
    sh1 = tode.Shape(wl.arch, wl.d_model, wl.n_heads, 1, wl.seq, 0, wl.ln_eps)
    r = rows_of(wl, 2)
    host = {n: wls.layer_params(wl, n) for n in (wl.N - 2, 65, 1)}
    for n in (wl.N - 2, 65, 1):                 # F-points of the reversed grid (N - n not a multiple of cf)
        assert (wl.N - n) % wl.cf != 0
        ref = tode.psi(lg[n + 1, r, :].cpu().numpy(), Zg[n, r, :].cpu().numpy(), host[n], wl.h, sh1)
        got = lg[n, r, :].cpu().numpy()
        base = lg[n + 1, r, :].cpu().numpy().astype(np.float64)
        e = relerr(got - base, ref - base)
        bar = increment_tolerance(tol, ref, base, 1)
        print(f"  F-point {n}: increment err {e:.2e} (bar {bar:.2e})")
        assert e <= bar


def test_full_mc_deep_narrow_against_the_stored_oracle_sequence():
    """The deep-narrow configuration at its full size (8 sequences of 2048 tokens, one head of 128, 256
    layers, 3 levels, F-relaxation), as bench.py launches it (this is where the 256-row attention blocks and
    the row-local chains run at full length; the 2-rows-per-wavefront LayerNorm of rows this short runs at the same length
    in test_gpu_chain.py's comparisons, launch by launch).  Z_0 and lambda_N are copied exactly; Z and
    lambda at every C-point against the oracle's complete iterate of one sequence, computed offline (a
    quarter of an hour): see check_against_stored_sequence; the full-batch residual norms against the
    oracle's, stored by tests/golden/make_resnorm_golden.py (an hour and a half); and after the closing
    F-relaxation every F-point satisfies Z_{n+1} = Phi(Z_n) and lambda_n = Psi(lambda_{n+1}; Z_n),
    recomputed by the oracle on one sequence."""
    wl = wls.named_workloads()["mc_deep_narrow"]
    tol = TOL[wl.dtype]
    print(f"[case] full size {wl.name}: B={wl.batch} S={wl.seq} d={wl.d_model} N={wl.N} cf={wl.cf} L={wl.levels} "
          f"it={wl.iters} relax={wl.relax}", flush=True)
    dm = DeviceModel(wl)
    opts = mb.mgrit_opts(wl.N, wl.h, wl.cf, wl.levels, wl.iters, wl.relax)
    Z0, lamN = wls.initial_state(wl), wls.terminal_adjoint(wl)
    Zg, rg = mb.mgrit_forward(dm.desc, opts, dev(Z0), dm.blocks)
    lg, ag = mb.mgrit_adjoint(dm.desc, opts, Zg, dm.blocks, dev(lamN))
    torch.cuda.synchronize()
    assert torch.equal(Zg[0].cpu(), torch.from_numpy(Z0))
    assert torch.equal(lg[wl.N].cpu(), torch.from_numpy(lamN))
    for norms in (rg.cpu().numpy(), ag.cpu().numpy()):
        assert np.isfinite(norms).all() and norms[1] < norms[0], norms
    einc = check_against_stored_sequence(wl, stored_sequence("mc_deep_narrow", 5), Zg, lg, tol)
    # the pair of calls that bench.py times: the same results, bit for bit, at this size too
    ws = torch.empty(mb.mgrit_workspace_bytes(dm.desc, opts, 1), dtype=torch.uint8, device="cuda")
    Z2, r2 = mb.mgrit_forward(dm.desc, opts, dev(Z0), dm.blocks, adjoint_workspace=ws)
    l2, a2 = mb.mgrit_adjoint(dm.desc, opts, Z2, dm.blocks, dev(lamN), workspace=ws, linearised=True)
    torch.cuda.synchronize()
    assert torch.equal(Z2, Zg) and torch.equal(r2, rg) and torch.equal(l2, lg) and torch.equal(a2, ag)
    del Z2, l2, ws
    gold = golden("mc_deep_narrow")
    check_norms("forward", rg.cpu().numpy(), gold["forward"], tol, gold["increment_norm"], einc["Z"])
    check_norms("adjoint", ag.cpu().numpy(), gold["adjoint"], tol, gold["adjoint_increment_norm"], einc["lambda"])
    sh1 = tode.Shape(wl.arch, wl.d_model, wl.n_heads, 1, wl.seq, 0, wl.ln_eps)
    r = rows_of(wl, 2)
    for n in (0, 129, 254):                     # Z_{n+1} is an F-point: n + 1 not a multiple of cf
        assert (n + 1) % wl.cf != 0
        base = Zg[n, r, :].cpu().numpy().astype(np.float64)
        ref = tode.phi(base, dm.host[n], wl.h, sh1)
        e = relerr(Zg[n + 1, r, :].cpu().numpy() - base, ref - base)
        bar = increment_tolerance(tol, ref, base, 1)
        print(f"  Z F-point {n + 1}: increment err {e:.2e} (bar {bar:.2e})")
        assert e <= bar
    for n in (wl.N - 2, 130, 1):                # lambda_n is an F-point of the reversed grid
        assert (wl.N - n) % wl.cf != 0
        base = lg[n + 1, r, :].cpu().numpy().astype(np.float64)
        ref = tode.psi(base, Zg[n, r, :].cpu().numpy(), dm.host[n], wl.h, sh1)
        e = relerr(lg[n, r, :].cpu().numpy() - base, ref - base)
        bar = increment_tolerance(tol, ref, base, 1)
        print(f"  lambda F-point {n}: increment err {e:.2e} (bar {bar:.2e})")
        assert e <= bar
