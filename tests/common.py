"""Shared test plumbing: loads the seeded workload into the HIP library and into the oracle, and runs
the two in lockstep with the teacher-forcing rule for decisions inside the guard band."""
from __future__ import annotations

from dataclasses import dataclass, field
from typing import List, Optional

import numpy as np
import torch

import paper_2312_04916_amd as ee
from oracle import oracle as O
from workload import ModelShape, model_tensor, model_tensor_list

GUARD = 1e-2  # oracle confidence within this of the threshold, or top-2 logit gap below it: follow the GPU


def ee_config_of(shape: ModelShape, max_positions: int, **tuning) -> ee.ee_config:
    return ee.config_of_shape(shape, max_positions, **tuning)


def load_gpu_model(shape: ModelShape, seed: int = 0, gain_jitter: float = 0.0, max_positions: int = 256,
                   max_rows: int = 64, max_seqs: int = 1, **tuning) -> ee.Model:
    """Generates every tensor on the device with the workload generator and hands it to the library.
    tuning: prefill_rows, gemm_min_workgroups of ee_config."""
    m = ee.Model(ee_config_of(shape, max_positions, **tuning), max_rows, max_seqs)
    for kind, idx in model_tensor_list(shape):
        t = model_tensor(shape, kind, idx, seed, "cuda:0", gain_jitter).contiguous()
        m.set_tensor(int(kind), idx, t)
        torch.cuda.synchronize()
        del t
    return m


def cut_projections(cfg: ee.ee_config, rows: int, prompt: bool, max_rows: int, max_seqs: int) -> str:
    """Which projections of a layer are cut along K for so many rows: letters of QOGD (Q|K|V, O, gate|up, down)."""
    kernels = (ee.EE_K_QKV, ee.EE_K_OPROJ, ee.EE_K_SWIGLU, ee.EE_K_DOWN)
    return "".join(c for c, k in zip("QOGD", kernels) if ee.gemm_route(cfg, k, rows, prompt, max_rows, max_seqs)[0] == ee.EE_ROUTE_CUT)


# Relative error allowed on hidden states, logits and confidences (error over the largest reference magnitude).
# The stated bounds of the path are 1e-4 (fp32 model) and 2e-2 (bf16 model); the bf16 path keeps every activation
# as two bf16 terms and reaches a few 1e-4, so the tests hold it to 2e-3: losing an activation's second term
# (an error of 2^-9 per element) must not pass.
TOL = {"f32": 1e-4, "bf16": 2e-3}


def tol_for(shape) -> float:
    """TOL of the shape's dtype, widened for deep bf16 models: the differences in accumulation order feed through every
    further layer, so the residual stream's error grows with depth (measured: 3e-4 after 2 layers of the 7B widths,
    6e-4 after 24 layers of the 1.3B widths, 3.1e-3 after all 32 layers of the 7B shape)."""
    return TOL[shape.dtype] * (max(1.0, shape.n_layers / 8.0) if shape.dtype == "bf16" else 1.0)
# Confidences (absolute): a soft-max probability moves by up to p (1 - p) times the error of the logit differences,
# and the logits (magnitude about 16 in the workloads) are held to TOL relative to their largest: 0.25 * 2 * 2e-3 * 16.
TOL_CONF = {"f32": 1e-4, "bf16": 1.6e-2}
# Heads scored on every prompt position with the leading bf16 term of their input only (ee_config::scored_head_terms
# = 1, the default): each input element is then off by up to 2^-9 of itself, the logits by about 1e-3 of their
# largest.  Measured against the two-term heads at the 7B widths over 2048 (head, position) pairs: confidences differ
# by at most 3.8e-3 (mean 5e-4), the negative log-likelihoods by at most 2.4e-2 at a mean of 16.6, 8 arg maxes flip,
# all between candidates 1e-3 apart.  Allowed: 8e-3 on confidences, 1e-2 relative on the log-likelihoods, arg max
# inside the guard band as everywhere.
TOL_CONF_ONE_TERM = 8e-3
TOL_NLL_ONE_TERM = 1e-2


def flip_guard(dg: dict, head_terms: int) -> float:
    """Largest gap between the oracle's two best logits at which the other arg max is still accepted: the guard band,
    and for one-term scored heads 4e-3 of the best logit if that is more (each of the two logits is off by up to
    about 2e-3 of its size there)."""
    return GUARD if head_terms == 2 else max(GUARD, 4e-3 * abs(dg["top1"]))


def rel_err(a: np.ndarray, ref: np.ndarray) -> float:
    return float(np.max(np.abs(a.astype(np.float64) - ref.astype(np.float64))) / max(np.max(np.abs(ref)), 1e-30))


def kv_check(a: np.ndarray, ref: np.ndarray, dtype: str, what="", layer: int = 0) -> dict:
    """Cached K or V of layer `layer` (0-based) against the reference, element by element.

    fp32 model: |a - ref| <= 1e-4 |ref| + 1e-5 rms(ref).
    bf16 model: both sides store K and V rounded to bf16, so whatever the two differ by before the rounding moves an
    element by a whole bf16 step (at most 2^-7 of its magnitude) when it straddles a rounding boundary; the fraction
    of elements that does so is the error before rounding over the step (2^-8 .. 2^-7 of the magnitude).  In layer 0
    that error is one GEMM's accumulation order (measured: <= 0.4 % of the elements differ, nothing beyond one step);
    deeper it is what the residual stream has gathered on the way (measured at the 1.3B shape: 13 % of the elements
    at layer 12, 25 % at layer 23, up to 6e-3 rms beyond one step; 5 % at layer 1 of the 7B and 30B widths, 17 % at layer 3 of a 128-wide model).  Allowed:
    one step plus (5e-4 in layer 0, else min(4e-3 * layer, 1.6e-2)) * rms(ref) per element, and at most
    (1 % in layer 0, else min(6 % + 6 % * layer, 80 %)) of the elements differing (at layer 31 of the 7B shape half of
    them do: the residual stream's error, 3e-3 there, is then as large as the step itself).  With single-term bf16
    activations about a third of the layer-0 elements differ.
    """
    a64, r64 = a.astype(np.float64), ref.astype(np.float64)
    assert a64.shape == r64.shape and np.all(np.isfinite(a64)), what
    rms = float(np.sqrt(np.mean(r64 * r64)))
    diff = np.abs(a64 - r64)
    if dtype == "f32":
        bound = 1e-4 * np.abs(r64) + 1e-5 * rms
        frac, max_frac = 0.0, 0.0
    else:
        extra = 5e-4 if layer == 0 else min(4e-3 * layer, 1.6e-2)
        bound = 2.0 ** -7 * np.abs(r64) + extra * rms
        frac = float(np.mean(a64 != r64))
        max_frac = 0.01 if layer == 0 else min(0.06 + 0.06 * layer, 0.8)
    worst = float(np.max(diff - bound))
    stats = {"layer": layer, "max_abs": float(diff.max()), "rms": rms, "frac_differ": frac}
    assert worst <= 0.0, (what, stats, int(np.argmax(diff - bound)))
    assert frac <= max_frac, (what, stats)
    return stats


@dataclass
class LockstepReport:
    tokens: List[int] = field(default_factory=list)
    exit_layers: List[int] = field(default_factory=list)
    teacher_forced: int = 0
    forced_full: int = 0
    max_hidden_err: float = 0.0
    max_logit_err: float = 0.0
    max_conf_err: float = 0.0
    mismatches: List[str] = field(default_factory=list)


def _judge(rep: LockstepReport, step: int, diag: dict, tau: float, gpu_exits_here: bool, gpu_tok: int, is_final: bool,
           evaluated: bool) -> bool:
    """Compares one head evaluation of the oracle with what the GPU did there.  Returns True when the
    step ends at this head (following the GPU inside the guard band)."""
    if not is_final:
        if not evaluated:
            if gpu_exits_here:
                rep.mismatches.append(f"step {step}: GPU left at layer {diag['layer']} where exits are off")
            return False
        fires = diag["conf"] >= tau
        if fires != gpu_exits_here:
            if abs(diag["conf"] - tau) <= GUARD:
                rep.teacher_forced += 1
            else:
                rep.mismatches.append(f"step {step}: exit decision at layer {diag['layer']} differs "
                                      f"(oracle conf {diag['conf']:.6f}, tau {tau}, gpu exits {gpu_exits_here})")
        if not gpu_exits_here:
            return False
    if gpu_tok != diag["argmax"]:
        gap = diag["top1"] - diag["top2"]
        if gap < GUARD and gpu_tok == diag["arg2"]:
            rep.teacher_forced += 1
        else:
            rep.mismatches.append(f"step {step}: token at layer {diag['layer']} differs (oracle {diag['argmax']}, "
                                  f"gpu {gpu_tok}, top-2 gap {gap:.6f})")
    return True


def lockstep(gm: ee.Model, cache: ee.KvCache, om: O.Model, prompt, n_new: int, tau: float, max_pending: int,
             seq: int = 0, check_hidden: bool = True, logits: Optional[torch.Tensor] = None,
             max_positions: Optional[int] = None, pipeline: bool = False) -> LockstepReport:
    """Generates n_new tokens on the GPU and drives the oracle through the same decisions.  pipeline: the cache is
    in pipeline mode (no deferred lists on the GPU side; the oracle still generates by KV recomputation, the two
    methods give the same output); the hidden state is then not compared, a second stream is moving it on."""
    check_hidden = check_hidden and not pipeline
    sh = om.cfg
    L, n_exits = sh.n_layers, sh.n_exits
    rep = LockstepReport()
    st = O.State(om, max_positions or (len(prompt) + n_new + 1), max_pending)

    def check_state(step, diag):
        if check_hidden:
            rep.max_hidden_err = max(rep.max_hidden_err, rel_err(cache.read_hidden(seq), st.last_hidden()))
        if logits is not None:
            rep.max_logit_err = max(rep.max_logit_err, rel_err(logits[0].cpu().numpy(), st.last_logits()))

    # prefill: every head is evaluated on the last prompt position; the rule picks the first token
    diags = st.prefill(prompt)
    tok, ex, conf = ee.prefill(gm, cache, seq, prompt, tau)
    for i, dg in enumerate(diags):
        fin = i == n_exits
        if _judge(rep, 0, dg, tau, ex == dg["layer"], tok, fin, tau < 1.0):
            rep.max_conf_err = max(rep.max_conf_err, abs(float(conf[i]) - dg["conf"]))
            break
    rep.tokens.append(int(tok))
    rep.exit_layers.append(int(ex))
    if check_hidden:  # after prefill both hold the last prompt position at full depth
        rep.max_hidden_err = max(rep.max_hidden_err, rel_err(cache.read_hidden(seq), st.last_hidden()))

    seqs = ee.Sequences(L, pipeline=pipeline)
    seqs.start(seq, tok)
    for step in range(1, n_new):
        ro, tk, pm = seqs.rows([seq])
        cur = seqs.current[seq]
        nt, exl, cf = ee.decode_step(gm, cache, [seq], ro, tk, pm, tau)
        g_tok, g_ex = int(nt[0]), int(exl[0])
        forced = st.step_begin(cur)
        rep.forced_full += int(forced)
        evaluated = (not forced) and tau < 1.0
        while True:
            depth, dg = st.step_advance(evaluated)
            fin = depth == L
            if dg is None:
                if g_ex == depth:
                    rep.mismatches.append(f"step {step}: GPU left at layer {depth} where exits are off")
                continue
            if _judge(rep, step, dg, tau, g_ex == depth, g_tok, fin, evaluated):
                rep.max_conf_err = max(rep.max_conf_err, abs(float(cf[0]) - dg["conf"]))
                check_state(step, dg)
                break
            if fin:
                break
        st.step_commit(g_tok)
        seqs.update([seq], nt, exl)
        rep.tokens.append(g_tok)
        rep.exit_layers.append(g_ex)
        if not pipeline and cache.pending(seq) != st.n_pending():
            rep.mismatches.append(f"step {step}: pending {cache.pending(seq)} vs oracle {st.n_pending()}")
    rep.state = st
    rep.seqs = seqs
    return rep


def build_pair(shape: ModelShape, seed: int = 0, gain_jitter: float = 0.0, max_positions: int = 256,
               max_rows: int = 64, max_seqs: int = 1, **tuning):
    """(oracle model, GPU model) over the same seeded tensors: each tensor is generated once on the device
    (the generator is bit-identical on CPU and GPU), handed to the library, and copied to the host for the
    oracle."""
    from oracle.from_workload import config_of
    from workload import to_numpy

    om = O.Model(config_of(shape))
    gm = ee.Model(ee_config_of(shape, max_positions, **tuning), max_rows, max_seqs)
    for kind, idx in model_tensor_list(shape):
        t = model_tensor(shape, kind, idx, seed, "cuda:0", gain_jitter).contiguous()
        gm.set_tensor(int(kind), idx, t)
        om.set_tensor(int(kind), idx, to_numpy(t))
        torch.cuda.synchronize()
        del t
    return om, gm
