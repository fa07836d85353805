"""GPU parity of decode steps by the number of rows they carry, against the CPU oracle's cache-free forward: every row
count at which the projections change kernel, row tile or pass (3 | 4 staged / packed rows, 16 | 17, 32 | 33, 64 | 66
rows), on widths that leave ragged column groups, with one and with several column tiles per workgroup."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2312_04916_amd as ee
from oracle.from_workload import build_model
from workload import ModelShape, model_tensor, model_tensor_list, prompt_tokens

from common import TOL, cut_projections, ee_config_of, kv_check, load_gpu_model, rel_err
from test_gpu_prefill import check_prefill

pytestmark = pytest.mark.gpu

SHAPES = {
    "d128": ModelShape(3, 128, 4, 32, 352, 1056, (1,), "bf16", 0.02, 0.3),
    "d192": ModelShape(2, 192, 3, 64, 224, 544, (1,), "bf16", 0.02, 0.3),
    # wide enough that projections are cut over K (CUT_STEPS): 65 k-tiles and 17 panels of which the last holds one pair, 89
    # k-tiles, 9 panels of which the last holds four tiles
    "d1024": ModelShape(2, 1024, 8, 128, 2080, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5),
    "d1024w": ModelShape(2, 1024, 8, 128, 2848, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5),
    "d3072": ModelShape(2, 3072, 24, 128, 1056, 544, (1,), "bf16", 0.02, 0.3 / 24 ** 0.5),
    "d5632": ModelShape(2, 5632, 44, 128, 352, 544, (1,), "bf16", 0.02, 0.3 / 44 ** 0.5),
}
# The projections of a step that are cut, by rows (the rule is host arithmetic: test_routes.py checks this table without a
# GPU): with 64-row tiles each of the four in one shape or another, with 128-row tiles one and two of those per panel.
STEP_LIMITS = dict(max_rows=160, max_seqs=4)
CUT_STEPS = {
    "d1024": {33: "", 64: "", 66: "D", 128: "QOGD", 129: "QOGD"},
    "d1024w": {33: "D", 64: "D"},
    "d3072": {33: "OG", 64: "OG"},
    "d5632": {33: "QOG"},
}
PROMPT_SHAPES = {
    "d1024": SHAPES["d1024"],
    "d1536": ModelShape(2, 1536, 12, 128, 2080, 544, (1,), "bf16", 0.02, 0.3 / 12 ** 0.5),
}
CUT_PROMPTS = {  # (tokens, prefill_rows): the projections that are cut in each pass
    "d1024": {(33, 0): ["QOGD"], (64, 0): ["QOGD"], (65, 0): ["QOGD"], (128, 0): ["QOGD"], (129, 0): ["QOD"], (200, 128): ["QOGD", "QOGD"]},
    "d1536": {(129, 0): ["QOGD"], (200, 0): ["QOGD"], (256, 0): ["QOGD"]},
}


@pytest.mark.parametrize("name,min_wgs", [("d128", 0), ("d192", 0), ("d128", 16), ("d192", 6), ("d1024", 0), ("d1024w", 0), ("d3072", 0), ("d5632", 0)])
def test_full_depth_step_over_a_given_number_of_rows(name, min_wgs):
    shape = SHAPES[name]
    om = build_model(shape, 5, gain_jitter=0.1)
    gm = load_gpu_model(shape, 5, gain_jitter=0.1, max_positions=128, gemm_min_workgroups=min_wgs, **STEP_LIMITS)
    n_seq, cap = 4, 40
    fed = [prompt_tokens(shape.vocab, 80, 60 + s).numpy().astype(np.int32) for s in range(n_seq)]
    for rows in CUT_STEPS.get(name, (1, 2, 3, 4, 5, 16, 17, 32, 33, 64, 66, 80, 81)):
        print(f"case: {name} tiles {min_wgs} rows {rows}", flush=True)
        ids = list(range(min(n_seq, rows)))
        lens = [7 + 5 * s for s in ids]
        pend = [(rows - len(ids)) // len(ids) + (1 if s < (rows - len(ids)) % len(ids) else 0) for s in ids]
        cache = ee.KvCache(gm, n_seq, 4 * 128, 32, cap)
        seqs = ee.Sequences(shape.n_layers)
        for s in ids:
            ee.prefill(gm, cache, s, fed[s][: lens[s]], 1.0)
            seqs.start(s, fed[s][lens[s]])
            for k in range(pend[s]):  # threshold 0: every token leaves at the first exit and stays deferred
                ro, tk, pm = seqs.rows([s])
                _, ex, _ = ee.decode_step(gm, cache, [s], ro, tk, pm, 0.0)
                assert int(ex[0]) == 1
                seqs.update([s], [fed[s][lens[s] + k + 1]], ex)
            assert cache.pending(s) == pend[s]
        ro, tk, pm = seqs.rows(ids)
        assert len(tk) == rows
        nt, ex, _ = ee.decode_step(gm, cache, ids, ro, tk, pm, 1.0)
        for s in ids:
            n = lens[s] + pend[s] + 1
            assert int(ex[s]) == shape.n_layers and cache.pending(s) == 0
            hid, ko, vo = om.forward_sequence(fed[s][:n])
            err = rel_err(cache.read_hidden(s), hid[shape.n_layers][n - 1])
            assert err <= TOL["bf16"], (rows, s, err)
            _, dg = om.head_row(len(shape.exit_layers), hid[shape.n_layers][n - 1])
            assert int(nt[s]) == dg["argmax"] or (dg["top1"] - dg["top2"] < 1e-2 and int(nt[s]) == dg["arg2"])
            for l in range(shape.n_layers):
                k, v = cache.read(s, l, 0, n)
                kv_check(k, ko[l], "bf16", "K", l), kv_check(v, vo[l], "bf16", "V", l)
        cache.close()
    gm.close()


@pytest.mark.parametrize("name,n,rows_env", [(name, *case) for name, cases in CUT_PROMPTS.items() for case in cases])
def test_short_prompts_whose_gemms_are_cut_over_the_contraction(name, n, rows_env):
    """Prompts around the row tiles of the prompt phase (64, 128 rows, one and two tiles, a second pass), at widths at which
    the four GEMMs are cut over K as CUT_PROMPTS says: at 1024 wide all of them up to one row tile, at 1536 with two."""
    print(f"case: cut prompt {name} n={n} rows_env={rows_env}", flush=True)
    check_prefill(PROMPT_SHAPES[name], n, 4, rows_env=rows_env, scored=False)


def test_head_over_more_than_half_a_batch_of_rows():
    """A step of 33 and of 64 sequences with a vocabulary of 129 column panels of 256 (the last one ragged): logits, arg max
    and confidence of the final head as each sequence gets them in a step of its own."""
    shape = ModelShape(2, 128, 4, 32, 352, 128 * 256 + 96, (1,), "bf16", 0.02, 0.3)
    gm = load_gpu_model(shape, 6, gain_jitter=0.1, max_positions=64, max_rows=64, max_seqs=64)
    logits = gm.enable_logits(64)
    for n in (33, 64):
        print(f"case: head over {n} rows", flush=True)
        ids = list(range(n))
        got = []
        for groups in ([ids], [[s] for s in ids]):
            cache = ee.KvCache(gm, 64, 64 * 64, 32, 4)
            seqs = ee.Sequences(shape.n_layers)
            z, tok, cf = [], [], []
            for s in ids:
                p = prompt_tokens(shape.vocab, 3 + s % 5, 90 + s).numpy()
                t, _, _ = ee.prefill(gm, cache, s, p, 1.0)
                seqs.start(s, t)
            for g in groups:
                ro, tk, pm = seqs.rows(g)
                nt, ex, c = ee.decode_step(gm, cache, g, ro, tk, pm, 1.0)
                z.append(logits[: len(g)].cpu().numpy().copy())
                tok.extend(int(t) for t in nt)
                cf.extend(float(v) for v in c)
            cache.close()
            got.append((np.concatenate(z), tok, cf))
        (za, ta, ca), (zb, tb, cb) = got
        assert rel_err(za, zb) <= TOL["bf16"]
        for s in ids:
            top = np.sort(zb[s])[-2:]
            assert ta[s] == int(za[s].argmax()) and (ta[s] == tb[s] or top[1] - top[0] < 1e-2), s
            want = 1.0 / np.exp(za[s].astype(np.float64) - za[s].max()).sum()
            assert abs(ca[s] - want) <= 1e-5 * want, (s, ca[s], want)  # 32-bit exponentials and sums over 32864 terms
    gm.close()


def test_head_whose_logits_are_all_minus_infinity():
    """Every logit of every row overflows to -inf: the token is the lowest index whichever kernel the head runs in (32 rows:
    16-column tiles, 33: 256-column panels), and can be fed back."""
    shape = ModelShape(2, 128, 4, 32, 352, 128 * 256 + 96, (1,), "bf16", 0.02, 0.3)
    gm = load_gpu_model(shape, 6, max_positions=64, max_rows=64, max_seqs=33)
    bf16 = dict(dtype=torch.bfloat16, device="cuda:0")
    for l in range(shape.n_layers):  # the layers add nothing: x stays the embedding row
        gm.set_tensor(ee.EE_T_WO, l, torch.zeros(128, 128, **bf16))
        gm.set_tensor(ee.EE_T_WD, l, torch.zeros(128, 352, **bf16))
    embed = torch.zeros(shape.vocab, 128, **bf16)
    embed[:, 0] = 4.0
    head = torch.zeros(shape.vocab, 128, **bf16)
    head[:, 0] = -3.0e38  # times 4 times the RMS scale: past the largest float32
    gm.set_tensor(ee.EE_T_EMBED, 0, embed)
    gm.set_tensor(ee.EE_T_FINAL_HEAD, 0, head)
    logits = gm.enable_logits(33)
    for n in (32, 33):
        print(f"case: all logits -inf over {n} rows", flush=True)
        cache = ee.KvCache(gm, 33, 33 * 64, 32, 4)
        seqs = ee.Sequences(shape.n_layers)
        for s in range(n):
            seqs.start(s, ee.prefill(gm, cache, s, [1, 2, 3], 1.0)[0])
        for _ in range(2):
            ro, tk, pm = seqs.rows(list(range(n)))
            nt, ex, _ = ee.decode_step(gm, cache, list(range(n)), ro, tk, pm, 1.0)
            assert bool(torch.isneginf(logits[:n]).all())
            assert list(nt) == [0] * n
            seqs.update(list(range(n)), nt, ex)
        cache.close()
    gm.close()


@pytest.mark.parametrize("missing", ["none", "some", "all"])
def test_workspace_without_scratch_for_partial_sums(missing):
    """A workspace that lacks some or all of the scratch at its end (the size that the library asked for before it cut GEMMs
    along K) is accepted, half of it is not, and a prompt gives the same K and V."""
    shape = ModelShape(2, 1024, 8, 128, 2080, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5)
    without = 18149376  # of this model with 64 rows and one sequence
    cfg = ee_config_of(shape, 256)
    full = C.c_size_t()
    assert ee.lib().ee_model_bytes(C.byref(cfg), 64, 1, None, C.byref(full)) == 0 and full.value > without
    n_bytes = {"none": full.value, "some": (without + full.value) // 2, "all": without}[missing]
    print(f"case: workspace of {n_bytes} of {full.value} bytes", flush=True)
    gm = load_gpu_model(shape, 5, gain_jitter=0.1, max_positions=256)
    # the same tensors in a model over a workspace of n_bytes, whose prompts are compared
    weights, workspace = torch.empty_like(gm.weights), torch.empty(n_bytes, dtype=torch.uint8, device="cuda:0")
    create = lambda n, h: ee.lib().ee_model_create(  # noqa: E731
        C.byref(cfg), weights.data_ptr(), gm.weight_bytes, workspace.data_ptr(), n, 64, 1, None, C.byref(h))
    if missing == "all":
        assert create(without // 2, C.c_void_p()) == -2
    h = C.c_void_p()
    assert create(n_bytes, h) == 0
    ee.lib().ee_model_free(gm.h)
    gm.h, gm.weights, gm.workspace = h, weights, workspace
    for kind, idx in model_tensor_list(shape):
        gm.set_tensor(int(kind), idx, model_tensor(shape, kind, idx, 5, "cuda:0", 0.1).contiguous())
    torch.cuda.synchronize()
    om = build_model(shape, 5, gain_jitter=0.1)
    cache = ee.KvCache(gm, 1, 256, 32, 4)
    for n in (33, 100, 200):
        cache.reset(0)
        prompt = prompt_tokens(shape.vocab, n, 3).numpy().astype(np.int32)
        ee.prefill(gm, cache, 0, prompt, 1.0)
        hid, ko, vo = om.forward_sequence(prompt)
        assert rel_err(cache.read_hidden(0), hid[shape.n_layers][n - 1]) <= TOL["bf16"]
        for l in range(shape.n_layers):
            k, v = cache.read(0, l, 0, n)
            kv_check(k, ko[l], "bf16", "K", l), kv_check(v, vo[l], "bf16", "V", l)
    cache.close()
    gm.close()


def many_sequences(gm, cache, shape, n, fed, n_first):
    seqs = ee.Sequences(shape.n_layers)
    for s in range(n):
        ee.prefill(gm, cache, s, fed[s][:n_first], 1.0)
        seqs.start(s, fed[s][n_first])
    return seqs


def test_cut_projections_in_the_static_workspace():
    """Steps of 40 sequences whose down projection is cut along K: the scratch lies in the step's workspace, so the library's
    own static one gives the same bits."""
    shape, n = SHAPES["d1024w"], 40
    gm = load_gpu_model(shape, 5, gain_jitter=0.1, max_positions=64, max_rows=64, max_seqs=n)
    assert cut_projections(gm.cfg, n, False, 64, n) == "D"
    fed = [prompt_tokens(shape.vocab, 16, 200 + s).numpy().astype(np.int32) for s in range(n)]
    got = []
    for static in (False, True):
        print(f"case: 40 sequences, static workspace {static}", flush=True)
        cache = ee.KvCache(gm, n, n * 64, 32, 4)
        seqs = many_sequences(gm, cache, shape, n, fed, 5)
        out = []
        for k in range(3):
            ro, tk, pm = seqs.rows(list(range(n)))
            nt, ex, cf = ee.decode_step(gm, cache, list(range(n)), ro, tk, pm, 1.0, static_workspace=static)
            out += [nt.copy(), cf.copy()]
            seqs.update(list(range(n)), [f[6 + k] for f in fed], ex)
        for s in (0, 17, n - 1):
            out.append(cache.read_hidden(s))
            out += [t for l in range(shape.n_layers) for t in cache.read(s, l, 0, 8)]
        got.append(out)
        cache.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    gm.close()


def test_cut_projections_in_a_pipeline_fill():
    """Pipeline mode, 40 sequences, every token leaves at the first exit: its pass through the layers above runs on the fill
    stream in that stream's workspace, with the down projections cut along K.  Their K and V against the oracle's (the K
    and V of layer 2 are formed behind layer 1's down projection)."""
    shape = ModelShape(3, 1024, 8, 128, 2848, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5)
    n, steps = 40, 4
    om = build_model(shape, 5, gain_jitter=0.1)
    gm = load_gpu_model(shape, 5, gain_jitter=0.1, max_positions=64, max_rows=64, max_seqs=n)
    assert cut_projections(gm.cfg, n, False, 64, n) == "D"
    fed = [prompt_tokens(shape.vocab, 16, 300 + s).numpy().astype(np.int32) for s in range(n)]
    print("case: pipeline fills of 40 rows", flush=True)
    cache = ee.KvCache(gm, n, n * 64, 32, 15)
    cache.set_pipeline(True)
    seqs = many_sequences(gm, cache, shape, n, fed, 5)
    seqs.pipeline = True
    for k in range(steps):
        ro, tk, pm = seqs.rows(list(range(n)))
        _, ex, _ = ee.decode_step(gm, cache, list(range(n)), ro, tk, pm, 0.0)
        assert list(ex) == [1] * n
        seqs.update(list(range(n)), [f[6 + k] for f in fed], ex)
    cache.flush(list(range(n)))
    for s in (0, 17, n - 1):
        _, ko, vo = om.forward_sequence(fed[s][: 5 + steps])
        for l in range(shape.n_layers):
            assert cache.filled(s, l) == 5 + steps
            k, v = cache.read(s, l, 0, 5 + steps)
            kv_check(k, ko[l], "bf16", "K", l), kv_check(v, vo[l], "bf16", "V", l)
    cache.close()
    gm.close()


@pytest.mark.parametrize("structure", [dict(exit_norm=False), dict(tie_embeddings=True), dict(exit_mlp=True), dict(exit_layer=True)],
                         ids=lambda s: next(iter(s)))
def test_head_in_panels_behind_every_exit_structure(structure):
    """The heads of 33 sequences in 256-column panels, at an exit of each structure and at the end: logits, arg max and
    confidence as each sequence gets them in a step of its own."""
    shape = ModelShape(2, 128, 4, 32, 352, 128 * 256 + 96, (1,), "bf16", 0.02, 0.3, **structure)
    n = 33
    gm = load_gpu_model(shape, 6, gain_jitter=0.1, max_positions=64, max_rows=64, max_seqs=n)
    assert ee.gemm_route(gm.cfg, ee.EE_K_HEAD, n, False, 64, n)[0] == ee.EE_ROUTE_PANELS
    logits = gm.enable_logits(n)
    ids = list(range(n))
    fed = [prompt_tokens(shape.vocab, 16, 400 + s).numpy().astype(np.int32) for s in ids]
    for tau, leaves_at in ((0.0, 1), (1.0, 2)):
        print(f"case: panels behind {structure}, threshold {tau}", flush=True)
        got = []
        for groups in ([ids], [[s] for s in ids]):
            cache = ee.KvCache(gm, n, n * 64, 32, 4)
            seqs = many_sequences(gm, cache, shape, n, fed, 5)
            z, tok, cf = [], [], []
            for g in groups:
                ro, tk, pm = seqs.rows(g)
                nt, ex, c = ee.decode_step(gm, cache, g, ro, tk, pm, tau)
                assert list(ex) == [leaves_at] * len(g)
                torch.cuda.synchronize()
                z.append(logits[: len(g)].cpu().numpy().copy())
                tok.extend(int(t) for t in nt)
                cf.extend(float(v) for v in c)
            cache.close()
            got.append((np.concatenate(z), tok, cf))
        (za, ta, ca), (zb, tb, cb) = got
        assert rel_err(za, zb) <= TOL["bf16"]
        for s in ids:
            top = np.sort(zb[s])[-2:]
            assert ta[s] == int(za[s].argmax()) and (ta[s] == tb[s] or top[1] - top[0] < 1e-2), s
            want = 1.0 / np.exp(za[s].astype(np.float64) - za[s].max()).sum()
            assert abs(ca[s] - want) <= 1e-5 * want, (s, ca[s], want)  # 32-bit exponentials and sums over 32864 terms
    gm.close()
