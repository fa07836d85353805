"""GPU parity of decode steps by the number of rows they carry, against the CPU oracle's cache-free forward: every row
count at which the projections change kernel, row tile or pass (3 | 4 staged / packed rows, 16 | 17, 32 | 33, 64 | 66
rows), on widths that leave ragged column groups, with one and with several column tiles per workgroup."""
import numpy as np
import pytest

import paper_2312_04916_amd as ee
from oracle.from_workload import build_model
from workload import ModelShape, prompt_tokens

from common import TOL, kv_check, load_gpu_model, rel_err
from test_gpu_prefill import check_prefill

pytestmark = pytest.mark.gpu

SHAPES = {
    "d128": ModelShape(3, 128, 4, 32, 352, 1056, (1,), "bf16", 0.02, 0.3),
    "d192": ModelShape(2, 192, 3, 64, 224, 544, (1,), "bf16", 0.02, 0.3),
}


@pytest.mark.parametrize("name,min_wgs", [("d128", 0), ("d192", 0), ("d128", 16), ("d192", 6)])
def test_full_depth_step_over_a_given_number_of_rows(name, min_wgs):
    shape = SHAPES[name]
    om = build_model(shape, 5, gain_jitter=0.1)
    gm = load_gpu_model(shape, 5, gain_jitter=0.1, max_positions=128, max_rows=128, max_seqs=4, gemm_min_workgroups=min_wgs)
    n_seq, cap = 4, 40
    fed = [prompt_tokens(shape.vocab, 80, 60 + s).numpy().astype(np.int32) for s in range(n_seq)]
    for rows in (1, 2, 3, 4, 5, 16, 17, 32, 33, 64, 66, 80, 81):
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


@pytest.mark.parametrize("n,rows_env", [(33, 0), (64, 0), (65, 0), (128, 0), (129, 0), (200, 128)])
def test_short_prompts_whose_gemms_are_cut_over_the_contraction(n, rows_env):
    """Prompts around the row tiles of the prompt phase (64, 128 rows, one and two tiles, a second pass), on a width at
    which all four GEMMs are cut over K: 32 and 65 k-tiles, 17 column panels of which the last holds a single pair."""
    print(f"case: cut prompt n={n} rows_env={rows_env}", flush=True)
    shape = ModelShape(2, 1024, 8, 128, 2080, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5)
    check_prefill(shape, n, 4, rows_env=rows_env, scored=False)
