"""Decode attention of batches whose K and V are read past the caches (384 MB and more over the layers of a step, the line itself
included): one row per sequence, several, and sequences with two query tiles among them.  The step over all sequences against the
oracle (the short ones) and against each sequence's own step, whose K and V lie far below the line (all of them)."""
import numpy as np
import pytest

import paper_2312_04916_amd as ee
from oracle.from_workload import build_model
from workload import ModelShape, prompt_tokens

from common import TOL, load_gpu_model, rel_err

pytestmark = pytest.mark.gpu

LAYERS = 8
LINE = (384 << 20) // (LAYERS * 4 * 1024)  # positions, 1024 wide


def shape_of(head_dim, exits=(1,)):
    return ModelShape(LAYERS, 1024, 1024 // head_dim, head_dim, 352, 544, exits, "bf16", 0.02, 0.3 / 8 ** 0.5)


CASES = {  # head size, contexts that the step ends with (one more sequence brings them to the line), rows of each in that step
    # more than 512 (query tile, head) pairs: 4 waves; contexts of one tile and less, ragged ones, long ones
    "many": (64, [2, 32, 33, 34, 64] + [276] * 43, [1] * 48),
    "many_head32": (32, [2, 32, 33, 34, 64] + [276] * 43, [1] * 48),
    # fewer: 8 waves, the KV range split over two workgroups
    "few": (128, [6, 41, 701] + [1211] * 9, [1] * 12),
    "few_head32": (32, [6, 41, 701] + [1211] * 9, [1] * 12),
    # deferred tokens: up to 16 rows are one query tile, 17 and more two, which read what is a small part of all
    "rows": (128, [18, 34, 50, 70, 96] + [1211] * 9, [4, 16, 17, 20, 33] + [1, 2, 7] * 3),
    "rows_head64": (64, [18, 34, 50, 70, 96] + [1211] * 9, [4, 16, 17, 20, 33] + [1, 2, 7] * 3),
    "rows_head32": (32, [18, 34, 50, 70, 96] + [1211] * 9, [4, 16, 17, 20, 33] + [1, 2, 7] * 3),
}


def long_batch(name, over):
    """(shape, contexts, rows) of a step whose K and V lie `over` positions past the line."""
    head_dim, contexts, rows = CASES[name]
    return shape_of(head_dim), contexts + [LINE + over - sum(contexts)], rows + [1]


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("over", [-1, 0])
def test_step_over_a_batch_around_the_line(name, over):
    shape, contexts, rows = long_batch(name, over)
    n, L = len(contexts), shape.n_layers
    assert sum(contexts) == LINE + over and min(c - r for c, r in zip(contexts, rows)) > 0
    print(f"case: {name} {n} sequences, {sum(contexts)} positions, {sum(rows)} rows", flush=True)
    gm = load_gpu_model(shape, 7, gain_jitter=0.1, max_positions=2048, max_rows=256, max_seqs=n)
    logits = gm.enable_logits(n)
    cache = ee.KvCache(gm, n, LINE + 64 * (n + 1), 64, 40)
    fed = [prompt_tokens(shape.vocab, contexts[s], 30 + s).numpy().astype(np.int32) for s in range(n)]
    got, last = [], {}
    short = [s for s in range(n) if contexts[s] <= 96]
    for groups in ([list(range(n))], [[s] for s in range(n)]):
        seqs = ee.Sequences(L)
        z, cf = [], []
        for s in range(n):
            cache.reset(s)
            first = contexts[s] - rows[s]
            ee.prefill(gm, cache, s, fed[s][:first], 1.0)
            seqs.start(s, fed[s][first])
            for k in range(rows[s] - 1):  # every token leaves at the first exit and stays deferred
                ro, tk, pm = seqs.rows([s])
                _, ex, _ = ee.decode_step(gm, cache, [s], ro, tk, pm, 0.0)
                seqs.update([s], [fed[s][first + k + 1]], ex)
            assert cache.pending(s) == rows[s] - 1
        for g in groups:
            ro, tk, pm = seqs.rows(g)
            _, ex, c = ee.decode_step(gm, cache, g, ro, tk, pm, 1.0)
            assert list(ex) == [L] * len(g)
            z.append(logits[: len(g)].cpu().numpy().copy())
            cf.extend(float(v) for v in c)
        if len(groups) == 1:
            last = {s: cache.read_hidden(s) for s in short}
        got.append((np.concatenate(z), np.array(cf)))
    for s in range(n):
        assert rel_err(got[0][0][s], got[1][0][s]) <= TOL["bf16"], (s, contexts[s])
    assert np.allclose(got[0][1], got[1][1], rtol=5 * TOL["bf16"])
    om = build_model(shape, 7, gain_jitter=0.1)
    for s in short:
        hid, _, _ = om.forward_sequence(fed[s])
        assert rel_err(last[s], hid[L][-1]) <= TOL["bf16"], (s, contexts[s], rows[s])
    cache.close()
    gm.close()
