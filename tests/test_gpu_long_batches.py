"""Decode attention of batches whose K and V are read past the caches (64 MB a layer and more, the line itself included):
the step over all sequences against each sequence's own step, whose K and V lie far below the line."""
import numpy as np
import pytest

import paper_2312_04916_amd as ee
from workload import ModelShape, prompt_tokens

from common import TOL, load_gpu_model, rel_err

pytestmark = pytest.mark.gpu

LINE = (64 << 20) // (4 * 1024)  # positions of a layer of 1024 features
CASES = {
    # more than 512 (sequence, head) pairs: 4 waves; contexts of one tile and less, ragged ones, long ones
    "many": (ModelShape(2, 1024, 16, 64, 352, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5), [1, 31, 32, 33, 63] + [275] * 58),
    # fewer: 8 waves, the KV range split over two workgroups
    "few": (ModelShape(2, 1024, 8, 128, 352, 544, (1,), "bf16", 0.02, 0.3 / 8 ** 0.5), [5, 40, 700] + [1210] * 12),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("over", [-1, 0])
def test_step_over_a_batch_of_64_mb_a_layer(name, over):
    shape, lens = CASES[name]
    lens = lens + [LINE + over - sum(lens) - len(lens) - 1]  # (a step adds a position to each sequence)
    n = len(lens)
    assert lens[-1] > 0 and sum(lens) + n == LINE + over
    print(f"case: {name} {n} sequences, {sum(lens) + n} positions", flush=True)
    gm = load_gpu_model(shape, 7, gain_jitter=0.1, max_positions=2048, max_rows=64, max_seqs=n)
    logits = gm.enable_logits(n)
    cache = ee.KvCache(gm, n, LINE + 64 * (n + 1), 64, 4)
    got = []
    for groups in ([list(range(n))], [[s] for s in range(n)]):
        seqs = ee.Sequences(shape.n_layers)
        z, cf = [], []
        for s in range(n):
            cache.reset(s)
            p = prompt_tokens(shape.vocab, lens[s] + 1, 30 + s).numpy().astype(np.int32)
            ee.prefill(gm, cache, s, p[:-1], 1.0)
            seqs.start(s, p[-1])
        for g in groups:
            ro, tk, pm = seqs.rows(g)
            _, _, c = ee.decode_step(gm, cache, g, ro, tk, pm, 1.0)
            z.append(logits[: len(g)].cpu().numpy().copy())
            cf.extend(float(v) for v in c)
        got.append((np.concatenate(z), np.array(cf)))
    for s in range(n):
        assert rel_err(got[0][0][s], got[1][0][s]) <= TOL["bf16"], (s, lens[s])
    assert np.allclose(got[0][1], got[1][1], rtol=5 * TOL["bf16"])
    cache.close()
    gm.close()
