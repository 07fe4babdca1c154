"""The attention work list for batches of every shape of it: equal lengths,
lengths around a bin (32 keys) and a query block (128), empty records, more
records than threads (1024), a length limit above 1024 bins.  A record's hidden
state does not depend on its batch, so every batch equals, bit for bit, the
same records a few at a time (tolerance zero)."""
from __future__ import annotations

import numpy as np
import pytest

from synth.configs import ModelConfig
from tests.gpu_common import make_model, say

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 255, 256, 257, 511, 512]


def _hidden(pl, ids, lengths):
    import torch
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)

    class Batch:
        B, h_cu, T = len(lengths), cu, int(cu[-1])
    db = Batch()
    db.ids, db.cu = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda()
    return pl.hidden(db, 1)[:db.T].cpu().numpy()


@pytest.mark.parametrize("max_pos,precision", [(512, "bf16"), (512, "fp32"), (8192, "bf16"), (70000, "bf16"),
                                               (70000, "fp32")])
def test_every_record_is_listed_once(max_pos, precision):
    from paper_2606_15650_amd import api
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=128, n_heads=2, ffn=256, vocab=500, n_labels=9, max_pos=max_pos)
    _, m = make_model(cfg, precision, 0)
    pl = Pipeline(m)
    rng = np.random.default_rng(max_pos)
    top = min(max_pos, 3000)
    for name, L in [("one", [7]), ("edges", EDGES), ("edges back", EDGES[::-1]), ("empty", [0, 5, 0, 0, 129, 0]),
                    ("equal", [40] * 70), ("equal, many", [3] * 2500), ("mixed", rng.integers(0, 70, 1500)),
                    ("around 1024", rng.integers(1, 40, 1025)), ("longest", [1, top, 2, top, top - 31])]:
        L = np.asarray(L, np.int64)
        ids = rng.integers(0, cfg.vocab, int(L.sum())).astype(np.int32)
        api.device_errors(0, clear=True)
        got = _hidden(pl, ids, L)
        assert api.device_errors(0, clear=True) == 0
        say(f"[attention plan] {name}: {len(L)} records, {int(L.sum())} tokens, limit {max_pos}")
        step = max(1, len(L) // 8)
        want = np.concatenate([_hidden(pl, ids[L[:i].sum():L[:i + step].sum()], L[i:i + step])
                               for i in range(0, len(L), step) if L[i:i + step].sum()])
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("lengths", [EDGES, [513, 95, 1, 640]])
def test_fp32_attention_at_block_edges(lengths):
    """One layer against the float64 oracle: records around blocks of 32 keys,
    tiles of 64 and items of 128 rows, a longer one whose running reference
    grows."""
    from dataclasses import replace

    from oracle import encoder
    from paper_2606_15650_amd.pipeline import Pipeline
    from synth.configs import TINY
    cfg = replace(TINY, n_layers=1, max_pos=700)
    W, m = make_model(cfg, "fp32", 0)
    rng = np.random.default_rng(len(lengths))
    ids = rng.integers(0, cfg.vocab, sum(lengths)).astype(np.int32)
    got = _hidden(Pipeline(m), ids, lengths)
    ref = encoder.hidden_states(W, cfg, ids, np.concatenate([[0], np.cumsum(lengths)]), n_layers=1)
    # the bound of the repository's layer-by-layer FP32 test
    assert np.abs(got - ref).max() < 2e-5 * max(1.0, np.abs(ref).max())
