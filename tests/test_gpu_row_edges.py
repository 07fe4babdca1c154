"""Row kernels at the sizes where they can go wrong: label counts (odd) around
the classifier's blocks of 16 and its tiles of 16 tokens, record searches around
powers of 64, hidden states around 4096 elements and to an output aligned to
its elements only."""
from __future__ import annotations

import numpy as np
import pytest

from synth.configs import ModelConfig
from tests.gpu_common import make_model, say

pytestmark = pytest.mark.gpu


def _batch(ids, lengths):
    import torch
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)

    class Batch:
        B, h_cu, T, n_tokens = len(lengths), cu, int(cu[-1]), int(cu[-1])
    db = Batch()
    db.ids, db.cu = torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda()
    return db


@pytest.mark.parametrize("C", [1, 15, 17, 31, 33])
@pytest.mark.parametrize("hidden,precision", [(128, "fp32"), (128, "bf16"), (768, "bf16"), (1024, "fp32")])
def test_classifier_blocks_and_tiles(C, hidden, precision):
    import torch
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=hidden, n_heads=hidden // 64, ffn=128, vocab=300, n_labels=C, max_pos=512)
    W, m = make_model(cfg, precision, 0)
    pl = Pipeline(m)
    rng = np.random.default_rng(C)
    wc, bc = W["wc"].T.astype(np.float64), W["bc"].astype(np.float64)
    for T in (1, 15, 16, 17, 127, 129, 4097 if hidden == 128 else 300, 35000 if hidden == 128 and C == 17 else 2):
        L = [min(500, T - i) for i in range(0, T, 500)]
        db = _batch(rng.integers(0, cfg.vocab, T).astype(np.int32), L)
        x = pl.hidden(db, 1)[:T].cpu().numpy().astype(np.float64)
        lab, z, mg = (t[:T].cpu().numpy() for t in pl.ner(db, logits=True, margin=True))
        torch.cuda.synchronize()
        say(f"[classifier] {C} labels, {hidden} {precision}, {T} tokens")
        # a chain of `hidden` FP32 multiply-adds, then the bias
        bound = (hidden + 1) * 2.0 ** -24 * (np.abs(x) @ np.abs(wc).T + np.abs(bc))
        assert (np.abs(z - (x @ wc.T + bc)) <= bound).all()
        np.testing.assert_array_equal(lab, z.argmax(1))
        top = np.sort(z, 1)
        np.testing.assert_array_equal(mg, top[:, -1] - top[:, -2] if C > 1 else np.full(T, np.inf))


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("T", [65536 - 16, 65536, 65536 + 1, 2 * 65536 + 17])
def test_classifier_around_a_tile_per_wave(T, precision):
    """256 workgroups of 16 waves hold 65,536 tokens at once; the waves go on
    from there."""
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=256, n_heads=4, ffn=128, vocab=300, n_labels=17, max_pos=512)
    W, m = make_model(cfg, precision, 0)
    pl = Pipeline(m)
    db = _batch(np.random.default_rng(T).integers(0, cfg.vocab, T).astype(np.int32),
                [min(512, T - i) for i in range(0, T, 512)])
    x = pl.hidden(db, 1)[:T].cpu().numpy().astype(np.float64)
    lab, z, _ = (t[:T].cpu().numpy() for t in pl.ner(db, logits=True, margin=True))
    say(f"[classifier] {precision}, {T} tokens")
    wc, bc = W["wc"].T.astype(np.float64), W["bc"].astype(np.float64)
    bound = (cfg.hidden + 1) * 2.0 ** -24 * (np.abs(x) @ np.abs(wc).T + np.abs(bc))
    assert (np.abs(z - (x @ wc.T + bc)) <= bound).all()
    np.testing.assert_array_equal(lab, z.argmax(1))


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 4095, 4096, 4097, 9000])
def test_embedding_finds_records(B):
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=128, n_heads=2, ffn=128, vocab=300, n_labels=9, max_pos=512)
    W, m = make_model(cfg, "fp32", 0)
    pl = Pipeline(m)
    rng = np.random.default_rng(B)
    L = rng.integers(0, 4, B)
    L[-1] = 3
    ids = rng.integers(0, cfg.vocab, int(L.sum())).astype(np.int32)
    got = pl.hidden(_batch(ids, L), 0)[:len(ids)].cpu().numpy()
    # one long record has the same rows at the same positions
    pos = np.concatenate([np.arange(n) for n in L])
    for p in range(3):
        at = np.flatnonzero(pos == p)
        for i in at[:: max(1, len(at) // 4)]:
            one = ids[i - p:i + 1]
            np.testing.assert_array_equal(got[i], pl.hidden(_batch(one, [p + 1]), 0)[p].cpu().numpy())
    first = pl.hidden(_batch(ids[pos == 0], [1] * int((pos == 0).sum())), 0).cpu().numpy()
    np.testing.assert_array_equal(got[pos == 0], first[:int((pos == 0).sum())])


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_hidden_states_to_an_unaligned_output(precision, shift):
    import torch
    from paper_2606_15650_amd import api
    cfg = ModelConfig(n_layers=1, hidden=64, n_heads=1, ffn=128, vocab=300, n_labels=9, max_pos=512)
    _, m = make_model(cfg, precision, 0)
    rng = np.random.default_rng(1)
    for T in (1, 63, 64, 65, 128, 500):
        db = _batch(rng.integers(0, cfg.vocab, T).astype(np.int32), [T])
        n = m.workspace_size(T, 1)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        outs = []
        for s in (0, shift):
            buf = torch.full((T * 64 + 8,), -7.0, device="cuda")
            api.encoder_hidden(m, db.ids, db.cu, 1, T, 1, buf[s:], ws, n)
            torch.cuda.synchronize()
            assert (buf[:s] == -7).all() and (buf[s + T * 64:] == -7).all()
            outs.append(buf[s:s + T * 64].cpu().numpy())
        np.testing.assert_array_equal(outs[0], outs[1])


@pytest.mark.parametrize("T", [65535, 65536, 65537])
def test_layernorm_rows_per_wave(T):
    """One or two rows per wave, by the number of rows: the same bits."""
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=64, n_heads=1, ffn=128, vocab=300, n_labels=9, max_pos=512)
    _, m = make_model(cfg, "bf16", 0)
    pl = Pipeline(m)
    L = np.array([512] * (T // 512) + ([T % 512] if T % 512 else []))
    ids = np.random.default_rng(T).integers(0, cfg.vocab, T).astype(np.int32)
    got = pl.hidden(_batch(ids, L), 1)[:T].cpu().numpy()
    half = 64 * 512
    first = pl.hidden(_batch(ids[:half], L[:64]), 1)[:half].cpu().numpy()
    rest = pl.hidden(_batch(ids[half:], L[64:]), 1)[:T - half].cpu().numpy()
    np.testing.assert_array_equal(got, np.concatenate([first, rest]))


@pytest.mark.parametrize("C", [1, 9, 33])
def test_window_merge_over_short_and_long_records(C):
    """Record starts inside a wave's and a workgroup's tokens, empty records,
    windows merged beside records that need none: every record as alone."""
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = ModelConfig(n_layers=1, hidden=64, n_heads=1, ffn=128, vocab=300, n_labels=C, max_pos=64)
    _, m = make_model(cfg, "bf16", 0)
    pl = Pipeline(m)
    rng = np.random.default_rng(C)
    L = np.concatenate([rng.integers(0, 5, 300), [200, 1, 64, 65, 0, 0, 127], rng.integers(0, 90, 40), [300]])
    ids = rng.integers(0, cfg.vocab, int(L.sum())).astype(np.int32)
    T = len(ids)
    lab, z, mg = (x[:T].cpu().numpy() for x in pl.ner(_batch(ids, L), logits=True, margin=True, window=64, stride=32))
    at = np.concatenate([[0], np.cumsum(L)])
    for b in list(range(0, 300, 37)) + list(range(300, len(L))):
        if L[b] == 0:
            continue
        r = slice(at[b], at[b + 1])
        one = pl.ner(_batch(ids[r], [L[b]]), logits=True, margin=True, window=64, stride=32)
        for got, want in zip((lab, z, mg), one):
            np.testing.assert_array_equal(got[r], want[:L[b]].cpu().numpy())
