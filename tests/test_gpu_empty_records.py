"""Batches with very many empty records at one place: results as for the same
batch without them, and no call is much slower than with as many empty records
spread over it (a workgroup must not go through them one after the other)."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu
N_TYPES = 8
EMPTY = 400_000


def _us(fn):
    """Best of five: GPU time of a call, in microseconds."""
    import torch
    fn()
    best = 1e30
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 3 * 1e3)
    return best


def _lengths(full, where):
    """`full` with EMPTY zeros: at one place, or spread over it."""
    full = np.asarray(full, np.int64)
    if where == "one place":
        return np.concatenate([full[:len(full) // 2], np.zeros(EMPTY, np.int64), full[len(full) // 2:]])
    out = np.zeros((len(full), EMPTY // len(full) + 1), np.int64)
    out[:, 0] = full
    return out.ravel()


def _cu(lengths, dtype):
    import torch
    return torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(dtype)).cuda()


def _unrecord(spans, cu_spans, lengths):
    """Spans with the index of their record among those that are not empty."""
    n = int(cu_spans[-1])
    got = spans[:n].cpu().numpy()
    rec = got[:, 0] & 0xFFFFFFFF
    per = np.searchsorted(cu_spans.cpu().numpy(), np.arange(n), side="right") - 1
    np.testing.assert_array_equal(rec, per)  # (record r's spans are cu_spans[r] .. cu_spans[r + 1])
    index = np.cumsum(lengths > 0) - 1
    got[:, 0] += index[rec] - rec
    return got


def _compare(call, full):
    """call(lengths) -> (function, spans, cu_spans)"""
    out, us = {}, {}
    for where in ("none", "spread", "one place"):
        lengths = np.asarray(full, np.int64) if where == "none" else _lengths(full, where)
        fn, spans, cu_spans = call(lengths)
        us[where] = _us(fn)
        out[where] = _unrecord(spans, cu_spans, lengths)
        say(f"[empty records] {where}: {len(lengths)} records, {len(out[where])} spans, {us[where]:.1f} us")
    assert len(out["none"]) > 0
    np.testing.assert_array_equal(out["spread"], out["none"])
    np.testing.assert_array_equal(out["one place"], out["none"])
    from paper_2606_15650_amd import api
    assert api.device_errors() == 0
    assert us["one place"] < 3 * us["spread"] + 50


def test_decode_spans():
    import torch
    from paper_2606_15650_amd import api
    full = [200] * 2000
    T = sum(full)
    rng = np.random.default_rng(1)
    lab = rng.integers(1, 2 * N_TYPES + 1, T).astype(np.uint8)
    lab[rng.random(T) < 0.7] = 0
    off = np.stack([np.arange(T) % 200 * 3, np.arange(T) % 200 * 3 + 2], 1).astype(np.int32)
    d_lab, d_off = torch.from_numpy(lab).cuda(), torch.from_numpy(off).cuda()

    def call(lengths):
        B = len(lengths)
        cu, spans = _cu(lengths, np.int32), torch.empty((T, 3), dtype=torch.int64, device="cuda")
        cu_spans = torch.empty(B + 1, dtype=torch.int32, device="cuda")
        ws = torch.empty(api.decode_workspace_size(T, B), dtype=torch.uint8, device="cuda")
        return (lambda: api.decode_spans(d_lab, d_off, cu, B, T, N_TYPES, spans, T, cu_spans, ws, ws.numel()), spans,
                cu_spans)
    _compare(call, full)


def _batch(text, lengths):
    """What Pipeline reads of a batch that has a text only."""
    import torch

    class Batch:
        B, n_bytes = len(lengths), len(text)
    Batch.text = torch.from_numpy(np.frombuffer(text, np.uint8).copy()).cuda()
    Batch.cu_bytes = _cu(lengths, np.int64)
    return Batch


def _pipeline(names):
    import torch
    from paper_2606_15650_amd.pipeline import Pipeline
    from tests.gpu_common import make_cache
    pl = Pipeline.__new__(Pipeline)
    pl.cache, pl.device, pl._ws, pl.n_types = make_cache(names), torch.device("cuda:0"), {}, len(names)
    return pl


def test_recognize_spans():
    pl = _pipeline(["IP_ADDRESS", "HOSTNAME", "EMAIL_ADDRESS", "URL", "HASH"])
    records = [b"host.lan 10.0.0.1 x@y.org " + b"0123456789abcdef" * 2 + b" http://a.lan/" + b"p" * (i % 90)
               for i in range(1998)]
    # around the place, in one 64-byte word: an address, then a hash that only the record's start lets begin
    at = sum(map(len, records[:999]))
    records[999:999] = [b" " * (64 - at % 64 + 20) + b"10.0.0.1", b"0123456789abcdef" * 2]
    text, full = b"".join(records), [len(r) for r in records]

    def call(lengths):
        db = _batch(text, lengths)
        spans, cu_spans, _ = pl.recognize(db)

        def fn():
            s, c, _ = pl.recognize(db)
            spans[:] = s
            cu_spans[:] = c
        return fn, spans, cu_spans
    _compare(call, full)


def test_field_spans():
    pl = _pipeline(["IP_ADDRESS", "HOSTNAME"])
    records = [b"Source IP: 10.0.0.%d\nHost: a%d.lan\nNote: %s\n" % (i % 256, i, b"x" * (i % 70)) for i in range(8000)]
    text, full = b"".join(records), [len(r) for r in records]

    def call(lengths):
        db = _batch(text, lengths)
        config = {"Source IP": 1, "Host": 2}
        spans, cu_spans, _ = pl.fields(db, config)

        def fn():
            s, c, _ = pl.fields(db, config)
            spans[:] = s
            cu_spans[:] = c
        return fn, spans, cu_spans
    _compare(call, full)


def test_windowed_forward():
    """The window merge (the records' windows are listed on the host): a short
    record before the place and one after it in one wave of tokens."""
    import torch
    from paper_2606_15650_amd import api
    from synth.configs import TINY
    from tests.gpu_common import make_model
    _, m = make_model(TINY, "bf16", 0)
    full = [700] * 20 + [5, 7] + [700] * 20
    T = sum(full)
    ids = torch.from_numpy(np.random.default_rng(2).integers(0, TINY.vocab, T).astype(np.int32)).cuda()
    out, us = {}, {}
    for where in ("none", "spread", "one place"):
        lengths = np.asarray(full, np.int64) if where == "none" else _lengths(full, where)
        B, h_cu = len(lengths), np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
        cu, labels = torch.from_numpy(h_cu).cuda(), torch.empty(T, dtype=torch.uint8, device="cuda")
        z = torch.empty((T, TINY.n_labels), dtype=torch.float32, device="cuda")
        ws = torch.empty(m.windowed_workspace_size(h_cu, 512, 256), dtype=torch.uint8, device="cuda")
        us[where] = _us(lambda: api.ner_forward_windowed(m, ids, cu, h_cu, B, T, 512, 256, labels, z, None, ws,
                                                         ws.numel(), None))
        out[where] = labels.cpu().numpy(), z.cpu().numpy()
        say(f"[empty records] {where}: {B} records, windowed {us[where]:.1f} us")
    for where in ("spread", "one place"):
        np.testing.assert_array_equal(out[where][0], out["none"][0])
        np.testing.assert_array_equal(out[where][1], out["none"][1])
    assert us["one place"] < 3 * us["spread"] + 50
