"""pseudonymize where its kernels' splits can go wrong: records with more spans
than a wave (64) or the staged list (512) holds, entities around the SHA block
(55, 56, 64) and the cached length (96), invalid and preserved spans inside a
full wave of valid ones, 16-byte output chunks at every alignment, records
longer than one workgroup's chunks, no room at the end.  Bytes against the
oracle, with a span taken or skipped by the sequential rule."""
from __future__ import annotations

import random

import numpy as np
import pytest

from oracle import pseudonym as ops
from tests.gpu_common import say

pytestmark = pytest.mark.gpu
TYPES = ["T", "HOSTNAME", "IP_ADDRESS"]
KEY = b"0123456789abcdef"


def _run(records, spans, slug, cache, out_short=0, out_shift=0):
    """Output bytes per record, and the bytes after the output's capacity."""
    import torch
    from paper_2606_15650_amd import api
    dev = torch.device("cuda:0")
    text, cu = b"".join(records), np.concatenate([[0], np.cumsum([len(r) for r in records])]).astype(np.int64)
    rows = [(b, t, s, e) for b, sp in enumerate(spans) for t, s, e in sp]
    cs = np.concatenate([[0], np.cumsum([len(sp) for sp in spans])]).astype(np.int32)
    d_text = torch.from_numpy(np.frombuffer(text or b"\0", np.uint8).copy()).to(dev)
    d_cu, d_cs = torch.from_numpy(cu).to(dev), torch.from_numpy(cs).to(dev)
    raw = np.zeros((max(len(rows), 1), 3), np.int64)  # int32 record, type; int64 begin, end
    for i, (b, t, s, e) in enumerate(rows):
        raw[i] = b | t << 32, s, e
    d_sp = torch.from_numpy(raw).to(dev)
    want_len = len(b"".join(_want(records, spans, slug)))
    cap = max(want_len - out_short, 0)
    buf = torch.full((cap + 64 + out_shift,), 0xEE, dtype=torch.uint8, device=dev)
    d_out, d_co = buf[out_shift:], torch.zeros(len(records) + 1, dtype=torch.int64, device=dev)
    n_ws = api.pseudonymize_workspace_size(len(records), len(rows))
    ws = torch.empty(max(n_ws, 1), dtype=torch.uint8, device=dev)
    api.pseudonymize(cache, d_text, d_cu, len(records), d_sp, d_cs, len(rows), d_out, cap, d_co, ws, n_ws)
    torch.cuda.synchronize()
    co, host = d_co.cpu().numpy(), buf.cpu().numpy()
    assert (host[:out_shift] == 0xEE).all() and (host[out_shift + cap:] == 0xEE).all()
    out = host[out_shift:out_shift + cap].tobytes()
    return [out[co[b]:co[b + 1]] for b in range(len(records))], int(co[-1]), cap


def _want(records, spans, slug, preserve=()):
    out = []
    for text, sp in zip(records, spans):
        took, prev = [], 0
        for t, s, e in sp:
            if not (1 <= t <= len(TYPES) and prev <= s <= e <= len(text)) or t in preserve:
                continue
            took.append((t, s, e))
            prev = e
        out.append(ops.substitute(text, took, TYPES, KEY, slug))
    return out


def _record(rng, n_spans, lengths, gap):
    text, spans = b"", []
    for _ in range(n_spans):
        text += bytes(rng.randrange(32, 127) for _ in range(rng.randint(0, gap)))
        n = rng.choice(lengths)
        spans.append((rng.randint(1, 3), len(text), len(text) + n))
        text += bytes(rng.randrange(256) for _ in range(n))
    return text + b"." * rng.randint(0, gap), spans


@pytest.mark.parametrize("slug", [0, 1, 10, 64])
def test_span_counts_and_entity_lengths(slug):
    from paper_2606_15650_amd import api
    rng = random.Random(slug)
    lengths = [0, 1, 3, 4, 15, 16, 17, 31, 32, 33, 54, 55, 56, 63, 64, 65, 79, 80, 95, 96, 97, 119, 120, 200]
    pairs = [_record(rng, n, lengths, 12) for n in (0, 1, 63, 64, 65, 128, 129, 511, 512, 513, 700)]
    pairs += [_record(rng, 2, [n], 3) for n in lengths]  # (the last ends near the text's end)
    records, spans = [p[0] for p in pairs], [p[1] for p in pairs]
    cache = api.PseudonymCache(KEY, slug, TYPES, 1 << 14)
    api.device_errors(0, clear=True)
    say(f"[pseudonymize] {sum(map(len, spans))} spans, slug {slug}")
    want = _want(records, spans, slug)
    for _ in range(2):  # the second time from the table
        got, total, _ = _run(records, spans, slug, cache)
        assert got == want and total == len(b"".join(want))
    short = {(r[s:e]) for r, sp in zip(records, spans) for _, s, e in sp if e - s <= 96}
    n = sum(e - s <= 96 for sp in spans for _, s, e in sp)
    st = cache.stats()
    if slug:
        assert st["lookups"] == 2 * n and n <= st["hits"] <= 2 * n and st["entries"] >= len(short)
        assert {m["original"] for m in cache.export()} == short
    else:
        assert st["lookups"] == 0
    assert api.device_errors(0, clear=True) == 0


@pytest.mark.parametrize("at", [0, 1, 62, 63, 64, 100])
def test_invalid_and_preserved_spans_among_valid_ones(at):
    from paper_2606_15650_amd import api
    rng = random.Random(at)
    text, sp = _record(rng, 101, [1, 5, 20], 9)
    t, s, e = sp[at]
    bads = [(t, max(s - 30, 0), e), (0, s, e), (4, s, e), (t, e, s - 1), (t, s, len(text) + 1), (t, s, len(text))]
    lists = [sp[:at] + [bad] + sp[at + 1:] for bad in bads]
    cache = api.PseudonymCache(KEY, 8, TYPES, 1 << 12)
    api.device_errors(0, clear=True)
    got, _, _ = _run([text] * len(lists), lists, 8, cache)
    assert got == _want([text] * len(lists), lists, 8)
    assert api.device_errors(0, clear=True) & api.ERR_SPAN
    cache.set_preserve(["HOSTNAME"])
    # (_run's capacity is the length without preserved types, which is larger or smaller: give it room)
    want = _want([text], [sp], 8, preserve=(2,))
    got, total, cap = _run([text], [sp], 8, cache, out_short=-len(text))
    assert total == len(want[0]) <= cap and got == want
    assert api.device_errors(0, clear=True) == 0


@pytest.mark.parametrize("shift", [0, 1, 7, 15])
def test_output_chunks_at_every_alignment_and_short_capacity(shift):
    from paper_2606_15650_amd import api
    rng = random.Random(shift)
    pairs = [_record(rng, n, [4, 40], g) for n, g in [(1, 0), (3, 60), (0, 1), (0, 15), (0, 16), (0, 17), (0, 0), (40, 700),
                                                      (2, 9000), (600, 90)]]
    records, spans = [p[0] for p in pairs] * 2, [p[1] for p in pairs] * 2
    cache = api.PseudonymCache(KEY, 12, TYPES, 1 << 12)
    want = b"".join(_want(records, spans, 12))
    for short in (0, 1, 15, 16, 33, len(want) // 2, len(want)):
        api.device_errors(0, clear=True)
        got, total, cap = _run(records, spans, 12, cache, out_short=short, out_shift=shift)
        assert total == len(want) and b"".join(got) == want[:cap]
        assert bool(api.device_errors(0, clear=True) & api.ERR_OUT_CAP) == (short > 0)


@pytest.mark.parametrize("n_records", [16384, 16385, 40000, 63 * 16384 + 1])
def test_several_records_to_a_wave(n_records):
    """Above 16,384 records a wave lays out several: most empty, some with as
    many spans as one lane takes (8), with more, with a wave's and an invalid
    one among them."""
    from paper_2606_15650_amd import api
    rng = random.Random(n_records)
    records, spans = [b""] * n_records, [[] for _ in range(n_records)]
    special = [0, 1, 62, 63, 64, 65, n_records - 2, n_records - 1] + [rng.randrange(n_records) for _ in range(500)]
    for i, b in enumerate(special):
        records[b], spans[b] = _record(rng, [0, 1, 2, 7, 8, 9, 63, 64, 65, 130][i % 10], [0, 3, 20, 60], 9)
        if i % 7 == 3 and spans[b]:
            k = rng.randrange(len(spans[b]))
            spans[b][k] = (rng.choice([0, 4, 1]), spans[b][k][1], len(records[b]) + 1)
    cache = api.PseudonymCache(KEY, 10, TYPES, 1 << 14)
    api.device_errors(0, clear=True)
    say(f"[pseudonymize] {n_records} records, {sum(map(len, spans))} spans")
    got, total, _ = _run(records, spans, 10, cache)
    want = _want(records, spans, 10)
    assert total == len(b"".join(want)) and got == want
    assert api.device_errors(0, clear=True) == api.ERR_SPAN


def test_many_new_entities_at_once():
    """A table filled by one call, nearly every span an entity of its own: no
    more than a small part of the call goes into waiting for other entities'
    slots.  The outputs of the second call, from the table, are the same."""
    import torch
    from paper_2606_15650_amd import api
    from tests.test_gpu_empty_records import _us
    rng = random.Random(3)
    records, rows = [], []
    for i in range(2000):
        text = b""
        for _ in range(60):
            n = rng.randint(6, 20)
            rows.append((i | (1 + n % 3) << 32, len(text), len(text) + n))
            text += bytes(rng.choice(b"abcdefghij") for _ in range(n)) + b" "
        records.append(text)
    text = b"".join(records)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum([len(r) for r in records])]).astype(np.int64)).cuda()
    cs = torch.arange(0, 60 * 2000 + 1, 60, dtype=torch.int32, device="cuda")
    d_text = torch.from_numpy(np.frombuffer(text, np.uint8).copy()).cuda()
    d_sp = torch.from_numpy(np.array(rows, np.int64)).cuda()
    cap = len(text) + 40 * len(rows)
    out, cu_out = torch.empty(cap, dtype=torch.uint8, device="cuda"), torch.empty(2001, dtype=torch.int64, device="cuda")
    n_ws = api.pseudonymize_workspace_size(2000, len(rows))
    ws = torch.empty(n_ws, dtype=torch.uint8, device="cuda")
    cache = api.PseudonymCache(KEY, 10, TYPES, 1 << 18)

    def call():
        cache.clear()
        api.pseudonymize(cache, d_text, cu, 2000, d_sp, cs, len(rows), out, cap, cu_out, ws, n_ws)
    cold = _us(call)
    st, first = cache.stats(), out[:int(cu_out[-1])].clone()
    entities = [records[r & 0xFFFFFFFF][b:e] for r, b, e in rows]
    assert len(set(entities)) > 0.99 * len(rows) and st["lookups"] == len(rows)
    table = {m["original"] for m in cache.export()}  # (one whose 32 places are taken is not cached)
    assert len(table) > 0.99 * len(rows)
    api.pseudonymize(cache, d_text, cu, 2000, d_sp, cs, len(rows), out, cap, cu_out, ws, n_ws)
    assert torch.equal(out[:int(cu_out[-1])], first)
    assert cache.stats()["hits"] - st["hits"] == sum(e in table for e in entities)
    k = 37
    want = ops.substitute(records[k], [(int(r >> 32), b, e) for r, b, e in rows[60 * k:60 * k + 60]], TYPES, KEY, 10)
    assert first[int(cu_out[k]):int(cu_out[k + 1])].cpu().numpy().tobytes() == want
    cache.set_enabled(False)
    without = _us(call)
    say(f"[pseudonymize] {len(rows)} new entities {cold:.1f} us, without a table {without:.1f} us")
    assert cold < 3.3 * without
    assert api.device_errors(0, clear=True) == 0


def test_many_invalid_spans():
    """Every second span invalid: the calls end with the error bit and the valid
    spans replaced, and the invalid ones do not queue up for the bit."""
    import torch
    from paper_2606_15650_amd import api
    from tests.test_gpu_empty_records import _us
    B, per = 1024, 60
    records = [bytes(97 + (i + j) % 26 for j in range(per * 10)) for i in range(B)]
    cu = torch.arange(0, B * per * 10 + 1, per * 10, dtype=torch.int64, device="cuda")
    cs = torch.arange(0, B * per + 1, per, dtype=torch.int32, device="cuda")
    d_text = torch.from_numpy(np.frombuffer(b"".join(records), np.uint8).copy()).cuda()
    cap = B * per * 40
    out, cu_out = torch.empty(cap, dtype=torch.uint8, device="cuda"), torch.empty(B + 1, dtype=torch.int64, device="cuda")
    n_ws = api.pseudonymize_workspace_size(B, B * per)
    ws = torch.empty(n_ws, dtype=torch.uint8, device="cuda")
    cache = api.PseudonymCache(KEY, 10, TYPES, 1 << 16)
    us = {}
    for kind in ("valid", "invalid"):
        lists = [[(1 + k % 3, 10 * k + 2, 10 * k + (8 if kind == "valid" or k % 2 else 1)) for k in range(per)] for _ in range(B)]
        rows = np.array([(b | t << 32, s, e) for b in range(B) for t, s, e in lists[b]], np.int64)
        d_sp = torch.from_numpy(rows).cuda()
        api.device_errors(0, clear=True)
        us[kind] = _us(lambda: api.pseudonymize(cache, d_text, cu, B, d_sp, cs, B * per, out, cap, cu_out, ws, n_ws))
        assert api.device_errors(0, clear=True) == (0 if kind == "valid" else api.ERR_SPAN)
        want = _want(records[:40], lists[:40], 10)
        assert out[:int(cu_out[40])].cpu().numpy().tobytes() == b"".join(want)
    say(f"[pseudonymize] {B * per} spans {us['valid']:.1f} us, every second invalid {us['invalid']:.1f} us")
    assert us["invalid"] < 3 * us["valid"]
