"""field_spans where its tiles can go wrong: lines, names, colons and values
over a tile's end (8192 bytes) at every offset, names of 32 and 33 bytes,
values past the staged window (448 bytes after the tile), tiles full of the
shortest fields, many record boundaries in one tile.  Bit-exact against the
oracle."""
from __future__ import annotations

import random

import numpy as np
import pytest

from oracle import fields as F
from synth.records import TYPE_NAMES_17
from tests.gpu_common import make_cache, say
from tests.test_gpu_fields import _fields_gpu, _text_batch

pytestmark = pytest.mark.gpu
LONG = b"N" * 32
CONFIG = {b"Host": 1, b"x": 2, b"See Also": 3, LONG: 4, LONG[:31]: 5, b"Hosts": 6}


def _check(records, label, least=1):
    rb = _text_batch(records, TYPE_NAMES_17)
    _, got = _fields_gpu(rb, make_cache(TYPE_NAMES_17), CONFIG)
    want = F.field_spans_batch(rb.text, rb.cu_bytes, CONFIG)
    say(f"[fields] {label}: {len(records)} records, {sum(map(len, want))} spans")
    assert sum(map(len, want)) >= least
    assert got == want, label


@pytest.mark.parametrize("shift", range(0, 64, 3))
def test_lines_over_a_tile_end(shift):
    import torch
    assert torch.cuda.is_available()
    out = []
    for i, line in enumerate([b"Host: abc", b"See Also: y", LONG + b": v", LONG + b"N: v", LONG[:31] + b": " + b"w" * 40,
                              b"x: " + b"q" * 60, b"Host:", b"Host: ", b"Host:a", b"x: 1"]):
        # every line begins `shift` bytes before a multiple of 8192
        at = sum(map(len, out))
        out.append(b"-" * ((-(at + 1 + shift)) % 8192) + b"\n" + line + (b"\n" if i % 2 else b""))
        if i % 3 == 0:
            out.append(b"")
    _check(out, f"lines from {shift} before a tile's end")
    _check([b"".join(out)], "the same in one record")
    _check([b"".join(out).replace(b"\n", b"", 1), b"Host: z"], "a first line without a break")


@pytest.mark.parametrize("length", [438, 441, 442, 443, 444, 445, 450, 8180, 8640, 17000])
def test_values_past_the_window(length):
    import torch
    assert torch.cuda.is_available()
    for tail in (b"", b"\n", b"\nHost: a"):
        first = b"-" * 8186 + b"\n" + b"x: " + b"v" * length + tail
        _check([first, b"Host: b\n"], f"a value of {length} from 8190")
        _check([first], "the same at the text's end")


def test_full_tiles_and_many_boundaries():
    import torch
    assert torch.cuda.is_available()
    rng = random.Random(7)
    _check([b"x: v\n" * 4000], "the shortest lines")
    _check([b"x: v"] * 3000, "the shortest records")
    _check([b"\n", b"", b"x: v", b"", b"Host", b": a", b"Host:", b" a", b"x: "] * 400, "fields cut by records")
    text = b"".join(rng.choice([b"Host: ", b"x: ", b"See Also: ", LONG + b": ", b"\n", b":", b" ", b"v", b"10.0.0.1\n"])
                    for _ in range(6000))
    for step in (1, 3, 5, 17, 200):
        _check([text[i:i + step] for i in range(0, min(len(text), 4000 * step), step)], f"records of {step}",
               least=step > 3)  # "x: v" has 4 bytes


def _key(name):
    """The library's key of a name (its zero-padded dwords and length)."""
    h = len(name) * 0x9E3779B1 & 0xFFFFFFFF
    for i in range(0, 32, 4):
        h = (h ^ int.from_bytes(name[i:i + 4].ljust(4, b"\0"), "little")) * 0x85EBCA6B & 0xFFFFFFFF
        h ^= h >> 15
    return h


def test_names_of_one_key():
    seen, pairs = {}, []
    for i in range(400000):
        name = b"f%x" % (i * 2654435761 % (1 << 40))
        other = seen.setdefault(_key(name), name)
        if other != name:
            pairs.append((other, name))
    assert len(pairs) >= 5
    text = b"".join(a + b": 1\n" + b + b": two\n" for a, b in pairs)
    for which in ((0,), (1,), (0, 1), (1, 0)):
        config = {p[k]: 1 + (2 * i + k) % 8 for i, p in enumerate(pairs[:16]) for k in which}
        rb = _text_batch([text, text[5:]], TYPE_NAMES_17)
        _, got = _fields_gpu(rb, make_cache(TYPE_NAMES_17), config)
        assert got == F.field_spans_batch(rb.text, rb.cu_bytes, config)
        assert sum(map(len, got)) > 0


@pytest.mark.parametrize("line", [b"a\n", b"ab: \n", b"a:b: c\n", b"n" * 32 + b": v\n", b"n" * 33 + b": v\n"])
def test_short_lines_that_hold_no_field_or_few(line):
    """As many lines as a tile can hold, without a ':' or with one that makes no
    configured field: a line costs no look past its name."""
    import torch
    from paper_2606_15650_amd import api
    from tests.test_gpu_empty_records import _us
    config = {"a": 1, "n" * 32: 2}

    def call(text, B):
        n = len(text)
        d_text = torch.from_numpy(np.frombuffer(text, np.uint8).copy()).cuda()
        cu = torch.linspace(0, n, B + 1, dtype=torch.float64).to(torch.int64).cuda()
        cap = n // 4 + 1
        spans, cs = torch.empty((cap, 3), dtype=torch.int64, device="cuda"), torch.empty(B + 1, dtype=torch.int32, device="cuda")
        ws = torch.empty(api.field_workspace_size(n, B), dtype=torch.uint8, device="cuda")
        return lambda: api.field_spans(d_text, cu, B, n, config, 2, spans, cap, cs, ws, ws.numel()), spans, cs
    count = 4_800_000 // len(line)
    fn, spans, cs = call(line * count, 1)
    many = _us(fn)
    n = int(cs[1])
    assert n == (count if len(line) == 36 and line[0] == ord("n") and line[32] == ord(":") else 0)
    if n:
        got = spans[:n].cpu().numpy()
        begin = np.arange(n) * len(line) + 34
        np.testing.assert_array_equal(got, np.stack([np.full(n, 2 << 32), begin, begin + 1], 1))
    few = _us(call((b"x" * 1199 + b"\n") * 4000, 1)[0])
    say(f"[fields] {count} lines {line[:8]}: {n} fields, {many:.1f} us, lines of 1200 bytes {few:.1f} us")
    assert many < 4 * few + 20
    assert api.device_errors() == 0
