"""recognize_spans on texts that load one part of it: matches as dense as they
can be, NER spans over many tiles (4096 bytes) with matches inside.  Bit-exact
against the oracle, and not much slower than the same bytes without them."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import recognizers as R
from tests.gpu_common import say
from tests.test_gpu_empty_records import _batch, _pipeline, _us
from tests.test_gpu_recognizers import _ner_device

pytestmark = pytest.mark.gpu
NAMES = ["IP_ADDRESS", "HOSTNAME", "EMAIL_ADDRESS", "URL", "HASH"]


def _run(records, ner=()):
    """Spans (record, type, begin, end), and the call."""
    from paper_2606_15650_amd import api
    from paper_2606_15650_amd.pipeline import spans_to_numpy
    pl, db = _pipeline(NAMES), _batch(b"".join(records), np.array([len(r) for r in records]))
    d_ner, d_cu, n = _ner_device(np.array(ner, np.int64).reshape(-1, 4), len(records))

    def call():
        return pl.recognize(db, d_ner, d_cu, n, span_cap=db.n_bytes // 2)
    spans, cu, _ = call()
    got = spans_to_numpy(spans, int(cu[-1]))
    assert api.device_errors() == 0
    return got, call


def _check(got, records, ner=()):
    rt = R.recognizer_types(NAMES)
    want = []
    for b, t in enumerate(records):
        spans = [(int(x[1]), int(x[2]), int(x[3])) for x in ner if x[0] == b]
        want += [(b, *w) for w in R.resolve_record(t, spans, rt)]
    np.testing.assert_array_equal(got, np.array(want, np.int64).reshape(-1, 4))


@pytest.mark.parametrize("word", [b"::1 ", b"10.0.0.1 ", b"a@b.co "])
def test_dense_matches(word):
    small = [word * (5000 // len(word)), b"x" + word * 3]
    got, _ = _run(small)
    _check(got, small)
    records = [word * (1200 // len(word))] * 1024
    got, call = _run(records)
    assert len(got) == 1024 * (1200 // len(word))
    _, none = _run([(b"x" * (len(word) - 1) + b" ") * (1200 // len(word))] * 1024)
    dense, plain = _us(call), _us(none)
    say(f"[recognize] {word}: {len(got)} spans, {dense:.1f} us, without matches {plain:.1f} us")
    assert dense < 5.5 * plain


@pytest.mark.parametrize("size", [1023, 1025, 4096, 20000, 300000])
def test_long_ner_spans(size):
    """NER spans around the length from which a wave marks them and over many
    tiles, with matches inside, at every offset in a 64-byte word."""
    words = [b"alpha ", b"10.0.0.1 ", b"host.lan ", b"x@y.org ", b"z" * 61 + b" "]
    rng = np.random.default_rng(size)
    body = b"".join(words[k] for k in rng.integers(0, len(words), size // 5))
    shifts = range(0, 66, 5) if size < 10000 else (0, 1, 64)
    records = [b"-" * (i % 7) + body[:size + 40] + b" 10.0.0.9 " + b"q" * (64 - i) for i in shifts]
    ner = [(r, 1 + r % 2, 3 + i // 2, 3 + i // 2 + size - r) for r, i in enumerate(shifts)]
    got, call = _run(records, ner)
    _check(got, records, ner)
    bare, none = _run(records)
    say(f"[recognize] NER spans of {size}: {len(got)} spans, {_us(call):.1f} us; without {len(bare)}, {_us(none):.1f} us")


def test_one_span_over_eight_megabytes():
    records = [b"alpha 10.0.0.1 beta x@y.org gamma host.lan " * 190000]
    size = len(records[0])
    got, call = _run(records, [(0, 2, 1, size - 1)])
    np.testing.assert_array_equal(got, [[0, 2, 1, size - 1]])
    one, none = _us(call), _us(_run(records)[1])
    say(f"[recognize] one NER span of {size} bytes {one:.1f} us, without it {none:.1f} us")
    assert one < 40 * none
