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
