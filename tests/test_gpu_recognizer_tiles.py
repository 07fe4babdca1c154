"""recognize_spans where its tiles can go wrong: matches and runs over a tile's
end (4096 bytes) at every offset, runs longer than the staged window, hashes
around 16-byte blocks and record starts, tiles with more record boundaries
than are staged, unions over several tiles.  Bit-exact against the oracle."""
from __future__ import annotations

import random

import numpy as np
import pytest

from oracle import recognizers as R
from tests.gpu_common import make_cache, say
from tests.test_gpu_recognizers import _per_record, _recognize_gpu, _text_batch

pytestmark = pytest.mark.gpu
TYPES = ["IP_ADDRESS", "HOSTNAME", "CVE_ID", "EMAIL_ADDRESS", "PORT", "URL", "MAC_ADDRESS", "HASH", "CPE"]
HEX = b"0123456789abcdef"
ENTITIES = [b"10.20.30.40", b"a1.b2.example", b"CVE-2021-44228", b"x.y@mail.corp", b"https://h.lan/p?q=1",
            b"00:1a:2b:3c:4d:5e", HEX * 2, HEX * 2 + HEX[:8], HEX * 4, b"2001:db8::1:2", b"cpe:2.3:a:x:y:1.0:*"]


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return torch


def _check(records, label):
    rb = _text_batch(records, TYPES)
    cache = make_cache(TYPES)
    rt = R.recognizer_types(TYPES)
    cu, arr = _recognize_gpu(rb, cache)
    got = _per_record(cu, arr, len(records))
    want = [R.resolve_record(t, [], rt) for t in records]
    say(f"[recognize] {label}: {len(records)} records, {sum(map(len, want))} spans")
    assert sum(map(len, want)) > 0
    for b, (g, w) in enumerate(zip(got, want)):
        assert g == w, (label, b, records[b][:80])


@pytest.mark.parametrize("shift", range(0, 48, 3))
def test_matches_over_a_tile_end(torch_dev, shift):
    out = []
    for i, e in enumerate(ENTITIES):  # every entity ends `shift` bytes after a multiple of 4096
        pad = 4096 - (len(e) + 1 - shift) % 4096
        out.append(b"w" * (pad - 1) + b" " + e + b"\n" + b"z" * ((4096 - (shift + 1)) % 4096))
    _check(out, f"entities ending {shift} past a tile")
    _check([b"".join(out)], "the same in one record")


def test_long_runs_and_many_boundaries(torch_dev):
    rng = random.Random(5)
    long_label = b"a" * 9000
    _check([long_label + b".net x " + long_label + b"@" + long_label + b".org", b"http://" + b"u" * 13000 + b" 1.2.3.4",
            b"http://h.lan/" + b"10.0.0.1/" * 1500, b"fe" * 5000 + b" " + HEX * 4], "runs past the window")
    # one-byte and empty records, hashes and addresses cut by record boundaries
    text = b"".join(rng.choice(ENTITIES) + rng.choice([b"", b" ", b".", b":", b"a", b"-", b"\n"]) for _ in range(1500))
    for step in (1, 3, 17, 40, 200):
        recs, at = [], 0
        while at < len(text):
            n = rng.randint(0, 2 * step)
            recs.append(text[at:at + n])
            at += n
        _check(recs, f"records of up to {2 * step} bytes")
