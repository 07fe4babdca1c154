"""decode_spans at the edges of its tiles (4096 tokens, 16 per thread) and past
the tile count up to which a workgroup sums the tiles before its own (16.8M
tokens): spans and record offsets bit-exact against a NumPy statement of the
BIO rule."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu
N_TYPES = 8


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return torch


def _reference(lab, cu):
    """Begin and end tokens of the spans, and cu_spans."""
    T = len(lab)
    typ = (lab.astype(np.int64) + 1) >> 1
    start = np.zeros(T + 1, bool)
    start[cu[cu < T]] = True
    prev = np.concatenate([[0], typ[:-1]])
    opens = (lab > 0) & ((lab & 1 == 1) | start[:T] | (prev != typ))
    # a span ends before the next token that is O, opens a span or starts a record
    stop = (lab == 0) | opens | start[:T]
    b = np.nonzero(opens)[0]
    s = np.concatenate([np.nonzero(stop)[0], [T]])
    e = s[np.searchsorted(s, b, side="right")]
    return b, e - 1, typ[b], np.searchsorted(b, cu).astype(np.int32)


@pytest.mark.parametrize("T,B", [(1, 1), (15, 3), (17, 40), (4095, 5), (4096, 1), (4097, 300), (8192, 4096),
                                 (70000, 9000), (4096 * 4096 + 5, 30000)])
def test_decode_at_tile_edges(torch_dev, T, B):
    torch = torch_dev
    from paper_2606_15650_amd import api
    rng = np.random.default_rng(T)
    cu = np.sort(rng.integers(0, T + 1, B - 1)).astype(np.int32)  # empty records among them
    cu = np.concatenate([[0], cu, [T]]).astype(np.int32)
    lab = rng.integers(1, 2 * N_TYPES + 1, T).astype(np.uint8)
    lab[rng.random(T) < 0.7] = 0
    run = rng.integers(0, T, max(1, T // 50))  # longer entities, some over a tile's end
    for k in range(1, 12):
        at = np.minimum(run + k, T - 1)
        lab[at] = np.where(lab[run] > 0, ((lab[run] + 1) >> 1) * 2, lab[at])
    off = np.stack([np.arange(T) * 3, np.arange(T) * 3 + 2], 1).astype(np.int32)
    b, e, t, want_cu = _reference(lab, cu)
    say(f"[decode] T={T} B={B}: {len(b)} spans")
    cap = len(b) + 3
    spans = torch.full((cap, 3), -1, dtype=torch.int64, device="cuda")
    cu_spans = torch.full((B + 1,), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(api.decode_workspace_size(T, B), dtype=torch.uint8, device="cuda")
    api.decode_spans(torch.from_numpy(lab).cuda(), torch.from_numpy(off).cuda(), torch.from_numpy(cu).cuda(), B, T,
                     N_TYPES, spans, cap, cu_spans, ws, ws.numel())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cu_spans.cpu().numpy(), want_cu)
    got = spans.cpu().numpy()
    rec = np.searchsorted(cu, b, side="right") - 1
    np.testing.assert_array_equal(got[:len(b), 0], rec | (t << 32))
    np.testing.assert_array_equal(got[:len(b), 1], off[b, 0])
    np.testing.assert_array_equal(got[:len(b), 2], off[e, 1])
    assert (got[len(b):] == -1).all()
    assert api.device_errors() == 0


@pytest.mark.parametrize("length", [31, 32, 33, 34, 63, 64, 65, 96, 97, 128, 129, 4094, 4095, 4096, 4097, 100000])
def test_long_spans(torch_dev, length):
    """A span of `length` tokens from every place around a tile's end on, ended by
    O, by another type, by its record or by the text."""
    torch = torch_dev
    from paper_2606_15650_amd import api
    parts, cu = [], [0]
    for i, at in enumerate([0, 1, 4060, 4063, 4064, 4095] if length < 10000 else [5]):
        pad = (at - sum(map(len, parts))) % 4096
        parts += [np.zeros(pad, np.uint8), np.array([3], np.uint8), np.full(length - 1, 4, np.uint8)]
        if i % 3 == 2:
            cu.append(sum(map(len, parts)))  # the record ends; the next begins with the same type
            parts.append(np.full(5, 4, np.uint8))
        else:
            parts.append(np.array([[0, 6][i % 2]], np.uint8))
    parts += [np.array([5], np.uint8), np.full(length - 1, 6, np.uint8)]  # to the text's end
    lab = np.concatenate(parts)
    T = len(lab)
    cu = np.array(cu + [T], np.int32)
    b, e, t, want_cu = _reference(lab, cu)
    off = np.stack([np.arange(T) * 3, np.arange(T) * 3 + 2], 1).astype(np.int32)
    say(f"[decode] spans of {length}: T={T}, {len(b)} spans")
    spans = torch.full((len(b), 3), -1, dtype=torch.int64, device="cuda")
    cu_spans = torch.empty(len(cu), dtype=torch.int32, device="cuda")
    ws = torch.empty(api.decode_workspace_size(T, len(cu) - 1), dtype=torch.uint8, device="cuda")
    d_lab, d_off, d_cu = (torch.from_numpy(x).cuda() for x in (lab, off, cu))

    def call():
        api.decode_spans(d_lab, d_off, d_cu, len(cu) - 1, T, N_TYPES, spans, len(b), cu_spans, ws, ws.numel())
    call()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cu_spans.cpu().numpy(), want_cu)
    got = spans.cpu().numpy()
    np.testing.assert_array_equal(got[:, 0], (np.searchsorted(cu, b, side="right") - 1) | (t << 32))
    np.testing.assert_array_equal(got[:, 1], off[b, 0])
    np.testing.assert_array_equal(got[:, 2], off[e, 1])
    assert api.device_errors() == 0
    if length == 100000:
        from tests.test_gpu_empty_records import _us
        us = _us(call)
        say(f"[decode] spans of {length}: {us:.0f} us")
        assert us < 5000  # (labels one by one: a load's latency each, over 10 ms)
