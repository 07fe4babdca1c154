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
