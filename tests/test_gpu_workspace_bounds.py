"""Calls in exactly the workspace that they need, on the densest inputs and at
sizes around a tile: nothing is written past it, and the spans are right."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu
GUARD = 8192


def _call(fn, need, cap, B):
    """fn(spans, cu_spans, workspace pointer holder, bytes) in `need` bytes before a guard."""
    import torch
    from paper_2606_15650_amd import api
    ws = torch.full((need + GUARD,), 0xEE, dtype=torch.uint8, device="cuda")
    spans = torch.full((cap + 1, 3), -1, dtype=torch.int64, device="cuda")
    cu_spans = torch.empty(B + 1, dtype=torch.int32, device="cuda")
    fn(spans, cu_spans, ws, need)
    torch.cuda.synchronize()
    assert api.device_errors() == 0
    assert bool((ws[need:] == 0xEE).all()) and bool((spans[cap] == -1).all())
    with pytest.raises(api.AnonError):
        fn(spans, cu_spans, ws, need - 1)
    return spans[:int(cu_spans[-1])].cpu().numpy(), cu_spans.cpu().numpy()


def _slack(size):
    return size - 256  # (the sizes asked for have room to align the first buffer)


def _text(unit, n):
    import torch
    text = (unit * (n // len(unit) + 1))[:n]
    return torch.from_numpy(np.frombuffer(text, np.uint8).copy()).cuda()


@pytest.mark.parametrize("n", [4, 8, 100, 8188, 8192, 8196, 16384, 30000])
def test_fields_of_four_bytes(n):
    import torch
    from paper_2606_15650_amd import api
    B = n // 4  # a record each: "a: b"
    text, cu = _text(b"a: b", n), torch.arange(0, n + 1, 4, dtype=torch.int64, device="cuda")
    say(f"[workspace] {B} fields of four bytes")
    got, cs = _call(lambda s, c, ws, k: api.field_spans(text, cu, B, n, {"a": 1}, 1, s, B, c, ws, k),
                    _slack(api.field_workspace_size(n, B)), B, B)
    np.testing.assert_array_equal(cs, np.arange(B + 1))
    np.testing.assert_array_equal(got, np.stack([np.arange(B) | (1 << 32), np.full(B, 3), np.full(B, 4)], 1))


@pytest.mark.parametrize("n", [2, 4, 100, 4094, 4096, 4098, 8192, 12290])
def test_addresses_of_two_bytes(n):
    import torch
    from paper_2606_15650_amd import api
    B = n // 2  # a record each: "::"
    text, cu = _text(b"::", n), torch.arange(0, n + 1, 2, dtype=torch.int64, device="cuda")
    rt = api.recognizer_types(["IP_ADDRESS", "MAC_ADDRESS"])
    say(f"[workspace] {B} addresses of two bytes")
    got, cs = _call(lambda s, c, ws, k: api.recognize_spans(text, cu, B, n, rt, 2, None, None, 0, s, B, c, ws, k),
                    _slack(api.recognize_workspace_size(n, B)), B, B)
    np.testing.assert_array_equal(cs, np.arange(B + 1))
    np.testing.assert_array_equal(got, np.stack([np.arange(B) | (1 << 32), np.zeros(B), np.full(B, 2)], 1))


@pytest.mark.parametrize("T", [1, 15, 16, 17, 100, 4095, 4096, 4097, 8192, 9000])
def test_spans_of_one_token(T):
    import torch
    from paper_2606_15650_amd import api
    lab = torch.ones(T, dtype=torch.uint8, device="cuda")
    off = torch.stack([torch.arange(T), torch.arange(T) + 1], 1).to(torch.int32).cuda()
    cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    tiles = (T + 4095) // 4096
    bits = (2 * ((T + 15) // 16) + 255) // 256 * 256
    say(f"[workspace] {T} spans of a token")
    got, cs = _call(lambda s, c, ws, k: api.decode_spans(lab, off, cu, 1, T, 1, s, T, c, ws, k),
                    2 * bits + 8 * (tiles + 1), T, 1)
    assert cs.tolist() == [0, T]
    np.testing.assert_array_equal(got, np.stack([np.full(T, 1 << 32), np.arange(T), np.arange(T) + 1], 1))
