"""GEMM tiles chosen by row count: whatever tile the library picks for a batch,
a record's hidden state has the bits that one forced 256x256 (FP32:
256x128) tile gives it
(every tile forms an output with the same MFMA sequence, so the tolerance is
zero).  Row counts lie on both sides of the tile edges (32, 64, 128, 192, 256)
and of the points where the choice changes."""
from __future__ import annotations

from dataclasses import replace

import numpy as np
import pytest

import synth
from synth.configs import BASE, LARGE
from tests.gpu_common import make_model, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    return torch


def _lengths(T):
    """Records of at most 512 tokens adding up to T, the last ones ragged."""
    L = []
    while T > 0:
        n = min(T, 512 if len(L) % 3 else 97)
        L.append(n)
        T -= n
    return np.asarray(L, np.int64)


@pytest.mark.parametrize("size,precision", [("base", "bf16"), ("large", "bf16"), ("large", "fp8"), ("base", "fp32")])
def test_default_tiles_equal_the_widest_tile(torch_dev, size, precision):
    import torch
    from paper_2606_15650_amd import api
    from paper_2606_15650_amd.pipeline import Pipeline
    cfg = replace(BASE if size == "base" else LARGE, n_layers=1, vocab=2000)
    scales = np.full(4, 2.0 ** -6, np.float32) if precision == "fp8" else None
    _, m = make_model(cfg, precision, 0, act_scales=scales)
    wide, name = {"bf16": (11, "256x256"), "fp8": (7, "256x256"), "fp32": (3, "256x128")}[precision]
    assert name in m.tile_configs()[wide]
    pl = Pipeline(m)
    rng = np.random.default_rng(3)
    for T in (1, 31, 33, 64, 65, 129, 257, 300, 449, 700, 1100, 2094, 3111, 4097, 6150, 9000, 12289, 16385):
        L = _lengths(T)
        cu = np.concatenate([[0], np.cumsum(L)]).astype(np.int32)

        class Batch:
            B, h_cu = len(L), cu
        db = Batch()
        db.T = T
        db.ids = torch.from_numpy(rng.integers(0, cfg.vocab, T).astype(np.int32)).cuda()
        db.cu = torch.from_numpy(cu).cuda()
        m.set_tiles([-1] * 4)
        got = pl.hidden(db, 1)
        m.set_tiles([wide] * 4)
        want = pl.hidden(db, 1)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(got).all())
        assert torch.equal(got, want), f"{T} rows"
    assert api.device_errors() == 0
    m.close()
