"""The single-pass forward's decay gaps on both sides of the length up to which a tile scans the tile
totals itself (64 tiles = 8192 tokens) instead of reading block sums: 63, 64 and 65 tiles, ragged ends
and short sequences, gates slow enough for every level to weigh, against the float64 oracle (bf16 bar
2e-2).  The forward in a backward-sized workspace forms the block sums at every length: same bar."""

import numpy as np
import pytest

from oracle import mamba2
from synthetic import WORKLOADS, generate
from tests.gpu_util import device_inputs, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [64, 192, 256, 320, 8064, 8128, 8192, 8256, 8320])
def test_forward_around_scan_limit(T):
    import torch
    import paper_2506_04761_amd as ll
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = WORKLOADS["ll_mamba2_bf16_T2048"].with_(B=1, H=2, T=T, dist="slow", seed=300 + T)
    x = generate(w)
    rows = np.unique(np.concatenate([np.arange(max(0, T - 130), T), np.arange(0, T, 61)]))
    ref = mamba2.quadratic(x["q"], x["k"], x["v"], x["log_alpha"], x["lam"], rows=rows)
    d = device_inputs(x, "bf16")
    a = (d["q"], d["k"], d["v"], d["log_alpha"], d["lam"], 64)
    for ws in (None, ll.ll_mamba2_bwd_workspace(d["q"], d["v"], 64)):
        o = ll.ll_mamba2_fwd(*a, workspace=ws).float().cpu().numpy().astype(np.float64)
        assert rel_err(o[:, rows], ref) <= 2e-2
