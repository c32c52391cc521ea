"""Log-linear Gated DeltaNet by pairs of chunks (the unit of the WY kernel, the tree and the read-out) where
pairs can go wrong: an odd chunk count leaves the last pair half full, sequences of one or two chunks have
no tree and no read-out, and more pairs than compute units give the persistent workgroups a second turn for
some of them.  Sampled heads against the float64 quadratic form; bf16 inputs with fp32 accumulation, normalised max-abs error <= 2e-2 as for the forward."""

import numpy as np
import pytest

from oracle import gdn
from synthetic import WORKLOADS, generate
from tests.gpu_util import rel_err, run_gdn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,chunks", [
    (1, 300, 1),  # one chunk each: a workgroup takes two sequences
    (1, 515, 1),  # 258 of them on 256 compute units, the last with one sequence
    (3, 1, 1),
    (1, 300, 2),  # one full pair each, 300 on 256 compute units
    (2, 70, 3),   # 280 pairs: full and half-full ones in turn
    (3, 40, 5),   # 360 pairs, a tree of one level over an odd pair count
    (1, 90, 6),   # 270 full pairs
])
@pytest.mark.parametrize("with_lambda", [True, False])
def test_pairs(d, B, H, chunks, with_lambda):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = WORKLOADS["ll_gdn_bf16_T8192"].with_(B=B, H=H, T=64 * chunks, dk=d, dv=d, dist="gdn_slow", seed=700 + H)
    x = generate(w)
    got = run_gdn(x, 64, with_lambda=with_lambda)
    assert np.isfinite(got).all()
    for h in (0, H // 2, H - 1):
        y = {n: a[:, :, h:h + 1] for n, a in x.items()}
        lam = y["lam"] if with_lambda else np.ones_like(y["lam"])
        ref = gdn.quadratic(y["q"], y["k"], y["v"], y["log_alpha"], y["beta"], lam)
        err = rel_err(got[:, :, h:h + 1], ref)
        print(f"GDN pairs d={d} B={B} H={H} chunks={chunks} head {h} lambda={with_lambda}: rel err {err:.3e}", flush=True)
        assert err <= 2e-2, err


@pytest.mark.parametrize("d", [64, 128])
def test_gates_above_one_grow(d):
    """log_alpha > 0 is the caller's to avoid, but is computed like any other: against the oracle, with the
    growth over the sequence kept within a factor of e^2.6."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = WORKLOADS["ll_gdn_bf16_T8192"].with_(B=1, H=2, T=320, dk=d, dv=d, dist="gdn_slow", seed=31)
    x = generate(w)
    x["log_alpha"] = np.abs(np.random.default_rng(d).standard_normal(x["log_alpha"].shape)).astype(np.float32) * 0.01
    ref = gdn.quadratic(x["q"], x["k"], x["v"], x["log_alpha"], x["beta"], x["lam"])
    err = rel_err(run_gdn(x, 64), ref)
    print(f"GDN d={d} growing gates: rel err {err:.3e}", flush=True)
    assert err <= 2e-2


@pytest.mark.parametrize("at", [3, 63, 64, 200])
def test_nan_gate_reaches_every_later_row(at):
    """A gate that is not a number makes its token's row and all later ones of the head NaN, and no other head's."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = generate(WORKLOADS["ll_gdn_bf16_T8192"].with_(B=1, H=2, T=320, dk=64, dv=64, dist="gdn_slow", seed=32))
    x["log_alpha"][0, at, 1] = np.nan
    o = run_gdn(x, 64)
    assert np.isnan(o[0, at:, 1]).all() and np.isfinite(o[0, :, 0]).all()
