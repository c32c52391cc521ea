"""Decoding at the edges of the token window (the tokens since the last multiple of W = 8, 16 or 32, by the batch's
size, are kept as rows; the step that opens a window merges the last one): states of few levels,
whose window is shorter than W, sequences around one and several merges, a gate that resets the
state, decays under which levels vanish, the kernels with 64 rows of d_v per workgroup (large batches)
and a state copied in the middle of a window.  References and bars are those of test_gpu_decode.py and test_gpu_gdn_decode.py:
the float64 oracle, normalised max error 1e-4 (fp32) and 2e-2 (bf16)."""

import numpy as np
import pytest

from oracle import fenwick, gdn, mamba2
from synthetic import WORKLOADS, generate
from tests.gpu_util import rel_err, to_dev

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}
DIST = {"mamba2": "slow", "gdn": "gdn_slow"}


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_04761_amd  # noqa: F401


def inputs(variant, dtype, d, T, H=3, seed=0):
    w = WORKLOADS["ll_gdn_bf16_T8192" if variant == "gdn" else "ll_mamba2_bf16_T65536"]
    return generate(w.with_(dtype=dtype, B=1, H=H, T=T, dk=d[0], dv=d[1], C=16, dist=DIST[variant], seed=seed + T))


class Decoder:
    """One state fed token by token with the rows of x."""

    def __init__(self, variant, x, dtype, L, rep=1):
        import torch
        import paper_2506_04761_amd as ll
        self.ll, self.torch, self.variant, self.L = ll, torch, variant, L
        rows = lambda n, dt: to_dev(np.repeat(x[n][0], rep, axis=1), dt).unsqueeze(1)  # [T, 1, H rep, ...]
        self.a = {n: rows(n, dtype) for n in ("q", "k", "v")}
        self.a.update({n: rows(n, "f32") for n in ("log_alpha", "lam", "beta") if n in x})
        T, B, H, dk = self.a["q"].shape
        dv = self.a["v"].shape[-1]
        self.state = torch.full((ll.ll_decode_state_bytes(B, H, dk, dv, L),), 0xFF, dtype=torch.uint8, device="cuda")
        init = ll.ll_gdn_decode_init if variant == "gdn" else ll.ll_mamba2_decode_init
        init(self.state, B, H, dk, dv, L, self.a["q"].dtype)

    def feed(self, t0, t1, state=None):
        state = self.state if state is None else state
        outs = []
        for t in range(t0, t1):
            y = {n: z[t] for n, z in self.a.items()}
            if self.variant == "gdn":
                o = self.ll.ll_gdn_decode_step(y["q"], y["k"], y["v"], y["log_alpha"], y["beta"], y["lam"], state, t, self.L)
            else:
                o = self.ll.ll_mamba2_decode_step(y["q"], y["k"], y["v"], y["log_alpha"], y["lam"], state, t, self.L)
            outs.append(o[0].float())
        self.torch.cuda.synchronize()
        return self.torch.stack(outs).cpu().numpy().astype(np.float64)  # [T, H, d_v]


def reference(variant, x):
    if variant == "gdn":
        return gdn.recurrent(x["q"], x["k"], x["v"], x["log_alpha"], x["beta"], x["lam"])[0]
    return mamba2.recurrent(x["q"], x["k"], x["v"], x["log_alpha"], x["lam"])[0]


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
@pytest.mark.parametrize("dtype,d,Ts", [
    ("f32", (16, 16), (1, 2, 4, 8, 9, 16, 17, 64, 65)),
    ("f32", (64, 64), (1, 2, 16, 32, 33, 130)),
    ("bf16", (64, 64), (4, 32, 65)),
    ("bf16", (128, 64), (1, 8, 33, 97)),
    ("bf16", (128, 128), (2, 31, 32, 64, 161)),
])
def test_window_edges(variant, dtype, d, Ts):
    for T in Ts:
        x = inputs(variant, dtype, d, T)
        err = rel_err(Decoder(variant, x, dtype, fenwick.num_levels(T)).feed(0, T), reference(variant, x))
        print(f"{variant} {dtype} {d} T={T}: {err:.2e}", flush=True)
        assert err <= TOL[dtype], (T, err)


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
def test_reset_gate(variant):
    """log_alpha = -inf (alpha = 0) forgets everything before its token: inside a window, at the merge
    and after it."""
    x = inputs(variant, "f32", (64, 64), 100)
    for t in (20, 63, 64, 70):
        x["log_alpha"][:, t] = -np.inf
    ref = reference(variant, x)
    got = Decoder(variant, x, "f32", fenwick.num_levels(100)).feed(0, 100)
    assert np.isfinite(got).all() and rel_err(got, ref) <= TOL["f32"]


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
@pytest.mark.parametrize("d", [(64, 64), (128, 64), (128, 128)])
def test_large_batch(variant, d):
    """1026 heads take the 64-row workgroups, 3 the 16-row ones: each of the 342 copies of a head
    gives the same row bit for bit, within the bar of the oracle."""
    T = 70
    x = inputs(variant, "bf16", d, T)
    x = dict(x, lam=np.concatenate([x["lam"], np.ones(x["lam"].shape[:-1] + (1,), np.float32)], axis=-1))
    got = Decoder(variant, x, "bf16", x["lam"].shape[-1], rep=342).feed(0, T).reshape(T, 3, 342, d[1])
    assert (got == got[:, :, :1]).all()
    assert rel_err(got[:, :, 0], reference(variant, x)) <= TOL["bf16"]


@pytest.mark.parametrize("rep", [1, 11])
@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
def test_copied_state(variant, rep):
    """A state copied in the middle of a window continues like the original, and the original is not
    touched by the copy's steps."""
    x = inputs(variant, "bf16", (128, 128), 110)
    dec = Decoder(variant, x, "bf16", fenwick.num_levels(110), rep)
    dec.feed(0, 77)
    fork = dec.state.clone()
    a, b = dec.feed(77, 110, fork), dec.feed(77, 110)
    assert (a == b).all() and rel_err(b[:, ::rep], reference(variant, x)[77:]) <= TOL["bf16"]


@pytest.mark.parametrize("dtype,d,rep", [("f32", (16, 16), 1), ("bf16", (128, 128), 1), ("bf16", (128, 128), 400)])
def test_decayed_levels(dtype, d, rep):
    """Some heads decay so fast that their higher levels' scales reach zero (which are then not read), others
    not at all: 600 tokens, every position and head against the oracle."""
    T = 600
    x = inputs("mamba2", dtype, d, T)
    x["log_alpha"][:, :, 0] = -3.0
    x["log_alpha"][:, :, 1] = 0.0
    x["log_alpha"][:, 300:, 2] = -1.0  # the first half's levels vanish while the sequence runs
    got = Decoder("mamba2", x, dtype, fenwick.num_levels(T), rep).feed(0, T).reshape(T, 3, rep, d[1])
    ref = reference("mamba2", x)
    for h in range(3):
        assert rel_err(got[:, h, 0], ref[:, h]) <= TOL[dtype], h
    assert (got == got[:, :, :1]).all()


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
@pytest.mark.parametrize("dtype,d,rep", [
    ("bf16", (64, 64), 42),     # 126 heads: Gated DeltaNet keeps every level as a matrix
    ("bf16", (64, 64), 43),     # 129 heads: windows of 8 tokens
    ("f32", (16, 16), 342),     # 1026 heads: 8
    ("bf16", (128, 128), 42),   # 126 heads: 8, the most of this size
    ("bf16", (128, 128), 43),   # 129 heads: 16 tokens
    ("bf16", (128, 64), 100),   # 300 heads: 16
    ("f32", (64, 64), 200),     # 600 heads: 16, 16 rows of d_v per workgroup
    ("f32", (64, 64), 700),     # 2100 heads: 32 (Gated DeltaNet 16), 64 rows
    ("bf16", (64, 64), 1400),   # 4200 heads: 32
    ("bf16", (128, 128), 350),  # 1050 heads: 32
])
def test_window_lengths(variant, dtype, d, rep):
    """Every length of the window at its edges: a state too short for one, the first merges, some more tokens."""
    for T in (2, 17, 33, 100):
        x = inputs(variant, dtype, d, T)
        got = Decoder(variant, x, dtype, fenwick.num_levels(T), rep).feed(0, T).reshape(T, 3, rep, d[1])
        assert (got == got[:, :, :1]).all(), T
        assert rel_err(got[:, :, 0], reference(variant, x)) <= TOL[dtype], T


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
@pytest.mark.parametrize("rep", [1, 43, 200, 1400])  # every length of the window (Gated DeltaNet: and none)
def test_steps_of_both_types_on_one_state(variant, rep):
    """d = 64 is compiled for fp32 and bf16, and a state belongs to neither: steps of the two types in turn, with
    values that both hold exactly, give the sequence's rows, each within the bar of its output's type."""
    T = 100
    x = inputs(variant, "bf16", (64, 64), T)
    ref = reference(variant, x)
    dec = {dt: Decoder(variant, x, dt, fenwick.num_levels(T), rep) for dt in ("f32", "bf16")}
    order = ["f32" if t % 3 == 0 or 60 < t < 80 else "bf16" for t in range(T)]
    got = np.concatenate([dec[dt].feed(t, t + 1, dec["bf16"].state) for t, dt in enumerate(order)])
    got = got.reshape(T, 3, rep, 64)
    assert (got == got[:, :, :1]).all()
    for dt in ("f32", "bf16"):
        rows = [t for t in range(T) if order[t] == dt]
        err = rel_err(got[rows, :, 0], ref[rows])
        print(f"{variant} {dt} rows of a mixed sequence, {3 * rep} heads: {err:.2e}", flush=True)
        assert err <= TOL[dt]


@pytest.mark.parametrize("at,reset", [(3, 5), (10, 20), (10, 33), (31, 32), (31, 64), (40, 70)])
@pytest.mark.parametrize("name", ["k", "v"])
@pytest.mark.parametrize("rep", [1, 200, 700])  # every length of the window
def test_reset_drops_what_is_not_finite(at, reset, name, rep):
    """Mamba-2: after alpha = 0 the levels and the tokens before it are not read, so an infinity or a NaN among
    them ends there: the rows after the reset are those of the sequence without it."""
    T = 100
    x = inputs("mamba2", "f32", (64, 64), T)
    x["log_alpha"][:, reset] = -np.inf
    ref = reference("mamba2", x)
    x[name][0, at, 0, 5], x[name][0, at, 1, 7] = np.inf, np.nan
    got = Decoder("mamba2", x, "f32", fenwick.num_levels(T), rep).feed(0, T).reshape(T, 3, rep, 64)[:, :, 0]
    assert not np.isfinite(got[at, 0]).all() and not np.isfinite(got[at, 1]).all()
    assert np.isfinite(got[reset + 1:]).all()
    assert rel_err(got[reset + 1:], ref[reset + 1:]) <= TOL["f32"] and rel_err(got[:, 2], ref[:, 2]) <= TOL["f32"]


@pytest.mark.parametrize("variant", ["mamba2", "gdn"])
@pytest.mark.parametrize("dtype,d,rep", [("bf16", (128, 128), 1), ("bf16", (128, 64), 50), ("f32", (64, 64), 43), ("f32", (16, 16), 1)])
def test_rows_that_begin_at_any_element(variant, dtype, d, rep):
    """q, k and v one element past an aligned address: the same bits as from aligned ones."""
    import torch
    x = inputs(variant, dtype, d, 40)
    a, b = (Decoder(variant, x, dtype, fenwick.num_levels(40), rep) for _ in range(2))
    for n in ("q", "k", "v"):
        z = b.a[n]
        b.a[n] = torch.cat([z.new_zeros(1), z.flatten()])[1:].view(z.shape)
        assert b.a[n].data_ptr() % 16 == z.element_size()
    assert (a.feed(0, 40) == b.feed(0, 40)).all()
