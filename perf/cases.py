"""The work that users of this library have it do, as cases to be timed and checked.

Each case is one pass through the public entry points of paper_2506_04761_amd: a forward pass
(ll_mamba2_fwd, ll_mamba2_fwd_grouped, ll_gdn_fwd), a training step (log_linear_mamba2 under
autograd), or a run of decoded tokens that continues a cached prompt (ll_mamba2_decode_step,
ll_gdn_decode_step).  Sizes are those of the workload table in synthetic/gen.py, their smaller and
ragged relatives, and generic ones.

`exact` computes the same outputs in float64 with plain torch, from the definitions alone.
"""

import math

import torch

import paper_2506_04761_amd as ll

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
NAMES = {"f32": ll.LL_F32, "bf16": ll.LL_BF16}


# ------------------------------------------------------------------------------------ the cases

def _fwd(name, B, H, T, dk, dv, dtype="bf16", C=64, Hqk=0, lam=True):
    c = {"kind": "fwd", "dtype": dtype, "B": B, "H": H, "Hqk": Hqk or H, "T": T, "dk": dk, "dv": dv, "C": C,
         "lam": lam}
    return {"name": name, **c} if name else c


def _train(name, B, H, T, dk, dv, dtype="bf16", C=64, Hqk=0):
    c = {"kind": "train", "dtype": dtype, "B": B, "H": H, "Hqk": Hqk or H, "T": T, "dk": dk, "dv": dv, "C": C,
         "lam": True}
    return {"name": name, **c} if name else c


def _gdn(name, B, H, T, d, lam=True):
    c = {"kind": "gdn", "dtype": "bf16", "B": B, "H": H, "Hqk": H, "T": T, "dk": d, "dv": d, "C": 64, "lam": lam}
    return {"name": name, **c} if name else c


def _decode(name, kind, B, H, dk, dv, t0, n, L, dtype="bf16", lam=True):
    c = {"kind": kind, "dtype": dtype, "B": B, "H": H, "dk": dk, "dv": dv, "t0": t0, "n": n, "L": L, "lam": lam}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one short prompt through one layer: latency and launches
        _fwd("fwd_short", 1, 8, 320, 64, 64),
        # a small batch of medium prompts (workload ll_mamba2_bf16_T2048)
        _fwd("fwd_2k", 2, 8, 2048, 64, 64),
        # a layer's prefill at full batch (workload ll_mamba2_bf16_T8192)
        _fwd("fwd_8k", 4, 32, 8192, 128, 64),
        # the headline: one long context (workload ll_mamba2_bf16_T65536)
        _fwd("fwd_64k", 1, 16, 65536, 128, 128),
        # the float32 path, a ragged length (the last tile is half full)
        _fwd("fwd_f32", 2, 8, 1984, 64, 64, dtype="f32"),
        # forward and backward at a ragged medium length
        _train("train_4k", 1, 12, 4032, 128, 128),
        # forward and backward of the paper's kernel benchmark: one query/key head for all 48 heads
        # (workload ll_mamba2_mva_bwd_bf16_T16384)
        _train("train_mva_16k", 2, 48, 16384, 128, 64, Hqk=1),
        # forward and backward of the long context (workload ll_mamba2_bwd_bf16_T65536)
        _train("train_64k", 1, 16, 65536, 128, 128),
        # Gated DeltaNet prefill (workload ll_gdn_bf16_T8192)
        _gdn("gdn_8k", 2, 16, 8192, 128),
        # Gated DeltaNet, a small layer at a ragged length
        _gdn("gdn_2k", 1, 8, 1984, 64),
        # 64 sequences of 16 heads decode 32 tokens from a cached prompt (the sizes of workloads
        # ll_mamba2_decode_bf16_T8192 and ll_gdn_decode_bf16_T8192)
        _decode("decode", "decode", 64, 16, 128, 128, 3000, 32, 14),
        _decode("gdn_decode", "gdn_decode", 64, 16, 128, 128, 3000, 32, 14),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "train", "gdn", "decode", "gdn_decode"])
    dk, dv = rng.choice([(64, 64), (128, 64), (128, 128)])
    if kind in ("decode", "gdn_decode"):
        # few to many sequences, from the first token to a few thousand tokens in
        B, H = _log_int(rng, 1, 64), rng.choice([3, 4, 8, 12, 16])
        t0, n = rng.choice([0, rng.randrange(1, 200), rng.randrange(200, 4000)]), rng.randrange(9, 33)
        dtype = "bf16"
        if rng.random() < 0.2:
            dtype, dk, dv = "f32", 64, 64
        L = (t0 + n - 1).bit_length() + 1 + rng.randrange(0, 3)
        return _decode(None, kind, B, H, dk, dv, t0, n, L, dtype=dtype, lam=rng.random() < 0.8)
    # 64-token chunks per sequence: one to 1024
    chunks = _log_int(rng, 1, {"fwd": 1024, "train": 256, "gdn": 128}[kind])
    cap = (1 << (20 if kind != "gdn" else 18)) // (64 * chunks)  # sequence-heads at this length
    BH = _log_int(rng, 1, max(1, min(cap, 128)))
    B = rng.choice([1, 1, 2, 3])
    H = max(1, BH // B)
    if kind == "gdn":
        return _gdn(None, B, H, 64 * chunks, rng.choice([64, 128]), lam=rng.random() < 0.8)
    Hqk = rng.choice([d for d in range(1, H + 1) if H % d == 0]) if rng.random() < 0.3 else H
    if rng.random() < 0.15:
        # the float32 path, at sizes where its time is not above the long bf16 cases
        d, C = rng.choice([(16, 16), (64, 64)])
        T = C * min(chunks, 64)
        make = _fwd if kind == "fwd" else _train
        return make(None, B, min(H, 16), T, d, d, dtype="f32", C=C)
    if kind == "train":
        return _train(None, B, H, 64 * chunks, dk, dv, Hqk=Hqk)
    return _fwd(None, B, H, 64 * chunks, dk, dv, Hqk=Hqk, lam=rng.random() < 0.8)


# ------------------------------------------------------------------------------------ inputs

def _gates(g, shape, H):
    """Log-gates -rate exp(noise / 2) as a Mamba-2 layer has them: the heads' rates spread from 0.001 to 1
    per token, varying from token to token.  Heads remember between one and a thousand tokens, so
    every level carries weight."""
    rate = torch.exp(torch.linspace(math.log(0.001), 0.0, H, device="cuda"))
    return -rate * torch.exp(0.5 * torch.randn(shape, generator=g, device="cuda"))


def _inputs(case, seed):
    """The tensors of one pass, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    kind, B, H, dk, dv = case["kind"], case["B"], case["H"], case["dk"], case["dv"]

    def rnd(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    x = {}
    if kind in ("decode", "gdn_decode"):
        N, n = case["t0"] + case["n"], case["n"]  # token-major: one row per step
        x["q"] = (rnd(n, B, H, dk) / math.sqrt(dk)).to(dt)
        k, vshape, gshape, L = rnd(N, B, H, dk), (N, B, H, dv), (N, B, H), case["L"]
        lshape = (n, B, H, L)
    else:
        T = case["T"]
        L = ll.ll_num_levels(T)
        x["q"] = (rnd(B, T, case["Hqk"], dk) / math.sqrt(dk)).to(dt)
        k, vshape, gshape, lshape = rnd(B, T, case["Hqk"], dk), (B, T, H, dv), (B, T, H), (B, T, H, L)
    if kind in ("gdn", "gdn_decode"):
        k = k / k.norm(dim=-1, keepdim=True)
        x["beta"] = torch.sigmoid(rnd(*gshape))
    else:
        k = k / math.sqrt(dk)
    x["k"] = k.to(dt)
    x["v"] = (rnd(*vshape) / math.sqrt(dv)).to(dt)
    x["log_alpha"] = _gates(g, gshape, H)
    x["lam"] = torch.nn.functional.softplus(rnd(*lshape)) if case["lam"] else None
    if kind == "train":
        x["d_o"] = rnd(*vshape).to(dt)
    return x


def _step(kind, x, t, i, state, L, out=None):
    """Token t of the sequence; its query and level weights are row i, or none of use if i is None."""
    q = x["k"][t] if i is None else x["q"][i]
    lam = None if i is None or x["lam"] is None else x["lam"][i]
    if kind == "decode":
        return ll.ll_mamba2_decode_step(q, x["k"][t], x["v"][t], x["log_alpha"][t], lam, state, t, L, out=out)
    return ll.ll_gdn_decode_step(q, x["k"][t], x["v"][t], x["log_alpha"][t], x["beta"][t], lam, state, t, L, out=out)


def prepare(case, seed):
    x = _inputs(case, seed)
    kind, B, H, dk, dv = case["kind"], case["B"], case["H"], case["dk"], case["dv"]
    st = {"case": case, "x": x}
    if kind in ("fwd", "gdn"):
        # a program that calls a layer again and again keeps its workspace
        variant = ll.LL_GDN if kind == "gdn" else ll.LL_MAMBA2
        need = ll.ll_workspace_size(variant, NAMES[case["dtype"]], B, case["T"], H, dk, dv, case["C"], case["lam"])
        st["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    elif kind == "train":
        for n in ("q", "k", "v", "log_alpha", "lam"):
            x[n].requires_grad_(True)
    else:
        # the prompt's state, cached; each pass works on its own copy of it
        L, dt = case["L"], DTYPES[case["dtype"]]
        prefix = torch.empty(ll.ll_decode_state_bytes(B, H, dk, dv, L), dtype=torch.uint8, device="cuda")
        init = ll.ll_mamba2_decode_init if kind == "decode" else ll.ll_gdn_decode_init
        init(prefix, B, H, dk, dv, L, dt)
        o = torch.empty((B, H, dv), dtype=dt, device="cuda")
        for t in range(case["t0"]):
            _step(kind, x, t, None, prefix, L, out=o)
        st["prefix"], st["state"] = prefix, torch.empty_like(prefix)
    return st


def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "fwd":
        fwd = ll.ll_mamba2_fwd if case["Hqk"] == case["H"] else ll.ll_mamba2_fwd_grouped
        return fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["lam"], case["C"], workspace=state["workspace"])
    if kind == "gdn":
        return ll.ll_gdn_fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["beta"], x["lam"], case["C"],
                             workspace=state["workspace"])
    if kind == "train":
        leaves = [x[n] for n in ("q", "k", "v", "log_alpha", "lam")]
        o = ll.log_linear_mamba2(*leaves, case["C"])
        return [o.detach(), *torch.autograd.grad(o, leaves, x["d_o"])]
    # decoding: fork the cached prompt, then one call per token
    state["state"].copy_(state["prefix"])
    return [_step(kind, x, case["t0"] + i, i, state["state"], case["L"]) for i in range(case["n"])]


# ------------------------------------------------------------------------------------ work

def work(case):
    """Bytes: inputs read once, outputs written once.  Flops: the chunkwise algorithm's, a
    multiplication and an addition each one."""
    kind, B, H, dk, dv = case["kind"], case["B"], case["H"], case["dk"], case["dv"]
    e = 2 if case["dtype"] == "bf16" else 4
    if kind in ("decode", "gdn_decode"):
        # the forked state is read and written once; every step reads its tokens, writes its outputs
        # and reads every level that holds tokens, a level of few tokens as their rows of k and v
        def levels(t):
            return sum(min((1 << b) * (dk + dv) * e, dk * dv * 4) for b in range(t.bit_length()) if t >> b & 1)
        L = case["L"] if case["lam"] else 0
        steps = range(case["t0"], case["t0"] + case["n"])
        tok = (2 * dk + 2 * dv) * e + 4 * (L + (2 if kind == "gdn_decode" else 1))
        per_level = 2 if kind == "decode" else 4
        flops = sum((per_level * bin(t).count("1") + 2) * dk * dv for t in steps)
        return {"bytes": B * H * (2 * levels(case["t0"]) + sum(levels(t) + tok for t in steps)), "flops": B * H * flops}
    T, C, Hqk = case["T"], case["C"], case["Hqk"]
    lv = max(0.0, math.log2(T / C))
    L = ll.ll_num_levels(T) if case["lam"] else 0
    qk, vo, gate = 2 * B * T * Hqk * dk * e, 2 * B * T * H * dv * e, 4 * B * T * H * (1 + L)
    per = 2 * C * (dk + dv) + 2 * dk * dv + (dk * dv * lv if case["lam"] else 2 * dk * dv)
    if kind == "gdn":
        # K K^T and the triangular solve of a chunk, the state's correction, on top of the above
        per += C * dk + C * (dk + dv) + 2 * dk * dv
        gate += 4 * B * T * H
    if kind == "train":
        per += 2 * C * (3 * dk + 2 * dv) + 2 * dk * dv + 5 * dk * dv * lv
        # forward's bytes, then q, k, v, gates, lambda, dO in and their gradients out
        return {"bytes": qk + vo + gate + 2 * qk + 3 * vo // 2 + 2 * gate, "flops": B * H * T * per}
    return {"bytes": qk + vo + gate, "flops": B * H * T * per}


def tolerance(case):
    # about four times the relative error seen against float64 on such cases: 3e-3 (Mamba-2), 4e-3
    # (Gated DeltaNet), 7e-7 (float32, decoding).  Of a training step the gradient of the log-gates
    # is the furthest off, a sum over all later tokens of differences that nearly cancel: 2e-2 at a
    # few thousand tokens, 3e-2 at 65536.
    f32 = case["dtype"] == "f32"
    if case["kind"] == "train":
        return {"rel": 2e-5 if f32 else 0.12 if case["T"] > 16384 else 0.08}
    return {"rel": 3e-6 if f32 else 1.6e-2}


# ------------------------------------------------------------------------------------ float64

def _bits(x):
    """bit_length of whole numbers: the Fenwick level of (t, s) is that of t xor s."""
    return torch.frexp(x.double())[1].long()


def _exact_mamba2(case, x):
    """O, and for a training step the gradients of sum(O dO), from the quadratic form, a block of rows
    and a group of heads at a time."""
    B, H, T, dk, dv, Hqk = (case[n] for n in ("B", "H", "T", "dk", "dv", "Hqk"))
    G, dev, f = H // Hqk, "cuda", torch.float64
    R = 256
    step = max(R, -(-T // 16))
    group = max(1, min(B * H, (1 << 27) // (R * max(T, R))))
    heads = lambda a: a.transpose(1, 2).reshape(B * H, T, *a.shape[3:])  # [B, T, H, ...] -> [BH, T, ...]
    rep = lambda a: heads(a.repeat_interleave(G, dim=2))
    q, k, v, la = rep(x["q"].detach()), rep(x["k"].detach()), heads(x["v"].detach()), heads(x["log_alpha"].detach())
    lam = None if x["lam"] is None else heads(x["lam"].detach())
    train = case["kind"] == "train"
    do = heads(x["d_o"]) if train else None
    L = ll.ll_num_levels(T)
    o = torch.empty((B * H, T, dv), dtype=f, device=dev)
    if train:
        gq, gk = (torch.zeros((B * H, T, dk), dtype=f, device=dev) for _ in range(2))
        gv, gla = torch.zeros((B * H, T, dv), dtype=f, device=dev), torch.empty((B * H, T), dtype=f, device=dev)
        glam = torch.zeros((B * H, T, L), dtype=f, device=dev)
    pos = torch.arange(T, device=dev)
    for h in range(0, B * H, group):
        s = slice(h, min(h + group, B * H))
        qs, ks, vs = q[s].to(f), k[s].to(f), v[s].to(f)
        cum = la[s].to(f).cumsum(1)
        if train:
            ds = do[s].to(f)
        for r in range(0, T, R):
            # keys in sixteenths of the sequence (few different sizes to allocate); those after the rows weigh 0
            e, n = min(r + R, T), min(T, -(-(r + R) // step) * step)
            # levels: one per R-token block of keys left of the diagonal block, one per pair inside it
            inner = _bits(pos[r:e, None] ^ pos[None, r:e])
            outer = _bits((r // R) ^ (pos[:r] // R)) + R.bit_length() - 1
            decay = cum[:, r:e, None] - cum[:, None, :n]
            decay.masked_fill_(pos[r:e, None] < pos[None, :n], -math.inf).exp_()
            w = decay
            if lam is not None:
                lm = lam[s, r:e].to(f)
                w = torch.zeros_like(decay)
                w[..., :r] = lm[..., outer]
                w[..., r:e] = lm.gather(2, inner.clamp(max=L - 1).expand(lm.shape[0], -1, -1))
                w *= decay
            p = qs[:, r:e] @ ks[:, :n].transpose(1, 2)
            if not train:
                o[s, r:e] = p.mul_(w) @ vs[:, :n]
                continue
            m = ds[:, r:e] @ vs[:, :n].transpose(1, 2)
            decay.mul_(p).mul_(m)  # a pair's share of its level's gradient
            p.mul_(w)
            m.mul_(w)
            o[s, r:e], gq[s, r:e] = p @ vs[:, :n], m @ ks[:, :n]
            gk[s, :n] += m.transpose(1, 2) @ qs[:, r:e]
            gv[s, :n] += p.transpose(1, 2) @ ds[:, r:e]
            a = 0
            for lv, c in zip(*(y.tolist() for y in outer.unique_consecutive(return_counts=True))):
                glam[s, r:e, lv] = decay[..., a:a + c].sum(2)
                a += c
            for lv in range(min(L, R.bit_length())):
                glam[s, r:e, lv] = (decay[..., r:e] * (inner == lv)).sum(2)
        if train:
            d = (qs * gq[s]).sum(2) - (ks * gk[s]).sum(2)
            gla[s] = d.flip(1).cumsum(1).flip(1)
    back = lambda a: a.reshape(B, H, T, *a.shape[2:]).transpose(1, 2).contiguous()
    if not train:
        return back(o)
    share = lambda a: back(a).reshape(B, T, Hqk, G, dk).sum(3)
    return [back(o), share(gq), share(gk), back(gv), back(gla), back(glam)]


def _exact_delta(q, k, v, log_alpha, beta, lam, first):
    """Gated DeltaNet outputs of the queries q [N, n, dk] at positions first, first + 1, ...:
    o_t = sum_s lambda_t^(l) beta_s (k_s . A_{s+1} ... A_t q_t) v_s with A = alpha (I - beta k k^T),
    the transitions applied to all queries together from the last token to the first."""
    f = torch.float64
    N, n, dk = q.shape
    T = first + n
    q, alpha = q.to(f).clone(), torch.exp(log_alpha.to(f))
    o = torch.zeros((N, n, v.shape[-1]), dtype=f, device=q.device)
    pos = torch.arange(first, T, device=q.device)
    for s in range(T - 1, -1, -1):
        i = max(0, s - first)  # the queries at s and after it
        ks, vs, bs = k[:, s].to(f), v[:, s].to(f), beta[:, s].to(f)
        w = bs[:, None] * torch.bmm(q[:, i:], ks[:, :, None])[..., 0]
        u = w if lam is None else w * lam[:, i:].gather(2, _bits(pos[i:] ^ s)[None, :, None].expand(N, -1, 1))[..., 0]
        o[:, i:].baddbmm_(u[..., None], vs[:, None, :])
        q[:, i:].baddbmm_(w[..., None], ks[:, None, :], alpha=-1.0)
        q[:, i:] *= alpha[:, s, None, None]
    return o


def exact(case, seed):
    x = _inputs(case, seed)
    kind, B, H = case["kind"], case["B"], case["H"]
    if kind in ("fwd", "train"):
        return _exact_mamba2(case, x)
    if kind == "gdn":
        heads = lambda a: None if a is None else a.transpose(1, 2).reshape(B * H, case["T"], *a.shape[3:])
        o = _exact_delta(*(heads(x[n]) for n in ("q", "k", "v", "log_alpha", "beta", "lam")), 0)
        return o.reshape(B, H, case["T"], -1).transpose(1, 2).contiguous()
    t0, n, BH = case["t0"], case["n"], B * H
    heads = lambda a: None if a is None else a.reshape(a.shape[0], BH, *a.shape[3:]).transpose(0, 1)
    q, k, v, la, lam = (heads(x[m]) for m in ("q", "k", "v", "log_alpha", "lam"))
    if kind == "gdn_decode":
        o = _exact_delta(q, k, v, la, heads(x["beta"]), lam, t0)
    else:
        f, pos = torch.float64, torch.arange(t0 + n, device="cuda")
        o = torch.empty((BH, n, case["dv"]), dtype=f, device="cuda")
        causal, lev = pos[t0:, None] >= pos[None], _bits(pos[t0:, None] ^ pos[None]).clamp(max=case["L"] - 1)
        for h in range(0, BH, 128):
            s = slice(h, h + 128)
            cum = la[s].to(f).cumsum(1)
            w = torch.exp(torch.where(causal, cum[:, t0:, None] - cum[:, None], -math.inf))
            if lam is not None:
                w = w * lam[s].to(f).gather(2, lev.expand(w.shape[0], -1, -1))
            o[s] = (w * (q[s].to(f) @ k[s].to(f).transpose(1, 2).contiguous())) @ v[s].to(f)
    return [o[:, i].reshape(B, H, -1) for i in range(n)]
