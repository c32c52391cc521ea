"""The backward with shared query/key heads at sizes where, for d_k > d_v, one workgroup takes a block of heads
(at least 1024 workgroups left, no nearly empty last round of 512): against the backward on q and k repeated to every head, its dq and dk summed over
each group.  Every head's dq and dk is rounded to bf16 there (relative 2^-9 each) and the sums here
once, so the two differ by at most about 1e-2 of the largest entry; dv, dlog_alpha and dlambda share their
arithmetic up to the order of fp32 sums (dlog_alpha: suffix sums of differences that nearly cancel)."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("B,H,Hqk,T", [
    (2, 64, 2, 2112),   # 17 tiles, the last half full: one head at a time (1088 workgroups are 2.1 rounds)
    (2, 64, 32, 2112),
    (2, 64, 2, 1984),   # 16 tiles, the last half full: blocks of 2 of 32 heads, summed at the end
    (2, 64, 32, 1984),  # the block is the whole group: dk written directly
    (1, 96, 1, 4096),   # blocks of 3 heads
])
def test_head_blocks_match_repeated_heads(B, H, Hqk, T, dk, dv):
    import torch
    import paper_2506_04761_amd as ll
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T + H + Hqk)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    G = H // Hqk
    q, k = ((rnd(B, T, Hqk, dk) / dk ** 0.5).bfloat16() for _ in range(2))
    v, do = (rnd(B, T, H, dv) / dv ** 0.5).bfloat16(), rnd(B, T, H, dv).bfloat16()
    la = -torch.nn.functional.softplus(rnd(B, T, H) - 3)
    lam = torch.nn.functional.softplus(rnd(B, T, H, ll.ll_num_levels(T)))
    got = ll.ll_mamba2_bwd(q, k, v, la, lam, do, 64)
    rep = lambda x: x.repeat_interleave(G, dim=2)
    ref = ll.ll_mamba2_bwd(rep(q), rep(k), v, la, lam, do, 64)
    fold = lambda x: x.double().reshape(B, T, Hqk, G, dk).sum(3)
    for name, a, b, tol in (("dq", got[0], fold(ref[0]), 1e-2), ("dk", got[1], fold(ref[1]), 1e-2),
                            ("dv", got[2], ref[2].double(), 1e-6), ("dlog_alpha", got[3], ref[3].double(), 1e-3),
                            ("dlambda", got[4], ref[4].double(), 1e-6)):
        err = float((a.double() - b).abs().max() / b.abs().max())
        print(f"{name}: {err:.2e}", flush=True)
        assert err <= tol, (name, err)
        if dk == dv and name in ("dv", "dlog_alpha", "dlambda"):  # one head per workgroup: the same operations
            assert torch.equal(a.double(), b), name


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("B,H,Hqk,T", [
    (8, 64, 1, 1984),  # blocks of 8 heads, the last tile half full
    (1, 96, 1, 4096),  # blocks of 3 heads
])
def test_heads_of_a_block_are_independent(B, H, Hqk, T, dk, dv):
    """dv, dlog_alpha and dlambda belong to one head: what a head of its block holds, be it 1e5 times as
    large or not finite, does not change a bit of the others'.  And each head's dlog_alpha, of scales
    from 1 to 1e4 within a block, against the backward that gives every head its own workgroup, on the
    head's own scale.  The two sum the same bf16 products in another order, so each term of a suffix sum
    differs by some 2^-23 of its parts q . dq and k . dk: up to 2^-23 sqrt(4096) = 8e-6 of the parts, which
    are a few times dlog_alpha's largest entry at most (seen: 4e-6 of that)."""
    import torch
    import paper_2506_04761_amd as ll
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T + H + dv)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = ((rnd(B, T, Hqk, dk) / dk ** 0.5).bfloat16() for _ in range(2))
    v, do = (rnd(B, T, H, dv) / dv ** 0.5).bfloat16(), rnd(B, T, H, dv).bfloat16()
    la = -torch.exp(torch.linspace(-7, 0, H, device="cuda")) * torch.exp(0.5 * rnd(B, T, H))
    lam = torch.nn.functional.softplus(rnd(B, T, H, ll.ll_num_levels(T)))
    loud = torch.arange(H, device="cuda") % 4 == 0
    base = ll.ll_mamba2_bwd(q, k, v, la, lam, do, 64)
    for value in ("scaled", "inf", "nan"):
        d = do.clone()
        if value == "scaled":
            d[:, :, loud] *= 1e5
        else:
            d[:, T // 3, loud] = float(value)
        got = ll.ll_mamba2_bwd(q, k, v, la, lam, d, 64)
        for name, a, b in (("dv", got[2], base[2]), ("dlog_alpha", got[3], base[3]), ("dlambda", got[4], base[4])):
            assert torch.equal(a[:, :, ~loud], b[:, :, ~loud]), (value, name)
    d = do * (10.0 ** (torch.arange(H, device="cuda") * 7 % 5))[:, None].bfloat16()
    got = ll.ll_mamba2_bwd(q, k, v, la, lam, d, 64)[3].double()
    rep = lambda x: x.repeat_interleave(H // Hqk, dim=2)
    ref = ll.ll_mamba2_bwd(rep(q), rep(k), v, la, lam, d, 64)[3].double()
    err = (got - ref).abs().amax(dim=(0, 1)) / ref.abs().amax(dim=(0, 1))
    print(f"dlog_alpha per head: {float(err.max()):.2e} (head {int(err.argmax())})", flush=True)
    assert float(err.max()) <= 5e-5


@pytest.mark.parametrize("dk,dv", [(128, 64)])
@pytest.mark.parametrize("B,H,Hqk,T", [
    (16, 64, 1, 256),  # blocks of 2 heads: 32 rows of dk summed at the end
    (16, 64, 1, 960),  # blocks of 8 heads, the last tile half full
])
def test_dk_is_no_further_from_float64_than_a_sum_of_rounded_heads(B, H, Hqk, T, dk, dv):
    """dk against float64: summing blocks of heads in fp32 takes roundings to bf16 out, so its error (2-norm)
    is below that of the sum of every head's dk rounded to bf16."""
    import torch
    import paper_2506_04761_amd as ll
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T + dv)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = ((rnd(B, T, Hqk, dk) / dk ** 0.5).bfloat16() for _ in range(2))
    v, do = (rnd(B, T, H, dv) / dv ** 0.5).bfloat16(), rnd(B, T, H, dv).bfloat16()
    la = -torch.exp(torch.linspace(-7, 0, H, device="cuda")) * torch.exp(0.5 * rnd(B, T, H))
    lam = torch.nn.functional.softplus(rnd(B, T, H, ll.ll_num_levels(T)))
    got = ll.ll_mamba2_bwd(q, k, v, la, lam, do, 64)[1].double()
    rep = lambda x: x.repeat_interleave(H // Hqk, dim=2)
    heads = ll.ll_mamba2_bwd(rep(q), rep(k), v, la, lam, do, 64)[1]
    per_head = heads.float().reshape(B, T, Hqk, H // Hqk, dk).sum(3).bfloat16().double()
    pos = torch.arange(T, device="cuda")
    level = torch.frexp((pos[:, None] ^ pos).double())[1].long()
    exact = torch.zeros_like(got)
    for h in range(H):
        cum = la[:, :, h].double().cumsum(1)
        w = torch.exp((cum[:, :, None] - cum[:, None]).masked_fill(pos[:, None] < pos, -torch.inf))
        w *= lam[:, :, h].double().gather(2, level.expand(B, -1, -1).clamp(max=lam.shape[-1] - 1))
        w *= do[:, :, h].double() @ v[:, :, h].double().transpose(1, 2).contiguous()
        exact[:, :, h // (H // Hqk)] += w.transpose(1, 2).contiguous() @ q[:, :, h // (H // Hqk)].double()
    err = lambda x: float((x - exact).norm() / exact.norm())
    print(f"dk: {err(got):.3e}, heads rounded one by one {err(per_head):.3e}", flush=True)
    assert err(got) < 0.95 * err(per_head)


@pytest.mark.parametrize("Hqk", [1, 16, 32])  # dq and dk from k_group_sum; dk from blocks of 2 heads; the same, nothing to sum
def test_shared_gradients_begin_at_any_element(Hqk):
    """dq and dk of shared heads one element past an aligned address: the same bits as at an aligned one."""
    import torch
    import paper_2506_04761_amd as ll
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, H, T, dk, dv = 2, 64, 1984, 128, 64
    g = torch.Generator(device="cuda").manual_seed(Hqk)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = ((rnd(B, T, Hqk, dk) / dk ** 0.5).bfloat16() for _ in range(2))
    v, do = (rnd(B, T, H, dv) / dv ** 0.5).bfloat16(), rnd(B, T, H, dv).bfloat16()
    la = -torch.nn.functional.softplus(rnd(B, T, H) - 3)
    lam = torch.nn.functional.softplus(rnd(B, T, H, ll.ll_num_levels(T)))
    ref = ll.ll_mamba2_bwd(q, k, v, la, lam, do, 64)
    dq, dkk = (torch.zeros(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view(q.shape) for _ in range(2))
    got = ll.ll_mamba2_bwd(q, k, v, la, lam, do, 64, grads=(dq, dkk, *(torch.empty_like(r) for r in ref[2:])))
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
