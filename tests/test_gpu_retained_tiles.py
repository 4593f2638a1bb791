"""Few retained slots beside a short Vague list.  Slot counts at the edges of a 16-token tile, of a wave's two tiles and of a
slice, empty slots that hold NaN, an infinite value; and one head per unit with rows that a narrow sketch has returned, whose
logits lie further apart than float32 exponentials reach.  The workspace holds other values before.  Reference: float64
attention over the retained rows and kvr_reconstruct's output; tolerance: the Vague weights keep 16 bits, the sums are
float32."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


@pytest.mark.parametrize("ret_cap", [1, 15, 16, 17, 33, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("G", [1, 2, 4])
@pytest.mark.parametrize("infinite", [False, True])
def test_slots_around_a_tile(ret_cap, G, infinite):
    from paper_2512_17917_amd import binding as kvr
    print("retained tiles", ret_cap, G, infinite, flush=True)
    g = torch.Generator(device="cuda").manual_seed(ret_cap * 8 + G)
    B, Hkv, r, w, cap = 2, 3, 3, 29, 300                       # 300 tokens: one workgroup per unit, 16 tiles' worth of waves
    dt = torch.bfloat16
    d = kvr.make_desc(B, Hkv * G, Hkv, r, w, dt, seed=9)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)
    k_ret, v_ret, sk, sv = rn(B, Hkv, ret_cap, D), rn(B, Hkv, ret_cap, D), rn(B, Hkv, r, w, D), rn(B, Hkv, r, w, D)
    q = rn(B, Hkv * G, D)
    n = ret_cap + cap
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(B * Hkv)]).view(B, Hkv, n).to(torch.int32)
    ret_pos, vague_pos = perm[..., :ret_cap].contiguous(), perm[..., ret_cap:].contiguous()
    if ret_cap > 4:
        for s in (0, 3, ret_cap - 1):
            ret_pos[1, 1, s] = -1
            k_ret[1, 1, s] = float("nan")
            v_ret[1, 1, s] = float("nan")
    if infinite:
        v_ret[0, 2, ret_cap // 2, 37] = float("inf")
    n_vague = torch.full((B, Hkv), cap, dtype=torch.int32, device="cuda")
    scores, out = torch.zeros(B, Hkv, n, device="cuda"), torch.zeros(B, Hkv * G, D, device="cuda")
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)
    kvr.kvr_attend_decode(d, q, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    kh, vh = torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda"), torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda")
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    empty = (ret_pos < 0).unsqueeze(-1)
    K = torch.cat([torch.where(empty, 0, k_ret), kh], dim=2).double()
    V = torch.cat([torch.where(empty, 0, v_ret), vh], dim=2).double()
    pos = torch.cat([ret_pos, vague_pos], dim=2).long()
    logit = torch.matmul(q.double().view(B, Hkv, G, D), K.transpose(2, 3).contiguous()) * d.softmax_scale
    p = torch.softmax(logit.masked_fill((pos < 0).unsqueeze(2), float("-inf")), dim=-1)
    finite = torch.where(torch.isfinite(V), V, 0)
    ref = torch.matmul(p, finite)
    hit = torch.zeros(B, Hkv, G, D, dtype=torch.bool, device="cuda")
    if infinite:
        hit[0, 2, :, 37] = True                                # and no other channel
    got = out.double().view(B, Hkv, G, D)
    assert bool((got[hit] == float("inf")).all())
    assert (got - ref)[~hit].abs().max().item() <= 2 ** -15 * finite.abs().max().item()
    want = torch.zeros(B, Hkv, n + 1, dtype=torch.float64, device="cuda")
    want.scatter_add_(2, torch.where(pos >= 0, pos, n), p.sum(2))
    assert (scores.double() - want[..., :n]).abs().max().item() <= 2e-5


@pytest.mark.parametrize("B,Hkv,G", [(1, 32, 1), (4, 8, 2), (4, 8, 4)])
@pytest.mark.parametrize("before", [50.0, 3e20, float("nan")])
def test_logits_far_apart(B, Hkv, G, before):
    """842 tokens, 79 slots, two sketch slots per row: 380 tokens in a slot, so that a rebuilt row is 20 times as large as a
    token's.  Every third retained row is one: logits of one tile lie up to some hundred apart."""
    from paper_2512_17917_amd import binding as kvr
    print("logits far apart", B, Hkv, G, before, flush=True)
    g = torch.Generator(device="cuda").manual_seed(7 * G + B)
    r, w, ret_cap, cap, dt = 3, 2, 79, 764, torch.bfloat16
    d = kvr.make_desc(B, Hkv * G, Hkv, r, w, dt, seed=71)
    rn = lambda x, *s: (x * torch.randn(*s, generator=g, device="cuda")).to(dt)
    k_ret, v_ret = rn(1, B, Hkv, ret_cap, D), rn(1, B, Hkv, ret_cap, D)
    k_ret[:, :, ::3] *= 30
    v_ret[:, :, ::3] *= 20
    sk, sv, q = rn(20, B, Hkv, r, w, D), rn(20, B, Hkv, r, w, D), rn(1, B, Hkv * G, D)
    n = ret_cap + cap
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(B * Hkv)]).view(B, Hkv, n).to(torch.int32)
    ret_pos, vague_pos = perm[..., :ret_cap].contiguous(), perm[..., ret_cap:].contiguous()
    n_vague = torch.full((B, Hkv), cap, dtype=torch.int32, device="cuda")
    scores, out = torch.zeros(B, Hkv, n, device="cuda"), torch.zeros(B, Hkv * G, D, device="cuda")
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap)
    ws[:ws.numel() // 4 * 4].view(torch.float32).fill_(before)
    kvr.kvr_attend_decode(d, q, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    kh, vh = torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda"), torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda")
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    K, V, Q = torch.cat([k_ret, kh], dim=2).double(), torch.cat([v_ret, vh], dim=2).double(), q.double().view(B, Hkv, G, D)
    KT = K.transpose(2, 3).contiguous()
    logit = torch.matmul(Q, KT) * d.softmax_scale
    assert (logit[..., :16].amax(-1) - logit[..., :16].amin(-1)).max().item() > 100
    p = torch.softmax(logit, dim=-1)
    # a logit is a float32 sum of 128 products: off by 128 * 2^-24 of the sum of their magnitudes at most, and a weight by
    # twice that of itself
    off = 2 * 128 * 2 ** -24 * (torch.matmul(Q.abs(), KT.abs()) * d.softmax_scale).max().item()
    got = out.double().view(B, Hkv, G, D)
    assert (got - torch.matmul(p, V)).abs().max().item() <= (2 ** -15 + off) * V.abs().max().item()
    want = torch.zeros(B, Hkv, n, dtype=torch.float64, device="cuda")
    want.scatter_add_(2, torch.cat([ret_pos, vague_pos], dim=2).long(), p.sum(2))
    assert (scores.double() - want).abs().max().item() <= G * (2e-5 + off)
