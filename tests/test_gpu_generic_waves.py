"""The generic attention kernel on both sides of its switch between 16 waves and four waves per workgroup (as many workgroups
as the chip has compute units, and one more row of them), for every head count, row count and storage type that it takes there,
with lists of different lengths and a workspace full of NaN.  Reference: float64 attention over the retained rows and
kvr_reconstruct's output."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


def _slices(tokens, units):
    """Workgroups per unit: about 1280 in all, whole 64 tokens each, at least 128 of a long list."""
    t = -(-(tokens * units // 1280) // 64) * 64
    return -(-tokens // max(t, 128 if tokens >= 1024 else 64))


F32, BF16 = torch.float32, torch.bfloat16
# float32: retained slots and list in one launch; bfloat16 with five rows: the list by itself
CASES = [(F32, *x, G, r) for x in ((167, 857, False), (168, 857, True), (1, 30, False)) for G in (1, 2, 4, 8) for r in (3, 4, 5)]
CASES += [(BF16, *x, G, 5) for x in ((65, 1024, False), (65, 1025, True)) for G in (1, 2, 4, 8)]


@pytest.mark.parametrize("dt,ret_cap,cap,wide,G,r", CASES)
def test_both_sides_of_the_switch(dt, ret_cap, cap, wide, G, r):
    from paper_2512_17917_amd import binding as kvr
    print("generic waves", dt, ret_cap, cap, G, r, flush=True)
    B, Hkv, w = 4, 8, 23
    launch = B * Hkv * _slices(cap if dt == BF16 else ret_cap + cap, B * Hkv)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert (launch > cus) == wide and launch <= cus + B * Hkv, (launch, cus)
    g = torch.Generator(device="cuda").manual_seed(cap * 64 + G * 8 + r)
    d = kvr.make_desc(B, Hkv * G, Hkv, r, w, dt, seed=5)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)
    k_ret, v_ret, sk, sv = rn(B, Hkv, ret_cap, D), rn(B, Hkv, ret_cap, D), rn(B, Hkv, r, w, D), rn(B, Hkv, r, w, D)
    q, n = rn(B, Hkv * G, D), ret_cap + cap
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(B * Hkv)]).view(B, Hkv, n).to(torch.int32)
    ret_pos, vague_pos = perm[..., :ret_cap].contiguous(), perm[..., ret_cap:].contiguous()
    if ret_cap > 4:                                            # an empty slot may hold anything
        ret_pos[1, 1, 3] = -1
        k_ret[1, 1, 3] = v_ret[1, 1, 3] = float("nan")
    n_vague = (cap - torch.arange(B * Hkv, device="cuda") * (cap // 40)).view(B, Hkv).to(torch.int32)
    n_vague[2, 3] = 0
    scores, out = torch.zeros(B, Hkv, n, device="cuda"), torch.zeros(B, Hkv * G, D, device="cuda")
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)
    kvr.kvr_attend_decode(d, q, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    kh, vh = torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda"), torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda")
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    live = torch.arange(cap, device="cuda") < n_vague.unsqueeze(-1)
    pos = torch.cat([ret_pos, torch.where(live, vague_pos, -1)], dim=2).long()
    held = (ret_pos >= 0).unsqueeze(-1)
    K = torch.cat([torch.where(held, k_ret, 0), kh], dim=2).double()
    V = torch.cat([torch.where(held, v_ret, 0), vh], dim=2).double()
    Q, KT = q.double().view(B, Hkv, G, D), K.transpose(2, 3).contiguous()
    p = torch.softmax((torch.matmul(Q, KT) * d.softmax_scale).masked_fill((pos < 0).unsqueeze(2), float("-inf")), dim=-1)
    # a logit is a float32 sum of 128 products: off by 128 * 2^-24 of the sum of their magnitudes at most, a weight by twice
    # that of itself; exponentials, sums over the tokens and the division by less than 64 * 2^-24; the matrix instructions of
    # bfloat16's retained slots keep as many bits
    off = (2 * 128 * (torch.matmul(Q.abs(), KT.abs()) * d.softmax_scale).max().item() + 64) * 2 ** -24
    got = out.double().view(B, Hkv, G, D)
    assert (got - torch.matmul(p, V)).abs().max().item() <= off * V.abs().max().item()
    want = torch.zeros(B, Hkv, n + 1, dtype=torch.float64, device="cuda")
    want.scatter_add_(2, torch.where(pos >= 0, pos, n), p.sum(2))
    assert (scores.double() - want[..., :n]).abs().max().item() <= G * off
