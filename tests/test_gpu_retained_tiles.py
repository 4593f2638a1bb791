"""Few retained slots next to a staged Vague list: the staged kernel's waves take the slots along, up to two 16-token tiles
each.  Slot counts at the edges of a tile and of the waves' two tiles (and one more, where the retained kernel has a launch of
its own again), empty slots that hold NaN, no position list, an infinite value.  Reference: float64 attention over the retained rows
and kvr_reconstruct's output; tolerance: the Vague weights keep 16 bits, the sums are float32."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


@pytest.mark.parametrize("ret_cap", [1, 15, 16, 17, 33, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("G", [1, 2, 4])
@pytest.mark.parametrize("infinite", [False, True])
def test_slots_taken_along(ret_cap, G, infinite):
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
