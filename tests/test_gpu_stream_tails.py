"""The streaming kernel over the Vague list where its tiles end: list capacities and device counts that leave every
remainder of a 16-token tile, of the fours a record load takes and of a workgroup's share, for the column counts of
kvr_attend_multi and for a decode call with eight heads.  Reference: float64 attention over kvr_reconstruct's output.
Tolerance: a weight keeps 16 bits (2^-16 of the largest value at most, all weights together sum to one) and the sums
are float32."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


@pytest.mark.parametrize("cap", [64, 67, 257, 1021])
@pytest.mark.parametrize("n_q,G", [(0, 8), (1, 4), (2, 4), (4, 4), (16, 1)])
def test_every_remainder(cap, n_q, G):
    from paper_2512_17917_amd import binding as kvr
    print("stream tails", cap, n_q, G, flush=True)
    g = torch.Generator(device="cuda").manual_seed(cap * 32 + n_q)
    B, Hkv, r, w, ret_cap = 4, 5, 3, 29, 33
    dt, nq = torch.bfloat16, max(n_q, 1)
    d = kvr.make_desc(B, Hkv * G, Hkv, r, w, dt, seed=cap)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)
    k_ret, v_ret, sk, sv = rn(B, Hkv, ret_cap, D), rn(B, Hkv, ret_cap, D), rn(B, Hkv, r, w, D), rn(B, Hkv, r, w, D)
    q = rn(B, nq, Hkv * G, D)
    n = ret_cap + cap
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(B * Hkv)]).view(B, Hkv, n).to(torch.int32)
    ret_pos, vague_pos = perm[..., :ret_cap].contiguous(), perm[..., ret_cap:].contiguous()
    n_vague = (cap - torch.arange(B * Hkv, device="cuda")).view(B, Hkv).to(torch.int32)      # cap, cap - 1, ... cap - 19
    n_ctx = torch.full((B,), n, dtype=torch.int32, device="cuda")
    scores = torch.zeros(B, Hkv, n, device="cuda")
    out = torch.zeros(B, nq, Hkv * G, D, device="cuda")
    if n_q:
        ws = torch.full((kvr.kvr_attend_multi_workspace_size(d, n_q, ret_cap, cap),), 255, dtype=torch.uint8, device="cuda")
        kvr.kvr_attend_multi(d, q, n_q, n_ctx, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    else:
        ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)              # NaN wherever nothing is written
        kvr.kvr_attend_decode(d, q[:, 0], k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out[:, 0], scores, n, ws)
    kh, vh = torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda"), torch.zeros(B, Hkv, cap, D, dtype=dt, device="cuda")
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    live = torch.arange(cap, device="cuda") < n_vague.unsqueeze(-1)
    pos = torch.cat([ret_pos, torch.where(live, vague_pos, -1)], dim=2).long()
    K, V = torch.cat([k_ret, kh], dim=2).double(), torch.cat([v_ret, vh], dim=2).double()
    want = torch.zeros(B, Hkv, n + 1, dtype=torch.float64, device="cuda")
    for t in range(nq):
        logit = torch.matmul(q[:, t].double().view(B, Hkv, G, D), K.transpose(2, 3).contiguous()) * d.softmax_scale
        seen = (pos >= 0) & (pos <= (n - nq + t if n_q else n))
        p = torch.softmax(logit.masked_fill(~seen.unsqueeze(2), float("-inf")), dim=-1)
        ref = torch.matmul(p, V).view(B, Hkv * G, D)
        assert (out[:, t].double() - ref).abs().max().item() <= 2 ** -15 * V.abs().max().item(), t
        want.scatter_add_(2, torch.where(pos >= 0, pos, n), p.sum(2))
    assert (scores.double() - want[..., :n]).abs().max().item() <= 2e-5 * nq
