"""Values of a live retained slot that are no finite numbers, in every form of the kernels that stream the slots: one to eight heads
of kvr_attend_decode (eight: the streaming kernel) and two to sixteen columns of kvr_attend_multi, on CUs of the list's launch and in a
launch of their own.  An infinite value reaches its own channel with its sign and no other; a NaN its own channel; a key with a NaN all
outputs of its unit.  What is not named comes out as attention in float64 over the slots and kvr_reconstruct's rows gives it:
a list token's weight has 16 bits, so within 2^-15 of the largest value (float32 sums add less than that)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
D, INF, NAN = 128, float("inf"), float("nan")


@pytest.fixture(scope="module")
def kvr():
    from paper_2512_17917_amd import binding
    return binding


@pytest.mark.parametrize("G,n_q", [(1, 0), (2, 0), (4, 0), (8, 0), (1, 2), (1, 4), (2, 4), (4, 2), (4, 4), (8, 2)])
@pytest.mark.parametrize("units,ret_cap,cap", [(3, 75, 700), (300, 20, 200)])
def test_live_slots_that_are_not_finite(kvr, G, n_q, units, ret_cap, cap):
    print("special rows", G, n_q, units, ret_cap, cap, flush=True)
    g = torch.Generator(device="cuda").manual_seed(units * 7 + G * 3 + n_q)
    dt, r, w, nq = torch.bfloat16, 3, 7, max(n_q, 1)
    d = kvr.make_desc(1, units * G, units, r, w, dt, seed=5)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    base = rn(units, 1, D)
    # queries near one direction, a slot that all of them find first: its weight is 1 and has no second and third part
    q = (base.unsqueeze(0) + 0.3 * rn(nq, units, G, D)).to(dt).view(1, nq, units * G, D)
    k_ret, v_ret, sk, sv = (rn(1, units, n, D).to(dt) for n in (ret_cap, ret_cap, r * w, r * w))
    k_ret[0, :, 5] = (2 * base[:, 0]).to(dt)
    n = ret_cap + cap
    perm = torch.argsort(torch.rand(units, n - nq, generator=g, device="cuda"), dim=1).to(torch.int32)
    new = torch.arange(n - nq, n, device="cuda", dtype=torch.int32).expand(units, nq)
    ret_pos = torch.cat([perm[:, :ret_cap - nq], new], dim=1).contiguous()      # the newest tokens in the last slots
    vague_pos = perm[:, ret_cap - nq:].contiguous()
    n_vague = torch.full((units,), cap, dtype=torch.int32, device="cuda")
    n_ctx = torch.full((1,), n, dtype=torch.int32, device="cuda")
    v_ret[0, 0, 5, 37], v_ret[0, 0, 5, 90] = INF, -INF        # a weight of 1
    v_ret[0, 0, 2, 38] = INF                                  # some weight
    v_ret[0, 1, 9, 3], v_ret[0, 1, 5, 64] = NAN, NAN
    k_ret[0, 2, 6, 11] = NAN
    scores, out = torch.zeros(units, n, device="cuda"), torch.zeros(nq, units * G, D, device="cuda")
    if n_q:
        ws = torch.full((kvr.kvr_attend_multi_workspace_size(d, n_q, ret_cap, cap),), 255, dtype=torch.uint8, device="cuda")
        kvr.kvr_attend_multi(d, q, n_q, n_ctx, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    else:
        ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)
        kvr.kvr_attend_decode(d, q[0], k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    kh, vh = (torch.zeros(units, cap, D, dtype=dt, device="cuda") for _ in range(2))
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    K, V = torch.cat([k_ret[0], kh], dim=1).double(), torch.cat([v_ret[0], vh], dim=1).double()
    V = torch.where(torch.isfinite(V), V, 0)
    pos = torch.cat([ret_pos, vague_pos], dim=1)
    got = out.view(nq, units, G, D).double()
    scored = torch.zeros(units, n, dtype=torch.float64, device="cuda")
    for t in range(nq):
        x = torch.matmul(q[0, t].view(units, G, D).double(), K.transpose(1, 2).contiguous()) * d.softmax_scale
        p = torch.softmax(x.masked_fill((pos > n - nq + t).unsqueeze(1), -INF), dim=2)
        scored.scatter_add_(1, pos.long(), p.sum(dim=1))
        want = torch.matmul(p, V)
        assert bool((got[t, 0, :, 37] == INF).all()) and bool((got[t, 0, :, 90] == -INF).all()) and bool((got[t, 0, :, 38] == INF).all()), t
        assert bool(torch.isnan(got[t, 1, :, 3]).all()) and bool(torch.isnan(got[t, 1, :, 64]).all()) and bool(torch.isnan(got[t, 2]).all())
        named = torch.zeros(units, G, D, dtype=torch.bool, device="cuda")
        named[0, :, [37, 38, 90]] = True
        named[1, :, [3, 64]] = True
        named[2] = True
        err = (got[t] - want).masked_fill(named, 0).abs().max().item()
        assert err <= 2.0 ** -15 * V.abs().max().item(), (t, err)
    keep = torch.arange(units, device="cuda") != 2
    assert bool(((scores[keep].double() - scored[keep]).abs() <= 2.0 ** -16 * scored[keep] + 1e-12).all())
