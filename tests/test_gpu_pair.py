"""The launches that hold list workgroups (64- and 16-channel kernels) and those of the retained slots: one to 25 rounds of 64
tokens a wave, lists that end inside a round, a wave and a workgroup, slices that end inside a tile, empty slots, any number of units.
Against attention in float64 over the rows that kvr_reconstruct gives (bit-exact against the oracle in its own tests).

Tolerance: a list token's weight has 16 bits in bf16 parts, so an output is off by at most 2^-16 of sum(p |v|), and float32
sums of n terms add less than 2^-20 of it for the n here; checked against 2^-15 of the largest |v| of the unit.  A
probability is off by its logit's error, 2^-20 of |q||k| / sqrt(128) (< 2^-17 for the rows below), relative."""
import pytest
import torch

pytestmark = pytest.mark.gpu
D = 128


@pytest.fixture(scope="module")
def kvr():
    from paper_2512_17917_amd import binding
    return binding


@pytest.mark.parametrize("units,G,r,w,ret_cap,cap", [
    (200, 4, 3, 20, 100, 12800),     # one workgroup per unit, 25 rounds
    (224, 2, 3, 333, 17, 12300),     # 25 rounds, the last two not in every wave; one slice of two tiles
    (120, 1, 3, 341, 1000, 12800),   # two turns or more; slices of several items per workgroup
    (8, 4, 3, 333, 3000, 6000),      # few rounds, many workgroups; slices that end inside a tile
    (9, 4, 3, 6, 1, 64),             # the smallest list that is staged
    (3, 1, 3, 6, 9300, 700),         # many slots and few units: short slices
    (1, 4, 3, 40, 9300, 3000),
    (200, 4, 3, 400, 100, 8704),     # 16 channels, three rows: 17 rounds
    (8, 2, 3, 1365, 2000, 3000),
    (200, 1, 4, 50, 100, 12288),     # four rows: 24 rounds
    (32, 4, 4, 300, 150, 700),       # lists of two rounds and a few slots each
    (9, 2, 4, 6, 1, 64),
])
def test_rounds_and_slices(kvr, units, G, r, w, ret_cap, cap):
    print("pair", units, G, r, w, ret_cap, cap, flush=True)
    g = torch.Generator(device="cuda").manual_seed(units * 7 + w)
    dt = torch.bfloat16
    d = kvr.make_desc(1, units * G, units, r, w, dt, seed=5)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)
    k_ret, v_ret, sk, sv = (rn(1, units, n, D) for n in (ret_cap, ret_cap, r * w, r * w))
    q = rn(1, units * G, D)
    n = ret_cap + cap
    perm = torch.argsort(torch.rand(units, n, generator=g, device="cuda"), dim=1).to(torch.int32)
    ret_pos, vague_pos = perm[:, :ret_cap].contiguous(), perm[:, ret_cap:].contiguous()
    empty = torch.rand(units, ret_cap, generator=g, device="cuda") < 0.1
    ret_pos[empty] = -1
    k_ret[0][empty] = float("nan")
    v_ret[0][empty] = float("nan")
    ends = [cap, 0, 1, 63, 64, 65, 511, 512, 513, cap - 1, cap - 64, cap // 2 + 1]
    n_vague = torch.tensor([min(max(ends[u % 12] if u % 24 < 12 else cap, 0), cap) for u in range(units)], dtype=torch.int32, device="cuda")
    scores, out = torch.zeros(units, n, device="cuda"), torch.zeros(units * G, D, device="cuda")
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)
    kvr.kvr_attend_decode(d, q, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    kh, vh = (torch.zeros(units, cap, D, dtype=dt, device="cuda") for _ in range(2))
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    assert torch.isfinite(out).all() and torch.isfinite(scores).all()
    for u in range(units):
        m = int(n_vague[u])
        K = torch.cat([torch.where(empty[u][:, None], 0, k_ret[0, u]), kh[u, :m]]).double()
        V = torch.cat([torch.where(empty[u][:, None], 0, v_ret[0, u]), vh[u, :m]]).double()
        pos = torch.cat([ret_pos[u], vague_pos[u, :m]]).long()
        x = (q[0, u * G:(u + 1) * G].double() @ K.T) * d.softmax_scale
        x[:, pos < 0] = float("-inf")
        if bool((pos < 0).all()):
            assert bool((out[u * G:(u + 1) * G] == 0).all())
            continue
        p = torch.softmax(x, dim=1)
        err = (out[u * G:(u + 1) * G].double() - p @ V).abs().max().item()
        assert err <= 2.0 ** -15 * V.abs().max().item(), (u, m, err)
        want = torch.zeros(n, dtype=torch.float64, device="cuda")
        want[pos[pos >= 0]] = p.sum(dim=0)[pos >= 0]
        assert bool(((scores[u].double() - want).abs() <= 2.0 ** -16 * want + 1e-12).all()), (u, m)


@pytest.mark.parametrize("units,G,n_q,w,ret_cap,cap", [
    (5, 8, 1, 20, 5000, 700),        # eight heads, kvr_attend_decode: slices larger than LDS holds the logits of
    (40, 8, 1, 333, 513, 300),
    (3, 4, 4, 40, 5000, 2000),       # 16 columns
    (3, 2, 4, 40, 5000, 300),        # eight
    (64, 1, 4, 6, 600, 900),         # four
    (9, 1, 2, 6, 17, 64),            # two; the newest tokens in the last tile
    (2, 1, 1, 6, 1, 64),
])
def test_streamed_list(kvr, units, G, n_q, w, ret_cap, cap):
    """The streaming kernel's launch, several queries with a causal mask (the newest n_q tokens are among the retained ones)."""
    print("streamed", units, G, n_q, w, ret_cap, cap, flush=True)
    g = torch.Generator(device="cuda").manual_seed(units * 5 + G)
    dt = torch.bfloat16
    d = kvr.make_desc(1, units * G, units, 3, w, dt, seed=5)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)
    k_ret, v_ret, sk, sv = (rn(1, units, n, D) for n in (ret_cap, ret_cap, 3 * w, 3 * w))
    q = rn(1, n_q, units * G, D)
    n = ret_cap + cap
    perm = torch.argsort(torch.rand(units, n, generator=g, device="cuda"), dim=1).to(torch.int32)
    for u in range(units):                   # the newest tokens: anywhere among the slots
        new = torch.arange(n - n_q, n, device="cuda", dtype=torch.int32)
        rest = perm[u][perm[u] < n - n_q]
        slot = torch.randperm(ret_cap, generator=g, device="cuda")[:n_q]
        head = torch.empty(ret_cap, dtype=torch.int32, device="cuda")
        mask = torch.ones(ret_cap, dtype=torch.bool, device="cuda")
        mask[slot] = False
        head[slot], head[mask] = new[:len(slot)], rest[:ret_cap - len(slot)]
        perm[u] = torch.cat([head, rest[ret_cap - len(slot):], new[len(slot):]])
    ret_pos, vague_pos = perm[:, :ret_cap].contiguous(), perm[:, ret_cap:].contiguous()
    empty = (torch.rand(units, ret_cap, generator=g, device="cuda") < 0.1) & (ret_pos < n - n_q)
    ret_pos[empty] = -1
    k_ret[0][empty] = float("nan")
    v_ret[0][empty] = float("nan")
    n_vague = torch.tensor([[cap, cap - 1, 64, 1, 0][u % 5] for u in range(units)], dtype=torch.int32, device="cuda")
    n_ctx = torch.full((1,), n, dtype=torch.int32, device="cuda")
    scores, out = torch.zeros(units, n, device="cuda"), torch.zeros(n_q, units * G, D, device="cuda")
    if G == 8:
        ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret_cap, cap).fill_(255)
        kvr.kvr_attend_decode(d, q[0], k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    else:
        size = kvr.kvr_attend_multi_workspace_size(d, n_q, ret_cap, cap)
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
        kvr.kvr_attend_multi(d, q, n_q, n_ctx, k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, scores, n, ws)
    if G == 8:                               # an infinite value reaches its own channel and no other
        slot, ref = int((ret_pos[0] >= 0).nonzero()[0]), out.clone()
        kept = v_ret[0, 0, slot, 37].clone()
        v_ret[0, 0, slot, 37] = float("inf")
        kvr.kvr_attend_decode(d, q[0], k_ret, v_ret, ret_pos, ret_cap, sk, sv, vague_pos, n_vague, cap, out, None, n, ws)
        assert bool((out[0, :G, 37] == float("inf")).all())
        out[0, :G, 37] = ref[0, :G, 37]
        # the list's tiles go to whichever wave is free: sums in another order, within the bound above
        assert (out - ref).abs().max().item() <= 2.0 ** -15 * max(x[torch.isfinite(x)].abs().max().item() for x in (v_ret, sv))
        v_ret[0, 0, slot, 37] = kept
    kh, vh = (torch.zeros(units, cap, D, dtype=dt, device="cuda") for _ in range(2))
    kvr.kvr_reconstruct(d, sk, sv, vague_pos, n_vague, cap, kh, vh)
    assert torch.isfinite(out).all() and torch.isfinite(scores).all()
    for u in range(units):
        m = int(n_vague[u])
        K = torch.cat([torch.where(empty[u][:, None], 0, k_ret[0, u]), kh[u, :m]]).double()
        V = torch.cat([torch.where(empty[u][:, None], 0, v_ret[0, u]), vh[u, :m]]).double()
        pos = torch.cat([ret_pos[u], vague_pos[u, :m]]).long()
        want = torch.zeros(n, dtype=torch.float64, device="cuda")
        for t in range(n_q):
            x = (q[0, t, u * G:(u + 1) * G].double() @ K.T) * d.softmax_scale
            x[:, (pos < 0) | (pos > n - n_q + t)] = float("-inf")
            if bool(torch.isinf(x).all()):
                assert bool((out[t, u * G:(u + 1) * G] == 0).all())
                continue
            p = torch.softmax(x, dim=1)
            err = (out[t, u * G:(u + 1) * G].double() - p @ V).abs().max().item()
            assert err <= 2.0 ** -15 * V.abs().max().item(), (u, t, m, err)
            want[pos[pos >= 0]] += p.sum(dim=0)[pos >= 0]
        assert bool(((scores[u].double() - want).abs() <= 2.0 ** -16 * want + 1e-12).all()), (u, m)
