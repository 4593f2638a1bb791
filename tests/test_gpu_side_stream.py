"""A lent second stream where the call takes it: sketches that only the general staged kernel holds, a list that fills the chip twice
over.  The capped form of the retained kernel next to it, with the logits of a whole slice in LDS and of 512 tokens at a time, ragged
last slices, empty slots, an empty unit: bit for bit against the call without the stream (the same sums in the same order), some units
against float64 over the slots and kvr_reconstruct's rows (weights with float32's 24 bits and sums of float32: 2^-18 of the largest
value), and by the entry point with the library's own scratch memory."""
import ctypes as C

import pytest
import torch

from tests.test_plan_cpu import SIDE_BY_SIDE

pytestmark = pytest.mark.gpu
D = 128


@pytest.mark.parametrize("units,G,r,w,ret,cap,how", SIDE_BY_SIDE)
def test_forked_call(units, G, r, w, ret, cap, how):
    from paper_2512_17917_amd import binding as kvr
    print("side stream", units, G, r, w, ret, cap, how, flush=True)
    g = torch.Generator(device="cuda").manual_seed(w)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    d = kvr.make_desc(1, units * G, units, r, w, torch.bfloat16, seed=5)
    q, K, V, SK, SV = rn(1, units * G, D), rn(1, units, ret, D), rn(1, units, ret, D), rn(1, units, r, w, D), rn(1, units, r, w, D)
    n = ret + cap
    perm = torch.argsort(torch.rand(units, n, generator=g, device="cuda"), dim=1).to(torch.int32)
    rp, vp = perm[:, :ret].contiguous(), perm[:, ret:].contiguous()
    rp[torch.rand(rp.shape, generator=g, device="cuda") < 0.1] = -1
    rp[3] = -1
    nv = torch.randint(cap - 300, cap + 1, (units,), generator=g, device="cuda").to(torch.int32)
    nv[3], nv[5] = 0, 1
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ATTEND, ret, cap)
    side = kvr.SideStream()
    side.fork, side.join = kvr.event_create(True), kvr.event_create(True)      # with timing: they tell that they were recorded
    got = []
    for sd in (side, None):
        for with_scores in (True, False):
            out, sc = torch.full((1, units * G, D), 9.0, device="cuda"), torch.ones(units, n, device="cuda")
            ws.fill_(255)                                   # what a call leaves unwritten is NaN
            kvr.kvr_attend_decode(d, q, K, V, rp, ret, SK, SV, vp, nv, cap, out, sc if with_scores else None, n, ws,
                                  sd.opts() if sd else None)
            got.append((out, sc))
    torch.cuda.synchronize()
    assert kvr.event_elapsed_ms(side.fork, side.join) > 0
    out, sc = torch.full((1, units * G, D), 9.0, device="cuda"), torch.ones(units, n, device="cuda")
    p = lambda x: C.c_void_p(x.data_ptr())
    opts, stream = side.opts(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert kvr.kvr_workspace_size(d, kvr.KVR_OP_ATTEND, ret, cap) <= kvr.KVR_STATIC_SCRATCH_BYTES
    assert kvr.lib().kvr_attend_decode_static(C.byref(d), p(q), p(K), p(V), p(rp), ret, p(SK), p(SV), p(vp), p(nv), cap, p(out), p(sc), n,
                                              C.byref(opts), stream) == kvr.KVR_OK
    torch.cuda.synchronize()
    for o, s in got:
        assert torch.isfinite(o).all() and torch.isfinite(s).all() and not o[0, 3 * G:4 * G].any()
        assert torch.equal(o, out) and (torch.equal(s, sc) or bool((s == 1).all()))
    assert torch.equal(got[0][1], got[2][1]) and not torch.equal(got[0][1], got[1][1])
    kh, vh = (torch.zeros(units, cap, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    kvr.kvr_reconstruct(d, SK, SV, vp, nv, cap, kh, vh)
    for u in (0, 5, 77, units - 1):
        m, live = int(nv[u]), rp[u] >= 0
        k, v = torch.cat([K[0, u][live], kh[u, :m]]).double(), torch.cat([V[0, u][live], vh[u, :m]]).double()
        x = torch.softmax((q[0, u * G:(u + 1) * G].double() @ k.T.contiguous()) * d.softmax_scale, dim=1)
        assert (out[0, u * G:(u + 1) * G].double() - x @ v).abs().max().item() <= 2.0 ** -18 * v.abs().max().item(), u
        want = torch.ones(n, dtype=torch.float64, device="cuda")
        want[torch.cat([rp[u][live], vp[u, :m]]).long()] += x.sum(dim=0)
        assert bool(((sc[u].double() - want).abs() <= 2.0 ** -23 * want + 2.0 ** -16 * (want - 1)).all()), u
