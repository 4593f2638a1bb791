"""kvr_compact against plain indexing: ranges of 256 source slots and their edges, a last range without a kept
row, more kept rows than max_keep or than the destination holds, both storage types.  Copies: exact."""
import pytest
import torch

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n,share,ret_cap,max_keep", [
    (1, 1.0, 3, 1), (255, 0.3, 130, 200), (512, 0.25, 600, 600), (513, 0.5, 400, 400), (6001, 0.2, 1500, 1500),
    (4097, 0.9, 700, 4097), (5000, 0.5, 3000, 900), (4100, 0.0, 5, 5), (2100, 1.0, 2101, 2100)])
def test_compact(dtype, n, share, ret_cap, max_keep):
    from paper_2512_17917_amd import binding as kvr
    g = torch.Generator().manual_seed(n)
    B, Hkv, D = 2, 3, 128
    d = kvr.make_desc(B, Hkv, Hkv, 3, 5, dtype, seed=1)
    k, v = (torch.randn(B, Hkv, n, D, generator=g).to(dtype) for _ in range(2))
    pos = torch.arange(n, dtype=torch.int32).expand(B, Hkv, n) + 7
    pos = torch.where(torch.rand(B, Hkv, n, generator=g) < share, pos, torch.full_like(pos, -1)).contiguous()
    pos[0, 0, -1] = -1                                   # nothing kept at the end of the list
    n_evict = (pos < 0).sum(-1).to(torch.int32)
    evict = torch.zeros(B, Hkv, n, dtype=torch.int32)
    for b in range(B):
        for h in range(Hkv):
            gone = torch.nonzero(pos[b, h] < 0).flatten().to(torch.int32)
            evict[b, h, :len(gone)] = gone
    kr, vr = (torch.full((B, Hkv, ret_cap, D), 3.0, dtype=dtype, device="cuda") for _ in range(2))
    rp = torch.full((B, Hkv, ret_cap), 99, dtype=torch.int32, device="cuda")
    print("[case]", dtype, n, share, ret_cap, max_keep, flush=True)
    kvr.kvr_compact(d, k.cuda(), v.cuda(), pos.cuda(), n, evict.cuda(), n_evict.cuda(), n, kr, vr, rp, ret_cap, max_keep)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(Hkv):
            slots = torch.nonzero(pos[b, h] >= 0).flatten()[:min(max_keep, ret_cap)]
            m = len(slots)
            for got, src in ((kr, k), (vr, v)):
                assert torch.equal(got[b, h, :m].cpu(), src[b, h, slots])
                assert not got[b, h, m:].any()
            assert torch.equal(rp[b, h, :m].cpu(), pos[b, h, slots])
            assert (rp[b, h, m:] == -1).all()
