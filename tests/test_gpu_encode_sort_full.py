"""The counting sort of the bulk insert with every place of its LDS in use: units whose lists are full, or one token short, on both sides of
the longest list that LDS holds, at most and at fewest waves for it, and at the line of seven waves.  Bit for bit against sequential
float32 sums in list order (kvr_hash_host for slots and signs): the k-th tokens of all slots are added together, k after k."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
D, LDS_INTS = 128, 160 * 1024 // 4


@pytest.mark.parametrize("w,cap", [(29, LDS_INTS - 17 * 29 - 1), (29, LDS_INTS - 17 * 29), (273, LDS_INTS - 17 * 273 - 1), (273, LDS_INTS - 17 * 273),
                                   (1920, LDS_INTS - 8 * 1920 - 1), (1920, LDS_INTS - 8 * 1920), (1921, 24000), (8192, 24576), (1, 5000)])
def test_full_lists(w, cap):
    from paper_2512_17917_amd import binding as kvr
    print("full lists", w, cap, flush=True)
    rng = np.random.default_rng(w + cap)
    units, r, rows = 3, 3, 60
    counts = np.array([cap, cap - 1, cap - 64], dtype=np.int32)
    d = kvr.make_desc(1, units, units, r, w, torch.float32, seed=w)
    K, V = (rng.standard_normal((units, rows, D)).astype(np.float32) for _ in range(2))
    S0 = rng.standard_normal((2, units, r, w, D)).astype(np.float32)
    slot = rng.integers(0, rows, size=(units, cap)).astype(np.int32)
    pos = np.stack([rng.permutation(1 << 17)[:cap] for _ in range(units)]).astype(np.int32)
    dev = lambda x: torch.as_tensor(x).cuda()
    sk, sv = dev(S0[0]), dev(S0[1])
    ws = kvr.alloc_workspace(d, kvr.KVR_OP_ENCODE, cap).fill_(255)
    kvr.kvr_encode(d, dev(K[None]), dev(V[None]), rows, dev(slot), dev(pos), dev(counts), cap, sk[None], sv[None], None, None, ws)
    torch.cuda.synchronize()
    hp = np.array([[int(x) for x in d.hash_params[i]] for i in range(r)], dtype=np.uint64)
    bk, sg = (C.c_int32 * r)(), (C.c_int32 * r)()
    for u in range(units):
        n = counts[u]
        J = pos[u, :n].astype(np.uint64)
        with np.errstate(over="ignore"):
            bucket = np.stack([(((hp[i, 0] * J + hp[i, 1]) >> np.uint64(32)) * np.uint64(w)) >> np.uint64(32) for i in range(r)]).astype(int)
            minus = np.stack([(hp[i, 2] * J + hp[i, 3]) >> np.uint64(63) for i in range(r)]).astype(bool)
        for e in (0, n // 2, n - 1):
            kvr.lib().kvr_hash_host(C.byref(d), int(J[e]), bk, sg)
            assert list(bk) == bucket[:, e].tolist() and [x < 0 for x in sg] == minus[:, e].tolist()
        for i in range(r):
            order = np.argsort(bucket[i], kind="stable")
            b = bucket[i][order]
            rank = np.arange(n) - np.searchsorted(b, b)                 # the how-manieth token of its slot
            k, v = S0[0, u, i].copy(), S0[1, u, i].copy()
            by_rank = np.argsort(rank, kind="stable")
            ends = np.searchsorted(rank[by_rank], np.arange(rank.max() + 2))
            for a, z in zip(ends[:-1], ends[1:]):
                e = order[by_rank[a:z]]
                k[bucket[i][e]] += K[u, slot[u, e]]
                v[bucket[i][e]] += np.where(minus[i][e][:, None], -V[u, slot[u, e]], V[u, slot[u, e]])
            assert np.array_equal(sk[u, i].cpu().numpy(), k), ("sketch_k", u, i)
            assert np.array_equal(sv[u, i].cpu().numpy(), v), ("sketch_v", u, i)
