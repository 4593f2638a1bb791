"""Buffers of a layer: each with a storage of its own (whoever keeps or saves one keeps or saves nothing else), zero
where nothing has been written."""
import pytest
import torch

from paper_2512_17917_amd import binding as kvr
from paper_2512_17917_amd.state import LayerState

BUFFERS = ("k_ret", "v_ret", "ret_pos", "scores", "sketch_k", "sketch_v", "vague_pos", "n_vague", "evict_slot",
           "evict_pos", "n_evict", "out")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_every_buffer_is_its_own_storage(dtype):
    d = kvr.make_desc(2, 8, 2, 3, 6, dtype, seed=1)
    ls = LayerState(d, n_recent=9, k_candidate=9, ret_cap=20, vague_cap=101, n_cap=131, device="cpu")
    for f in BUFFERS:
        x = getattr(ls, f)
        assert x.is_contiguous() and x.untyped_storage().nbytes() == x.numel() * x.itemsize, f
        assert bool((x == (-1 if f == "ret_pos" else 0)).all()), f
    assert len({getattr(ls, f).data_ptr() for f in BUFFERS}) == len(BUFFERS)


@pytest.mark.gpu
@pytest.mark.timeout(120)
def test_prompt_lists_are_zero_past_the_evictions(monkeypatch):
    """A prompt that all stays in the Recent queue (Slack): the eviction lists have room and no entry."""
    B, Hkv, N = 2, 3, 300
    d = kvr.make_desc(B, Hkv, Hkv, 3, 5, torch.bfloat16, seed=1)
    K, V = torch.randn(2, B, Hkv, N, 128, device="cuda").to(torch.bfloat16)
    empty = torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: empty(*a, **k).fill_(7))       # stale memory
    st, info = LayerState.from_prefill(d, K, V, K[:, :, 0].contiguous(), n_recent=100, k_candidate=50, max_new_tokens=4,
                                       init_scores=torch.rand(B, Hkv, N, device="cuda"), slack=250)
    assert info["evict_slot"].shape == (B, Hkv, 150) and not info["n_evict"].any()
    assert not info["evict_slot"].any() and not info["evict_pos"].any() and not st.n_vague.any()
    assert torch.equal(st.ret_pos[:, :, :N], torch.arange(N, dtype=torch.int32, device="cuda").expand(B, Hkv, N))
