"""Batches of very many short blocks: more than 2^32 work items in the launches over
(block, kv-head) pairs (HIP takes fewer along one dimension, so they go in pieces):
block means, and forwards whose rows must be those of each sequence alone."""
import pytest
import torch

from paper_2502_13189_amd import binding, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()


@pytest.mark.parametrize("dtype,T", [(torch.bfloat16, 1 << 20), (torch.float32, (1 << 19) + 37)])
def test_pool_of_one_key_blocks(dtype, T):
    """2^23 (bf16) pairs and a little over 2^22 (fp32): every mean is its key."""
    k = torch.randn((T, 8, 128), device=DEV).to(dtype)
    kbar = binding.pool(k, inputs.cu_seqlens((T,)), 1)
    for t in range(0, T, 1 << 18):
        assert torch.equal(kbar[t:t + (1 << 18)], k[t:t + (1 << 18)].float())


@pytest.mark.parametrize("dtype,n", [(torch.bfloat16, 130), (torch.float32, 66)])
def test_forward_of_two_key_blocks(dtype, n):
    """n sequences of 4096 two-key blocks, 8 kv-heads: pool (bf16), and both kinds of
    attention tiles, in more than one piece."""
    L, hq, hkv, B, topk = 8192, 8, 8, 2, 2
    lens = (L,) * (n - 1) + (L - 1,)
    T = sum(lens)
    gen = torch.Generator(device=DEV).manual_seed(7)
    q, k, v = (torch.randn((T, 8, 128), device=DEV, generator=gen).to(dtype) for _ in range(3))
    out, lse = binding.forward(q, k, v, inputs.cu_seqlens(lens), B, topk)
    assert torch.isfinite(lse).all()
    for s in (0, n // 2, n - 2, n - 1):
        a = s * L
        b = a + lens[s]
        o, l = binding.forward(q[a:b], k[a:b], v[a:b], inputs.cu_seqlens((b - a,)), B, topk)
        assert torch.equal(o, out[a:b]) and torch.equal(l, lse[:, a:b])
    binding.release_workspace()
