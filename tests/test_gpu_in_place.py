"""out written over q (the same memory and strides): every row of q is read before it is
overwritten, also where history and current-block tiles otherwise share one launch.
The same bits as with an out of its own."""
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


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((700, 0, 333), 8, 2, 128, 3),   # a small batch
    ((40000,), 8, 2, 512, 4),        # more work-groups than the chip holds at once
    ((20000, 9000), 4, 4, 64, 8),
    ((9000,), 8, 2, 2304, 2),        # two launches in any case
    ((500,), 4, 1, 512, 2),          # full attention
])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("packed", [False, True])
def test_out_over_q(seqlens, hq, hkv, B, topk, dtype, packed):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, dtype, B, 0.5, B, device=DEV)
    ref, rlse = binding.forward(q, k, v, cu, B, topk)
    if packed:  # q is a slice of a fused projection
        qkv = torch.cat([q, k, v], dim=1)
        q, k, v = qkv[:, :hq], qkv[:, hq:hq + hkv], qkv[:, hq + hkv:]
    out, lse = binding.forward(q, k, v, cu, B, topk, out=q)
    assert torch.equal(out, ref) and torch.equal(lse, rlse)
