"""Small batches let the gate count its selections and the scatter scan the
counts; larger ones (here: the same batch with a filler sequence that brings it
past 1024 bins) run the count and scan kernels.  Rows do not depend on the
batch they are in, so both must give the same bits, forward and dQ; dK and dV are fp32
sums that a small batch may take in shares, so they may round differently."""
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
    ((300,), 2, 2, 16, 2),
    ((700, 0, 333, 1), 8, 2, 16, 4),       # several sequences, one empty
    ((500, 260), 6, 2, 16, 12),            # groups of 3: 85 tokens per gate group, 255 rows
    ((130, 40), 100, 1, 16, 3),            # 2 tokens per gate group
    ((2000,), 4, 1, 16, 32),               # the largest slot count, 125 blocks
    ((8190,), 2, 2, 16, 6),                # 1022 bins, the last ones below the limit
    ((1025, 1023), 16, 16, 64, 3),         # one row past a routing chunk
    ((2544,), 16, 1, 16, 3),               # 159 gate groups, the last below the limit
    ((5104,), 16, 1, 64, 9),               # 319, from eight selections per row on
])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_small_routing_equals_general(seqlens, hq, hkv, B, topk, dtype):
    T, fill = sum(seqlens), 1040 * B
    q, k, v, cu = inputs.make(seqlens + (fill,), hq, hkv, 128, dtype, B, 0.5, T + B, device=DEV)
    big, blse = binding.forward(q, k, v, cu, B, topk)
    qs, ks, vs, cus = q[:T], k[:T], v[:T], cu[:-1].contiguous()
    out, lse = binding.forward(qs, ks, vs, cus, B, topk)
    assert torch.equal(out, big[:T]) and torch.equal(lse, blse[:, :T])
    if dtype == torch.bfloat16:
        dout = inputs.make_dout(q.shape, dtype, T, device=DEV)
        gb = binding.backward(q, k, v, cu, B, topk, big, blse, dout)
        gs = binding.backward(qs, ks, vs, cus, B, topk, out, lse, dout[:T])
        assert torch.equal(gs[0], gb[0][:T])
        for name, x, y in zip(("dk", "dv"), gs[1:], gb[1:]):
            # far fewer than all elements round to the other bf16 neighbour (2^-8 of the value)
            x, y = x.double(), y[:T].double()
            assert (x - y).norm() <= 2.0 ** -9 * y.norm(), name
