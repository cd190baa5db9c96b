"""Rows of a sequence's first topk blocks keep every past block; in sequences with
enough rows they attend their whole prefix in one causal tile instead of being
routed.  The sizes lie just above the size from which that is done (it depends on the
rows of all heads), with a second sequence below it.  Every row, and every gradient
element, against the oracle under the tolerances of tests/parity.py."""
import pytest
import torch

from paper_2502_13189_amd import binding, inputs
import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ((1200, 40), 128, 1, 64, 3),   # one kv-head, 2 tokens per 256-row tile
    ((3000, 700), 64, 4, 100, 4),  # blocks that do not divide the 64-key tile
    ((1100, 1), 64, 64, 512, 2),   # MHA: the head is all but the last, short block
    ((1300,), 128, 2, 16, 31),     # 31 head blocks, 4 tokens per tile; short blocks after them
]
FORWARD_CASES = CASES + [
    ((2500, 30), 128, 128, 16, 4),  # blocks that fill part of one 128-row work-group
    ((5200,), 16, 4, 2100, 2),     # a launch of its own for the causal tiles
]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()


def routed(q, k, v, cu, B, topk, dtype):
    r = parity.moba_parity(q, k, v, cu, B, topk, dtype=dtype)
    print("max_abs %.2e lse %.2e ties %d" % (r["max_abs"], r["lse_max_abs"], r["tie_rows"]))


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", FORWARD_CASES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_forward(seqlens, hq, hkv, B, topk, dtype):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, dtype, B, 0.5, B, device=DEV)
    routed(q, k, v, cu, B, topk, "f32" if dtype == torch.float32 else "bf16")


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", CASES)
def test_backward(seqlens, hq, hkv, B, topk):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, B, device=DEV)
    dout = inputs.make_dout(q.shape, q.dtype, B, device=DEV)
    print(parity.moba_backward_parity(q, k, v, cu, B, topk, dout))


def test_rows_do_not_depend_on_the_batch():
    """The rule looks at one sequence: a row's bits are the same alone and packed."""
    seqlens, hq, hkv, B, topk = (1200, 333, 1250), 128, 1, 64, 3
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, 3, device=DEV)
    out, lse = binding.forward(q, k, v, cu, B, topk)
    for s, L in enumerate(seqlens):
        a, b = int(cu[s]), int(cu[s + 1])
        o, l = binding.forward(q[a:b], k[a:b], v[a:b], inputs.cu_seqlens((L,)), B, topk)
        assert torch.equal(o, out[a:b]) and torch.equal(l, lse[:, a:b])
