"""dK/dV with a key tile's rows shared over several work-groups (fewer key tiles than
half of the CUs) and summed: more shares than chunks of rows, shares of one chunk, a
partial key tile, the largest batch that splits and the first that does not.
All gradients against the oracle under the bounds of tests/parity.py."""
import pytest
import torch

from paper_2502_13189_amd import binding, inputs
import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((1,), 1, 1, 4, 1),                # one row, one key
    ((200, 3), 2, 1, 128, 2),          # a full and a partial key tile, few chunks
    ((900,), 8, 1, 128, 3),            # eight shares
    ((1000, 517), 12, 4, 100, 4),      # groups of 3, partial key tiles
    ((8192,), 2, 2, 512, 2),           # 128 key tiles: two shares
    ((8200,), 2, 2, 512, 2),           # 130: no split
])
def test_split_gradients(seqlens, hq, hkv, B, topk):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, B, device=DEV)
    dout = inputs.make_dout(q.shape, q.dtype, B, device=DEV)
    print(parity.moba_backward_parity(q, k, v, cu, B, topk, dout))


def test_split_strided_and_repeatable(monkeypatch):
    """Gradients into views of one fused buffer; the same bits on every call, and
    within the bounds when the workspace cap leaves no room for the shares."""
    seqlens, hq, hkv, B, topk = (700, 333), 8, 2, 128, 3
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, 5, device=DEV)
    dout = inputs.make_dout(q.shape, q.dtype, 5, device=DEV)
    out, lse = binding.forward(q, k, v, cu, B, topk)
    ref = binding.backward(q, k, v, cu, B, topk, out, lse, dout)
    buf = torch.zeros((q.shape[0], hq + 2 * hkv, 128), device=DEV, dtype=q.dtype)
    got = binding.backward(q, k, v, cu, B, topk, out, lse, dout, dq=buf[:, :hq],
                           dk=buf[:, hq:hq + hkv], dv=buf[:, hq + hkv:])
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
    torch.cuda.synchronize()
    binding.release_workspace()
    one = None
    for mb in range(6, 64):
        monkeypatch.setenv("MOBA_WORKSPACE_LIMIT_BYTES", str(mb << 20))
        try:
            one = binding.backward(q, k, v, cu, B, topk, out, lse, dout)
            break
        except binding.MobaError as e:
            assert e.name == "MOBA_ERR_NO_MEMORY"
    monkeypatch.delenv("MOBA_WORKSPACE_LIMIT_BYTES")
    assert binding.workspace_held_bytes() <= mb << 20
    assert torch.equal(one[0], ref[0])
    for x, y in zip(one[1:], ref[1:]):
        assert (x.double() - y.double()).norm() <= 2.0 ** -9 * y.double().norm()
