"""fp32 attention at the edges of its tiles: 32-row work-groups (four per
128-row tile), 32-key subtiles dealt to four waves.  Every row against the
oracle under the fp32 tolerances of tests/parity.py (selection bit-exact)."""
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
    ((31, 32, 33), 1, 1, 8, 2),          # fewer keys than one subtile; row counts around 32
    ((127, 129, 0, 1), 3, 3, 32, 3),     # one subtile per block: three waves idle
    ((500,), 6, 2, 33, 4),               # groups of 3: rows of a token straddle work-groups
    ((400,), 64, 1, 129, 2),             # 64 heads of one token over two work-groups
    ((700, 90), 4, 1, 160, 3),           # five subtiles: the first wave takes two
    ((2000,), 2, 2, 3, 5),               # blocks of three keys, 667 bins
])
def test_f32_forward_tile_edges(seqlens, hq, hkv, B, topk):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.float32, B, 0.5, B + topk, device=DEV)
    r = parity.moba_parity(q, k, v, cu, B, topk, dtype="f32")
    print("max_abs %.2e lse %.2e" % (r["max_abs"], r["lse_max_abs"]))


@pytest.mark.parametrize("seqlens", [(1,), (33, 128), (385,)])
def test_f32_dense_strided(seqlens):
    """Dense fp32 on views of one fused projection, outputs in a wider buffer."""
    T = sum(seqlens)
    q, k, v, cu = inputs.make(seqlens, 4, 2, 128, torch.float32, 64, 0.0, T, device=DEV)
    qkv = torch.cat([q, k, v], dim=1)
    out = torch.zeros((T, 5, 128), device=DEV)[:, 1:]
    lse = torch.empty((4, T), device=DEV)
    binding.dense_forward(qkv[:, :4], qkv[:, 4:6], qkv[:, 6:], cu, out=out, lse=lse)
    ref, rlse = binding.dense_forward(q, k, v, cu)
    assert torch.equal(out, ref) and torch.equal(lse, rlse)
    parity.dense_parity(q, k, v, cu, dtype="f32")
