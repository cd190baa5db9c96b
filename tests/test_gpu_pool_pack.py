"""Block means at the edges of their reading loop (64 rows at a time, four loads
ahead) and packed tiles at sequence ends, in the launch that does both."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2502_13189_amd import binding, inputs
import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()


@pytest.mark.parametrize("B", [1, 63, 64, 65, 255, 256, 257, 448, 449, 1000])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_block_means(B, dtype):
    seqlens = (B, 0, 2 * B + 1, max(1, B - 1))
    q, k, v, cu = inputs.make(seqlens, 2, 2, 128, dtype, B, 0.5, B, device=DEV)
    kbar = binding.pool(k, cu, B).cpu().numpy().astype(np.float64)
    ref, kabs = oracle.pool(inputs.to_oracle(k), cu.numpy(), B, with_abs=True)
    # fp64 accumulation rounded once to fp32: within one fp32 ulp of the mean
    assert np.all(np.abs(kbar - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12 * kabs)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,n", [(128, 3), (129, 3), (129, 32), (129, 33), (1100, 255), (1100, 256)])
def test_block_means_of_both_sizes(B, n, dtype):
    """Either side of the line between the two work-group sizes (B = 128; pairs of 8
    kv-heads and n blocks at twice B and at 2048), a short last block."""
    T = n * B - 5
    _, k, _, cu = inputs.make((T,), 8, 8, 128, dtype, B, 0.5, B + n, device=DEV)
    kbar = binding.pool(k, cu, B).cpu().numpy().astype(np.float64)
    ref, kabs = oracle.pool(inputs.to_oracle(k), cu.numpy(), B, with_abs=True)
    assert np.all(np.abs(kbar - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12 * kabs)


@pytest.mark.parametrize("seqlens", [(1,), (63, 65), (64, 0, 128, 1), (257, 191)])
def test_packed_tiles(seqlens):
    """1 to 4 tiles in the last work-group of four; V beyond a sequence's end is the
    next one's and must not leak in."""
    q, k, v, cu = inputs.make(seqlens, 2, 1, 128, torch.bfloat16, 64, 0.5, 3, device=DEV)
    parity.dense_parity(q, k, v, cu, dtype="bf16")
    if max(seqlens) > 128:
        parity.moba_parity(q, k, v, cu, 64, 2, dtype="bf16")
