"""Decode at the edges of its tiles: 16-key matrix tiles, 64 keys per wave, 256-key
chunks, groups that fill part of the 16 head columns, chunk lists of sequences of very
different lengths, gate passes of 256 blocks and both selection methods.  Against
the oracle; rows with near-tied gate scores over every admissible selection."""
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


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((1, 15, 16, 17, 63, 64, 65), 3, 1, 16, 3),
    ((255, 1, 256, 257, 513), 10, 2, 48, 4),      # groups of 5
    ((5000, 2), 16, 1, 300, 3),                   # all 16 head columns; chunks end inside blocks
    ((2100,), 2, 2, 8, 9),                        # 263 blocks: a second gate pass
    ((2060, 300), 1, 1, 2, 12),                   # 1030 blocks: selection by argmax rounds
    ((513, 521, 1025, 1033, 2571), 2, 1, 8, 5),   # 64, 65, 128, 129, 321 past blocks: passes of 64 to 256
    ((17000,), 8, 1, 64, 64),                     # one combine share of 64 slots
    # full attention's two orders: 75 and 77 chunks of 32 kv-heads, either side of the line
    ((7,) * 75, 32, 32, 16, 3),
    ((7,) * 70 + (1300, 40), 32, 32, 16, 3),
])
@pytest.mark.parametrize("mode", ["moba", "full"])
def test_decode_tiles(seqlens, hq, hkv, B, topk, mode):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, B + topk, device=DEV)
    T, S = q.shape[0], len(seqlens)
    last = (cu[1:] - 1).to(torch.int64)
    qd = q[last.to(DEV)].contiguous()
    # the cache as a view of a wider buffer, as a layer's slice of a cache is
    kv = torch.cat([k, v, k], dim=1)
    out, lse = binding.decode(qd, kv[:, :hkv], kv[:, hkv:2 * hkv], cu, B,
                              0 if mode == "full" else topk, kbar=binding.pool(k, cu, B))
    torch.cuda.synchronize()
    rows = np.array([int(t) * hq + h for t in last for h in range(hq)], np.int64)
    q_rows = inputs.to_oracle(qd.reshape(S * hq, 128))
    kn, vn, cun = inputs.to_oracle(k), inputs.to_oracle(v), cu.numpy()
    gout = out.float().cpu().numpy().reshape(S * hq, 128)
    glse = lse.cpu().numpy().T.reshape(S * hq)
    if mode == "full":
        oout, olse = oracle.attend_rows(q_rows, T, hq, kn, vn, cun, max(seqlens),
                                        np.zeros((len(rows), 1), np.int32), rows)
        parity.compare_outputs(gout, glse, oout, olse, "bf16", mode)
    else:
        parity.check_rows_any_selection(gout, glse, q_rows, rows, T, hq, kn, vn, cun, B, topk, mode)
