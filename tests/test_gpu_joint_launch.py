"""History and current-block tiles in one launch of 128-row work-groups (blocks of
up to 2048 keys): tile remainders, groups whose 256-row plan tile splits unevenly,
waves without a key in a causal tile's last key tiles, no history at all."""
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


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((127, 129, 257), 1, 1, 64, 2),     # MHA row counts around 128 and 256
    ((700,), 3, 1, 300, 2),             # groups of 3: 85 tokens (255 rows) per plan tile
    ((190,), 100, 1, 50, 2),            # 2 tokens (200 rows): the second half holds 72
    ((600, 1), 2, 2, 2, 3),             # two-key blocks: many bins of few rows
    ((900,), 2, 1, 256, 1),             # top-1: causal tiles only
    ((4300,), 1, 1, 2048, 2),           # the longest blocks of the joint launch
    ((4200,), 1, 1, 2049, 2),           # and the first beyond it
    ((500,), 16, 2, 16, 3),             # 128 rows per block: one work-group each
    ((500,), 16, 2, 17, 3),             # 136 rows: two
])
def test_joint_tiles(seqlens, hq, hkv, B, topk):
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, B, device=DEV)
    r = parity.moba_parity(q, k, v, cu, B, topk, dtype="bf16")
    print("max_abs %.2e lse %.2e" % (r["max_abs"], r["lse_max_abs"]))


def test_smallest_workspace(monkeypatch):
    """Down to the smallest cap that is accepted, where the list of 128-row history tiles
    no longer fits and the two launches of 256-row ones run: the same bits."""
    q, k, v, cu = inputs.make((3000, 1500), 4, 2, 128, torch.bfloat16, 32, 0.5, 3, device=DEV)
    ref, rlse = binding.forward(q, k, v, cu, 32, 12)
    torch.cuda.synchronize()
    binding.release_workspace()

    def run(limit):
        monkeypatch.setenv("MOBA_WORKSPACE_LIMIT_BYTES", str(limit))
        try:
            return binding.forward(q, k, v, cu, 32, 12)
        except binding.MobaError as e:
            assert e.name == "MOBA_ERR_NO_MEMORY"
            return None

    lo, hi = 0, binding.workspace_bytes(4500, 4, 2, binding.num_blocks(cu, 32), 12)
    assert run(hi) is not None
    while hi - lo > 256:
        mid = (lo + hi) // 2
        if run(mid) is None:
            lo = mid
        else:
            hi = mid
    for limit in (hi, hi + 2048, hi + 8192, hi + 65536):
        out, lse = run(limit)
        assert torch.equal(out, ref) and torch.equal(lse, rlse)


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((8192, 8197), 32, 2, 16, 12),     # one key tile per history tile
    ((6000, 5, 11000), 32, 2, 48, 12),  # blocks across two key tiles
    ((14000, 14900), 32, 2, 100, 8),
])
def test_persistent_history(seqlens, hq, hkv, B, topk):
    """Batches large enough for the persistent history kernel; alone, their sequences
    are not: the same bits."""
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, B, device=DEV)
    entries = [binding.route_size(inputs.cu_seqlens((L,)), B, topk, hq)[1] for L in seqlens]
    assert sum(entries) >= 64 * 256 * 256 * 1.1 > 1.1 * max(entries)
    out, lse = binding.forward(q, k, v, cu, B, topk)
    for s, L in enumerate(seqlens):
        a, b = int(cu[s]), int(cu[s + 1])
        o, l = binding.forward(q[a:b], k[a:b], v[a:b], inputs.cu_seqlens((L,)), B, topk)
        assert torch.equal(o, out[a:b]) and torch.equal(l, lse[:, a:b])
