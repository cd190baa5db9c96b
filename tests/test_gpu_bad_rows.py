"""A query row whose gate scores are not finite (NaN, or all -inf) keeps no past block,
so fewer selections are routed than planned.  Its own results are undefined; every
other row's forward and dQ are the ones it has without the bad row."""
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


def bad_inputs(seqlens, hq, hkv, B, bad, kind, dtype, seed):
    """(clean q, q with the bad rows, k, v, cu): rows (t, h) of `bad` all NaN, or with
    scores of -inf in every block (dim 0 of every key is 2, theirs -3e38)."""
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, dtype, B, 0.5, seed, device=DEV)
    qb = q.clone()
    if kind == "-inf":
        k[:, :, 0] = 2.0
    for t, h in bad:
        if kind == "-inf":
            qb[t, h] = 0.0
            qb[t, h, 0] = -3.0e38
        else:
            qb[t, h] = float("nan")
    return q, qb, k, v, cu


def other_rows(q, bad):
    ok = torch.ones(q.shape[:2], dtype=torch.bool, device=DEV)
    for t, h in bad:
        ok[t, h] = False
    return ok


def close(x, y, ok):
    """The other rows of two runs: bf16 roundings may fall differently (2^-8 of a value;
    a softmax tile's running max is raised for all rows of a wave together)."""
    x, y = x[ok].double(), y[ok].double()
    assert torch.isfinite(x).all()
    assert (x - y).norm() <= 2.0 ** -8 * y.norm()


@pytest.mark.parametrize("kind", ["nan", "-inf"])
def test_large_batch(kind):
    """Past 1024 bins: the count and scan kernels, then the backward's row records."""
    seqlens, hq, hkv, B, topk = (900, 17000), 2, 2, 16, 3
    bad = [(200, 0), (201, 1), (899, 1), (3000, 0), (17899, 1)]
    q, qb, k, v, cu = bad_inputs(seqlens, hq, hkv, B, bad, kind, torch.bfloat16, 1)
    dout = inputs.make_dout(q.shape, q.dtype, 1, device=DEV)
    ok = other_rows(q, bad)
    ref, rlse = binding.forward(q, k, v, cu, B, topk)
    rdq = binding.backward(q, k, v, cu, B, topk, ref, rlse, dout)[0]
    out, lse = binding.forward(qb, k, v, cu, B, topk)
    dq = binding.backward(qb, k, v, cu, B, topk, out, lse, dout)[0]
    close(out, ref, ok)
    close(lse.T, rlse.T, ok)
    close(dq, rdq, ok)
