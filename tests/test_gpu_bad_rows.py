"""A query row whose gate scores are not finite (NaN, or all -inf) keeps no past block
in the prefill, so fewer selections are routed than planned.  Its own results are
undefined; every other row's forward, dQ and decode are the ones it has without the
bad row."""
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


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk,bad", [
    ((1500,), 2, 2, 64, 3, [(300, 0), (301, 0), (200, 1)]),    # chunk of 1024 tokens: 16 blocks
    ((600, 500), 8, 2, 64, 3, [(255, 5), (256, 0), (900, 7)]),  # 256 tokens, 4 blocks
    ((700,), 6, 2, 16, 8, [(140, 1), (143, 1), (699, 5)]),     # groups of 3
])
@pytest.mark.parametrize("kind", ["nan", "-inf"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_small_batch(seqlens, hq, hkv, B, topk, bad, kind, dtype):
    """The gate's own counts and the scanning scatter: the other rows against the clean
    run (fp32: bit for bit), and all of them bit for bit against the count and scan
    kernels (the same batch with a filler sequence that brings it past 1024 bins)."""
    T, fill = sum(seqlens), 1040 * B
    q, qb, k, v, cu = bad_inputs(seqlens + (fill,), hq, hkv, B, bad, kind, dtype, T)
    ok = other_rows(q[:T], bad)
    cus = cu[:-1].contiguous()
    ref, rlse = binding.forward(q[:T], k[:T], v[:T], cus, B, topk)
    big, blse = binding.forward(qb, k, v, cu, B, topk)
    out, lse = binding.forward(qb[:T], k[:T], v[:T], cus, B, topk)
    assert torch.equal(out[ok], big[:T][ok]) and torch.equal(lse.T[ok], blse.T[:T][ok])
    if dtype == torch.float32:
        assert torch.equal(out[ok], ref[ok]) and torch.equal(lse.T[ok], rlse.T[ok])
        return
    close(out, ref, ok)
    close(lse.T, rlse.T, ok)
    dout = inputs.make_dout(q.shape, dtype, T, device=DEV)
    rdq = binding.backward(q[:T], k[:T], v[:T], cus, B, topk, ref, rlse, dout[:T])[0]
    bdq = binding.backward(qb, k, v, cu, B, topk, big, blse, dout)[0]
    dq, dk, dv = binding.backward(qb[:T], k[:T], v[:T], cus, B, topk, out, lse, dout[:T])
    assert torch.equal(dq[ok], bdq[:T][ok])
    close(dq, rdq, ok)
    # keys outside the bad rows' own blocks do not see them
    reach = torch.ones((T, hkv), dtype=torch.bool, device=DEV)
    for t, h in bad:
        s0 = max(int(c) for c in cus if int(c) <= t)
        b0 = s0 + (t - s0) // B * B
        reach[b0:b0 + B, h // (hq // hkv)] = False
    assert torch.isfinite(dk[reach].float()).all() and torch.isfinite(dv[reach].float()).all()


@pytest.mark.parametrize("seqlens,hq,hkv,B,topk", [
    ((3000, 700, 900), 4, 2, 16, 3),     # 187 blocks: selection by rank
    ((20000, 300, 5000), 8, 2, 16, 5),   # 1249 blocks: by argmax rounds
])
@pytest.mark.parametrize("noalloc", [False, True])
def test_decode(seqlens, hq, hkv, B, topk, noalloc):
    """A bad row keeps as many blocks as any: more would overwrite other rows'
    selections.  Every other (sequence, head) of the batch keeps its bits."""
    q, k, v, cu = inputs.make(seqlens, hq, hkv, 128, torch.bfloat16, B, 0.5, 3, device=DEV)
    qd = q[(cu[1:] - 1).to(torch.int64).to(DEV)].contiguous()
    bad = [(0, 1), (1, hq - 1)]
    qb = qd.clone()
    for s, h in bad:
        qb[s, h] = float("nan")
    kbar = binding.pool(k, cu, B)

    def run(x):
        if not noalloc:
            return binding.decode(x, k, v, cu, B, topk, kbar=kbar)
        return binding.decode_noalloc(x, k, v, cu, B, topk, torch.empty_like(x),
                                      torch.empty((hq, len(seqlens)), device=DEV), kbar=kbar)

    ref, rlse = run(qd)
    out, lse = run(qb)
    ok = other_rows(qd, bad)
    assert torch.equal(out[ok], ref[ok]) and torch.equal(lse.T[ok], rlse.T[ok])
    assert torch.isnan(out[~ok].float()).all()
