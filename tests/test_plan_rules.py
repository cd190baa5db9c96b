"""bench.py credits each launch with the keys it attends, so it repeats the library's rules
for rows that are not routed; here they are compared with those rules themselves
(csrc/plan_rules.h, compiled for the host), on both sides of their lines."""
import ctypes
import os
import random
import subprocess

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "plan_rules.h"
extern "C" int head_blocks(long long L, int hq, int B, int topk) {
  return moba::head_blocks(L, hq, B, topk);
}
extern "C" int bwd_head_blocks(int hq, int B, int topk) {
  return moba::bwd_head_blocks(hq, B, topk);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2502_13189_amd", "csrc"), str(d / "shim.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.head_blocks.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return lib


def split(lib, seqlens, B, topk, hq):
    """(causal, routed) keys per query head, block by block."""
    causal = routed = 0
    for L in seqlens:
        head = lib.head_blocks(L, hq, B, topk)
        for c in range(-(-L // B)):
            m = min(L, (c + 1) * B) - c * B
            causal += m * (m + 1) // 2
            past = m * B * min(topk - 1, c)
            if c < head:
                causal += past
            else:
                routed += past
    return causal, routed


def test_launch_keys(rules):
    rng = random.Random(3)
    heads = set()
    for _ in range(400):
        B = rng.choice((1, 16, 100, 256, 1000, 4096))
        topk = rng.choice((1, 2, 3, 4, 8, 12, 32))
        hq = rng.choice((1, 4, 8, 32, 128))
        seqlens = [rng.randrange(0, 40 * B) for _ in range(rng.randrange(1, 4))]
        heads |= {rules.head_blocks(L, hq, B, topk) > 1 for L in seqlens if topk > 1}
        assert bench.launch_keys(seqlens, B, topk, hq) == split(rules, seqlens, B, topk, hq)
    assert heads == {False, True}


def test_backward_rule(rules):
    seen = set()
    for hq in (1, 8, 12, 16, 32, 64, 128):
        for B in (1, 64, 512, 700, 1024, 2048, 4096, 4600, 8192):
            for topk in (1, 2, 3, 4, 5, 8, 12, 16, 32, 64):
                want = bool(rules.bwd_head_blocks(hq, B, topk))
                assert bench.backward_takes_heads(hq, B, topk) == want
                seen.add(want)
    assert seen == {False, True}
