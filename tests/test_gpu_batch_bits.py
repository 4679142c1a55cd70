"""A row's result does not depend on the launch it is computed in, bit for bit (bf16, more than 64 rows a call).

The many-row GEMM adds a row's products in an order fixed by the matrix (gemm.h: SumPlan) whatever tiles, splits and
launches its row count is planned into, and the prefill attention kernel does the block kernel's operations.  So, compared
exactly: a sequence's logits do not depend on the other sequences of the call, a prompt's cached K/V do not depend on the
chunks (on the workspace's size, where it holds passes of 256 rows), and a prompt's last rows cached by the prefill equal
the same rows cached by a verify call.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import to_dev_i32

pytestmark = pytest.mark.gpu

# 128- and 64-wide heads, groups of 8 and 4 tiles, from one segment per k-step to several k-steps per segment
SHAPES = {"hd128": W.ModelShape(2, 384, 6, 2, 128, 1088, 2176, 1e-6, 1e6, True, "bf16"),
          "hd64": W.ModelShape(2, 320, 5, 5, 64, 672, 1056, 1e-6, 1e6, True, "bf16"),
          "gqa64": W.ModelShape(2, 512, 8, 2, 64, 1024, 4224, 1e-6, 1e6, False, "bf16"),
          "qwen32b": W.QWEN32B.with_layers(2), "qwen7b": W.QWEN7B.with_layers(2)}


@pytest.fixture(scope="module", params=list(SHAPES))
def model(request):
    from paper_2608_14787_amd import sdd as S
    m = S.Model(SHAPES[request.param])
    m.init_random(11, W.WEIGHT_SIGMA)
    return S, m, SHAPES[request.param]


HDR = 256  # a one-sequence cache's length, pending token and error word; the rotation table and K/V follow


def _cache(S, m, shape, n):
    """A cache of n positions whose K/V start as zeros (rows past the last one differ otherwise)."""
    kv = S.KVCache(m, 1, n)
    kv.buf[HDR + -(-n * shape.head_dim * 4 // 256) * 256:].zero_()
    return kv


def _verify(S, m, V, kv, seqs, drafts, ws):
    lg = torch.full((len(seqs), drafts.shape[1] + 1, V), float("nan"), device="cuda")
    kv.verify(to_dev_i32(seqs), drafts[seqs].contiguous(), lg, None, ws)
    return lg


def test_logits_do_not_depend_on_the_other_sequences(model):
    S, m, shape = model
    n, R = 8, 33
    kv, ws, ws1 = S.KVCache(m, n, 128), m.workspace(n * R), m.workspace(64)
    for s in range(n):
        kv.prefill(s, to_dev_i32(W.prompt(s, 5 + 7 * s, shape.vocab)), ws1)
    drafts = to_dev_i32(W.prompt(50, n * (R - 1), shape.vocab).reshape(n, R - 1))
    want = _verify(S, m, shape.vocab, kv, list(range(n)), drafts, ws)
    for seqs in ([0, 1], [6, 2, 4], [7, 5, 3, 1, 0], [1, 2, 3, 4, 5, 6, 7]):  # 66, 99, 165 and 231 rows
        got = _verify(S, m, shape.vocab, kv, seqs, drafts, ws)
        assert torch.equal(got, want[seqs]), (shape, seqs)
    assert kv.state()[2] == 0


def test_prompts_do_not_depend_on_the_workspace(model):
    S, m, shape = model
    for n in (66, 300, 1000, 1333, 2400):  # 1333: 1280 rows and 53
        caches = []
        for rows in (256, 512, 4096):
            kv, ws = _cache(S, m, shape, n), m.workspace(rows)
            kv.prefill(0, to_dev_i32(W.prompt(n, n + 1, shape.vocab)), ws)
            caches.append(kv.buf[HDR:].clone())
        assert torch.equal(caches[0], caches[1]) and torch.equal(caches[0], caches[2]), (shape, n)


@pytest.mark.parametrize("n", [65, 512, 1024, 1601])
def test_prefill_equals_verify(model, n):
    """Rows n - 65 .. n - 1 cached by the prefill of n rows (many-row GEMMs, prefill attention) and by a verify call of 65
    rows (many-row GEMMs, block attention) after a prefill of the n - 65 before them; n and n - 65 leave no pass of at
    most 64 rows (other GEMM kernels) over whole passes of 256."""
    S, m, shape = model
    assert all(r == 0 or r % 256 == 0 or r % 256 > 64 for r in (n, n - 65))
    toks = W.prompt(n, n + 1, shape.vocab)
    ws = m.workspace(512)
    ka, kb = _cache(S, m, shape, n), _cache(S, m, shape, n)
    ka.prefill(0, to_dev_i32(toks), ws)
    kb.prefill(0, to_dev_i32(toks[:n - 64]), ws)  # caches n - 65 rows, the next token pending
    lg = torch.empty((1, 65, shape.vocab), device="cuda")
    kb.verify(to_dev_i32([0]), to_dev_i32(toks[n - 64:n].reshape(1, 64)), lg, None, ws)
    assert ka.state()[2] == 0 and kb.state()[2] == 0
    assert torch.equal(ka.buf[HDR:], kb.buf[HDR:]), (shape, n)
