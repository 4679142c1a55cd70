"""The many-row GEMM (more than 64 rows per launch) at the edges of its tiles.

A batched verify of n sequences x (gamma + 1) rows runs every projection and the LM head on the many-row kernel; the
same blocks verified one sequence at a time (at most 64 rows) run on the 33-row kernels, whose parity with the oracle
is tested elsewhere.  Row counts sit at and around the tiles' edges (16-row tiles, 128- to 320-row blocks, several
row blocks), on narrow models (few tiles: K split, heads of 64 and of 128, column groups of 4 and 8 tiles, odd group
counts) and at the Qwen3-32B width (every tile shape).

Bar: both sides are BF16 forwards of one model that differ in the order of their fp32 sums, so each logit row is within
the BF16 parity bar of the other: max |z - z'| <= 2e-2 max |z'|.
"""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import row_tol_ok, to_dev_i32

pytestmark = pytest.mark.gpu

TOL = 2e-2
HD64 = W.ModelShape(2, 320, 5, 5, 64, 672, 1056, 1e-6, 1e6, True, "bf16")     # groups of 4 and 2 tiles, an odd LM head
HD128 = W.ModelShape(2, 384, 6, 2, 128, 1088, 2176, 1e-6, 1e6, True, "bf16")  # 17 gate/up and 17 LM-head groups of 8
GQA64 = W.ModelShape(1, 512, 8, 2, 64, 1024, 4224, 1e-6, 1e6, False, "bf16")


@pytest.fixture(scope="module")
def S():
    from paper_2608_14787_amd import sdd
    assert sdd.device_ok(), "needs a gfx950 device"
    return sdd


def _run(S, m, shape, n, R, seed):
    lens = W.rng(seed).integers(3, 60, size=n)
    gamma = R - 1
    kv = S.KVCache(m, n, 64 + R)
    ws, ws1 = m.workspace(n * R), m.workspace(64)
    for s in range(n):
        kv.prefill(s, to_dev_i32(W.prompt(seed + s, int(lens[s]), shape.vocab)), ws1)
    drafts = to_dev_i32(W.prompt(seed + 500, n * gamma, shape.vocab).reshape(n, gamma)) if gamma else \
        torch.empty((n, 0), dtype=torch.int32, device="cuda")
    lb = torch.full((n, R, shape.vocab), float("nan"), device="cuda")
    am = torch.full((n, R), -7, dtype=torch.int32, device="cuda")
    kv.verify(to_dev_i32(np.arange(n)), drafts, lb, am, ws)
    assert torch.equal(am.long(), lb.argmax(-1)), "argmax is the first index of the row's maximum"
    lb2 = torch.empty_like(lb)
    kv.verify(to_dev_i32(np.arange(n)), drafts, lb2, None, ws)
    assert torch.equal(lb, lb2), "repeated call (arrival counters left at zero, same bits)"
    l1 = torch.empty((1, R, shape.vocab), device="cuda")
    worst = 0.0
    for s in range(n):
        kv.verify(to_dev_i32([s]), drafts[s:s + 1].contiguous(), l1, None, ws1)
        ok, rel = row_tol_ok(lb[s].cpu().numpy(), l1[0].cpu().numpy(), TOL)
        worst = max(worst, float(rel.max()))
        assert ok.all(), (n, R, s, rel.max())
    assert kv.state()[2] == 0
    print(f"{n} x {R} rows: max rel {worst:.2e}", flush=True)


@pytest.mark.parametrize("shape", [HD64, HD128, GQA64], ids=["hd64", "hd128", "gqa64"])
@pytest.mark.parametrize("n,R", [(5, 13), (2, 40), (3, 43), (8, 32), (9, 29), (7, 55), (17, 61)])
def test_batched_equals_single_narrow(S, shape, n, R):
    m = S.Model(shape)
    m.init_random(3, W.WEIGHT_SIGMA)
    _run(S, m, shape, n, R, seed=700 + n)


def test_batched_equals_single_full_width(S):
    """65 to 1040 rows at the Qwen3-32B width: every tile shape, split and unsplit."""
    shape = W.QWEN32B.with_layers(1)
    m = S.Model(shape)
    m.init_random(4, W.WEIGHT_SIGMA)
    for n, R in ((5, 13), (4, 33), (6, 32), (8, 33), (10, 33), (8, 64), (26, 40)):
        _run(S, m, shape, n, R, seed=800 + n)


@pytest.mark.parametrize("rows", [16, 64, 256, 2048])
def test_prefill_chunks(S, rows):
    """A prompt prefilled through workspaces of every size gives the same next block (one chunk or several,
    chunks of at most 64 rows)."""
    m = S.Model(HD128)
    m.init_random(5, W.WEIGHT_SIGMA)
    n, R = 1333, 9
    toks = to_dev_i32(W.prompt(9, n, HD128.vocab))
    drafts = to_dev_i32(W.prompt(10, R - 1, HD128.vocab).reshape(1, R - 1))
    out = []
    for r in (rows, 128):
        kv, ws = S.KVCache(m, 1, n + R), m.workspace(r)
        kv.prefill(0, toks, ws)
        lg = torch.empty((1, R, HD128.vocab), device="cuda")
        kv.verify(to_dev_i32([0]), drafts, lg, None, ws)
        assert kv.state()[2] == 0
        out.append(lg[0].cpu().numpy())
    ok, rel = row_tol_ok(out[0], out[1], TOL)
    print(f"{rows}: {rel.max():.2e}", flush=True)
    assert ok.all(), rel.max()


@pytest.mark.parametrize("n,R", [(3, 33), (5, 33), (16, 64)])
def test_whole_rounds_then_split(S, n, R):
    """A vocabulary of 9496 16-column tiles: the LM head's column blocks (the last one only half inside the matrix) fill every
    compute unit twice or more, with 2, 3 and 4 row tiles per wave, and about half of them hold a segment's end."""
    shape = W.ModelShape(1, 4096, 4, 2, 128, 1024, 151936, 1e-6, 1e6, False, "bf16")
    m = S.Model(shape)
    m.init_random(7, W.WEIGHT_SIGMA)
    _run(S, m, shape, n, R, seed=900 + n)


def test_whole_rounds_then_split_prefill(S):
    """A 3000-row chunk at the Qwen3-32B width (a workgroup per tile, walking its segments) gives the next block that passes of
    64 rows give."""
    shape = W.QWEN32B.with_layers(2)
    m = S.Model(shape)
    m.init_random(8, W.WEIGHT_SIGMA)
    n, R = 3001, 9
    toks = to_dev_i32(W.prompt(11, n, shape.vocab))
    drafts = to_dev_i32(W.prompt(12, R - 1, shape.vocab).reshape(1, R - 1))
    out = []
    for rows in (4096, 99):
        kv, ws = S.KVCache(m, 1, n + R), m.workspace(rows)
        kv.prefill(0, toks, ws)
        lg = torch.empty((1, R, shape.vocab), device="cuda")
        kv.verify(to_dev_i32([0]), drafts, lg, None, ws)
        assert kv.state()[2] == 0
        out.append(lg[0].cpu().numpy())
    ok, rel = row_tol_ok(out[0], out[1], TOL)
    print(f"max rel {rel.max():.2e}", flush=True)
    assert ok.all(), rel.max()
