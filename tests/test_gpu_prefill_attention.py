"""The prefill attention kernel (chunks of more than 64 rows) against the block kernel.

A prompt prefilled in one or two large chunks runs the prefill kernel; the same prompt through a 16-row workspace runs in
chunks of at most 16 rows on the block kernel, whose parity with the oracle is tested elsewhere.  The next block's
logits read every cached K/V row.  Prompt lengths sit at and around the edges of the 48-query workgroups, 16-query
tiles, 32-position steps and the steps' rounds over the 8 waves; head counts cover every spread of KV heads over the XCDs
(8, 4, 3 and 40 KV heads) and query groups of 8, 7, 16 and 1 (tiles that split a row's heads).

Bar: both sides are BF16 forwards of one model that differ in the order of their GEMMs' fp32 sums, so each logit row is
within the BF16 parity bar of the other: max |z - z'| <= 2e-2 max |z'|.  (test_gpu_batch_bits.py compares the two kernels
behind the same GEMMs, bit for bit.)
"""
import pytest
import torch

import workloads as W
from gpu_helpers import row_tol_ok, to_dev_i32

pytestmark = pytest.mark.gpu

SHAPES = {"64/8x128": W.ModelShape(2, 256, 64, 8, 128, 512, 1056, 1e-6, 1e6, True, "bf16"),
          "28/4x128": W.ModelShape(2, 256, 28, 4, 128, 512, 1056, 1e-6, 1e6, False, "bf16"),
          "48/3x64": W.ModelShape(2, 256, 48, 3, 64, 512, 1056, 1e-6, 1e6, True, "bf16"),
          "40/40x64": W.ModelShape(2, 256, 40, 40, 64, 512, 1056, 1e-6, 1e6, False, "bf16")}


@pytest.mark.parametrize("name", list(SHAPES))
def test_prefill_attention_matches_block_attention(name):
    from paper_2608_14787_amd import sdd as S
    shape, R = SHAPES[name], 9
    m = S.Model(shape)
    m.init_random(6, W.WEIGHT_SIGMA)
    ws_small, ws_large = m.workspace(16), m.workspace(4096)
    for n in (66, 67, 97, 128, 129, 161, 255, 1023, 1601, 4613):  # n cached rows (4613: two chunks)
        toks = to_dev_i32(W.prompt(n, n + 1, shape.vocab))
        drafts = to_dev_i32(W.prompt(n + 1, R - 1, shape.vocab).reshape(1, R - 1))
        out = []
        for ws in (ws_large, ws_small):
            kv = S.KVCache(m, 1, n + R)
            kv.prefill(0, toks, ws)
            lg = torch.empty((1, R, shape.vocab), device="cuda")
            kv.verify(to_dev_i32([0]), drafts, lg, None, ws_small)
            assert kv.state()[2] == 0
            out.append(lg[0].cpu().numpy())
        ok, rel = row_tol_ok(out[0], out[1], 2e-2)
        print(f"{name} {n} rows: max rel {rel.max():.2e}", flush=True)
        assert ok.all(), (n, rel.max())
